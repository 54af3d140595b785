"""CPU test of the reductions' second stage on the host against a lane-by-lane
model of the kernel it stands for, bit for bit: thread t of nt adds the
workgroups t, t + nt, ... in that order; every lane then adds the value of its
partner (lane ^ 32, ^ 16, rotated by 8 in its row of 16, 7 - lane in its group of
8, ^ 1, ^ 2); lane 0 has the wavefront's sum, and the wavefronts are added in
order.  Counts below and above a wavefront, a workgroup (the threads wrap) and up to
the most the host takes (1,024 sums), for the round's 256 threads and the INT8
round's 512."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_36662_amd", "csrc")


@pytest.fixture(scope="module")
def finish(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    tmp = tmp_path_factory.mktemp("host_sums")
    src, lib = tmp / "host_sums.cpp", tmp / "host_sums.so"
    src.write_text('#include "host_sums.hpp"\nextern "C" void finish(const double* p, int ns, int nt, int nb, double* s) '
                   "{ autoloco::host_finish_sums(p, ns, nt, nb, s); }\n")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o",
                    str(lib)], check=True)
    f = C.CDLL(str(lib)).finish
    f.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_void_p]
    return f


def _model(partials, nt):
    """One sum's partials [nblocks] as the finishing kernel of nt threads adds them."""
    lane = np.arange(64)
    partner = [lane ^ 32, lane ^ 16, lane & ~15 | (lane + 8) % 16, lane & ~7 | 7 - lane % 8, lane ^ 1, lane ^ 2]
    threads = np.zeros(nt)
    for at in range(0, len(partials), nt):
        row = partials[at:at + nt]
        threads[:len(row)] += row
    total = None
    for w in range(nt // 64):
        x = threads[64 * w:64 * w + 64].copy()
        for p in partner:
            x = x + x[p]
        total = x[0] if total is None else total + x[0]
    return total


@pytest.mark.parametrize("nt", [256, 512])
@pytest.mark.parametrize("ns", [1, 3, 5, 33])
def test_equals_the_kernels_order(finish, ns, nt):
    rng = np.random.default_rng(ns + nt)
    most = 1024 // ns
    for nb in sorted({1, 2, 7, 8, 31, 63, 64, 65, 129, 255, 256, 257, 300, 341, 511, 512, 513, 700, most}):
        if nb > most:
            continue
        p = rng.standard_normal((ns, nb)) * 10.0 ** rng.integers(-6, 7, (ns, nb))
        p = np.ascontiguousarray(p)
        s = np.empty(ns)
        finish(p.ctypes.data, ns, nt, nb, s.ctypes.data)
        want = np.array([_model(p[j], nt) for j in range(ns)])
        assert np.array_equal(s.view(np.int64), want.view(np.int64)), nb


def test_a_nan_or_infinity_stays_in_its_sum(finish):
    p = np.ones((3, 130))
    p[0, 77], p[2, 3] = np.nan, np.inf
    s = np.empty(3)
    finish(p.ctypes.data, 3, 256, 130, s.ctypes.data)
    assert np.isnan(s[0]) and s[1] == 130.0 and np.isposinf(s[2])
