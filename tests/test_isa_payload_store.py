"""CPU check in the gfx950 assembly of where the BF16-payload round stores the
received mean: no store of theta or the momentum comes after a wait that the
mean's store is part of.

A wait for a load counts every vector memory instruction issued since, stores
included.  With the mean stored first, the wait for the momentum's load, the last
of a window, also waited for that store to complete before the window's other
stores went out."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_36662_amd", "csrc")
INCLUDE = os.path.join(ROOT, "include")

# (replicas, bf16 replicas, fused with statistics and reset or the plain update)
KERNELS = [(k, 0, 1) for k in (1, 2, 3, 4, 7, 8)] + [(k, 1, 0) for k in (7, 8, 9, 10, 16)]


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    return None


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    hipcc = _hipcc()
    if hipcc is None:
        pytest.skip("hipcc not available")
    tmp = tmp_path_factory.mktemp("isa_payload")
    src, out = tmp / "payload.hip", tmp / "payload.s"
    src.write_text('#include "round_kernels.hpp"\nnamespace autoloco {\n' + "".join(
        f"template __global__ void round_kernel<{k}, {('RT_F32', 'RT_BF16')[bf]}, {('false', 'true')[fu]}, true, "
        f"{('false', 'true')[fu]}, true>(RoundArgs);\n" for k, bf, fu in KERNELS) + "}\n")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", f"-I{INCLUDE}", f"-I{CSRC}", "--cuda-device-only", "-S", str(src), "-o", str(out)]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-3000:]
    return out.read_text()


def _waited_stores(lines, label, at):
    """Stores of 16 bytes a lane reached from instruction `at` after a vector-memory
    wait, with no load between, along any path."""
    todo, seen, found = [(at + 1, False)], set(), []
    while todo:
        i, waited = todo.pop()
        if (i, waited) in seen or i >= len(lines):
            continue
        seen.add((i, waited))
        line = lines[i].split(";")[0].strip()
        if line.startswith(("global_load", "s_endpgm")):
            continue
        if line.startswith("global_store_dwordx4") and waited:
            found.append(line)
            continue
        waited = waited or (line.startswith("s_waitcnt") and "vmcnt(" in line)
        m = re.match(r"s_(c?)branch\w*\s+(\.LBB\d+_\d+)", line)
        if m:
            todo.append((label[m.group(2)], waited))
        if not m or m.group(1):
            todo.append((i + 1, waited))
    return found


@pytest.mark.parametrize("k,bf,fused", KERNELS)
def test_no_store_waits_for_the_means(asm, k, bf, fused):
    symbol = f"_ZN8autoloco12round_kernelILi{k}ELi{bf}ELb{fused}ELb1ELb{fused}ELb1EEEvNS_9RoundArgsE"
    start = asm.index("\n" + symbol + ":")
    lines = asm[start:asm.index(".Lfunc_end", start)].split("\n")
    label = {l.split(":")[0]: i for i, l in enumerate(lines) if l.startswith(".LBB")}
    # 8 bytes a lane: the mean (with fp32 replicas, or without the reset, nothing else but the sums at the end)
    stores = [i for i, l in enumerate(lines) if l.strip().startswith("global_store_dwordx2")]
    assert stores, symbol
    for i in stores:
        assert not _waited_stores(lines, label, i), (symbol, lines[i].strip())
