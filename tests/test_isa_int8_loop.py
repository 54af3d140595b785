"""CPU check of the INT8 round's main loop in the gfx950 assembly, along the path
one iteration takes: for every worker count, replica type and flag subset, the
wait that proves this block's direct global-to-LDS loads have landed (it counts
on the stores issued after them), the LDS reads of a piece returned before the
next block's load overwrites it, the drained prologue, and block barriers that
wait for LDS traffic only and so leave the next block's loads in flight."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_36662_amd", "csrc")
INCLUDE = os.path.join(ROOT, "include")
VARIANTS = [(st, rs) for st in (0, 1) for rs in (0, 1)]


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
    tmp = tmp_path_factory.mktemp("isa")

    def one(v):
        rt, st, rs = v
        name = ("f32", "bf16")[rt]
        out = str(tmp / f"int8_{name}_s{st}r{rs}.s")
        cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", f"-I{INCLUDE}", f"-I{CSRC}", f"-DAL_RT={rt}", f"-DAL_RTNAME={name}",
               f"-DAL_STATS={st}", f"-DAL_RESET={rs}", "--cuda-device-only", "-S", os.path.join(CSRC, "int8_inst.hip"), "-o", out]
        p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert p.returncode == 0, p.stdout[-3000:]
        with open(out) as f:
            return v, f.read()

    todo = [(rt, st, rs) for rt in (0, 1) for st, rs in VARIANTS]
    with ThreadPoolExecutor(len(todo)) as pool:
        return dict(pool.map(one, todo))


def _loop_path(text, name):
    """The instructions of one iteration of a kernel's main loop, in the order they
    run: from the loop header on, conditional branches not taken, jumps followed,
    up to the branch back to the header."""
    body = text[text.index(name + ":"):]
    body = body[:body.index(".Lfunc_end")].split("\n")
    label = {l.split(":")[0]: i for i, l in enumerate(body) if re.match(r"^\.LBB\d+_\d+:", l)}
    i = next(i for i, l in enumerate(body) if l.startswith(".LBB") and "Loop Header" in l)
    head, out, seen = body[i].split(":")[0], [], set()
    i += 1
    while True:
        assert i not in seen, "the path does not come back to the loop header"
        seen.add(i)
        ins = body[i].split(";")[0].strip()
        m = re.match(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", ins)
        if m and m.group(1) == head:
            return body, out
        if m and ins.startswith("s_branch"):
            i = label[m.group(1)]
        else:
            out.append(ins)
            i += 1
        if i < len(body) and body[i].startswith(head + ":"):
            return body, out


@pytest.mark.parametrize("rt", [0, 1])
@pytest.mark.parametrize("st,rs", VARIANTS)
def test_prefetch_waits_on_the_loop_path(asm, rt, st, rs):
    text = asm[(rt, st, rs)]
    for k in range(1, 17):
        name = f"_ZN8autoloco17int8_round_kernelILi{k}ELi{rt}ELb{st}ELb{rs}EEEvNS_8Int8ArgsE"
        body, path = _loop_path(text, name)
        at = [i for i, l in enumerate(path) if l.startswith("global_load_lds")]
        per = 2 + (2 * min(k, 8) if rt == 0 else k)
        assert len(at) == per and all(path[i].endswith(" nt") for i in at), (k, len(at))
        # the wait for the pieces is the first vector-memory wait and comes before any LDS access
        w = next(i for i, l in enumerate(path) if "vmcnt(" in l)
        n = int(re.search(r"vmcnt\((\d+)\)", path[w]).group(1))
        assert n == 2 * (2 + (k if rs else 0)), (k, n)
        assert w < min(i for i, l in enumerate(path) if l.startswith(("ds_", "global_load_lds"))), k
        # at least that many stores (not counting the optional codes' 4-byte ones) follow the last direct load
        stores = sum(1 for l in path[at[-1]:] if re.match(r"global_store_dwordx[24] ", l))
        assert stores >= n, (k, stores, n)
        # one group of direct loads (above 8 workers theta's come later, after its second read); the LDS reads of a piece have returned before its next direct load is issued
        groups = [[at[0]]]
        for a, b in zip(at, at[1:]):
            if any(l.startswith("ds_") for l in path[a:b]):
                groups.append([])
            groups[-1].append(b)
        assert [len(g) for g in groups] == ([per] if k <= 8 else [per - 2, 2]), (k, [len(g) for g in groups])
        for g in groups:
            last = max(i for i in range(g[0]) if path[i].startswith("ds_read"))
            assert any("lgkmcnt(0)" in l for l in path[last:g[0]]), (k, "direct loads over pending LDS reads")
        # the block barriers do not wait for the direct loads
        bars = [i for i, l in enumerate(path) if l.startswith("s_barrier")]
        assert len(bars) == 2, k
        last = groups[0][-1]
        for b in bars:
            assert "lgkmcnt(0)" in path[b - 1] or "lgkmcnt(0)" in path[b - 2], k
            assert not any("vmcnt(0)" in l for l in path[last:b]), k
        # prologue: drained before the loop
        first = next(i for i, l in enumerate(body) if "global_load_lds" in l)
        assert any("s_waitcnt vmcnt(0)" in l for l in body[first:next(
            i for i, l in enumerate(body) if l.startswith(".LBB") and "Loop Header" in l)]), k
