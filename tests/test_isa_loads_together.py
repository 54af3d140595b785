"""CPU check in the gfx950 assembly that a kernel sends all the loads of a window
(every worker's vector, and theta's and the momentum's where it has them) before
it waits for the first of them.

Where nothing holds a window's loads together, the compiler moves some of them
behind the first uses of the others to save registers.  A wait then stands
between two loads of one window, and the window takes two or more trips to memory
instead of one.  So in every basic block, the loads between two vector-memory
waits must be whole windows."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_36662_amd", "csrc")
INCLUDE = os.path.join(ROOT, "include")


def _round(k, stats, update, reset, payload=0):
    """A round kernel of k fp32 replicas: (template, symbol, loads of one window)."""
    flags = [stats, update, reset, payload]
    return (f"round_kernel<{k}, RT_F32, {', '.join('true' if f else 'false' for f in flags)}>(RoundArgs)",
            f"_ZN8autoloco12round_kernelILi{k}ELi0E{''.join(f'Lb{f}E' for f in flags)}EEvNS_9RoundArgsE",
            k + 1 + update)


KERNELS = []
# the plain update of many fp32 replicas, with the mean as it is and through the BF16 payload
KERNELS += [_round(k, 0, 1, 0, p) for k in (12, 13, 14, 15, 16) for p in (0, 1)]
# the statistics alone of the most fp32 replicas
KERNELS += [_round(k, 1, 0, 0) for k in (15, 16)]
# AdamW's norm pass: every worker's gradient
KERNELS += [(f"grad_norm_kernel<{k}>(GradNormArgs)", f"_ZN8autoloco16grad_norm_kernelILi{k}EEEvNS_12GradNormArgsE", k)
            for k in (3, 8, 11, 12, 13, 14, 15, 16)]
# the shard step with one payload: two runs of theta, momentum and payload
KERNELS += [("shard_step_kernel<1>(ShardArgs)", "_ZN8autoloco17shard_step_kernelILi1EEEvNS_9ShardArgsE", 3)]


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
    tmp = tmp_path_factory.mktemp("isa_together")
    src, out = tmp / "together.hip", tmp / "together.s"
    src.write_text('#include "adamw_kernels.hpp"\n#include "shard_kernels.hpp"\nnamespace autoloco {\n' +
                   "".join(f"template __global__ void {t};\n" for t, _, _ in KERNELS) + "}\n")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", f"-I{INCLUDE}", f"-I{CSRC}", "--cuda-device-only", "-S", str(src), "-o", str(out)]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-3000:]
    return out.read_text()


def _blocks(text, symbol):
    start = text.index("\n" + symbol + ":")
    blocks = [[]]
    for line in text[start:text.index(".Lfunc_end", start)].split("\n"):
        if line.startswith(".LBB"):
            blocks.append([])
        blocks[-1].append(line.strip())
    return blocks


@pytest.mark.parametrize("symbol,loads", [k[1:] for k in KERNELS])
def test_no_wait_between_the_loads_of_a_window(asm, symbol, loads):
    whole = 0
    for block in _blocks(asm, symbol):
        runs, run = [], 0
        for line in block:
            if line.startswith("global_load_dwordx"):
                run += 1
            elif run and line.startswith("s_waitcnt") and "vmcnt(" in line:
                runs.append(run)
                run = 0
        runs.append(run)
        assert all(r % loads == 0 for r in runs), (symbol, runs)
        whole += sum(runs) // loads
    assert whole >= 1, symbol
