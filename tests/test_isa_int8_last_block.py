"""CPU check in the gfx950 assembly that the INT8 round does not read its last
block twice: the lane offset of the next block's loads is selected against zero
(on a workgroup's last block all lanes read the same 16 bytes), so the offset the
loads use is the result of that selection."""
import re
import subprocess

import pytest

from tests.test_isa_int8_loop import CSRC, INCLUDE, _hipcc, _loop_path

KERNELS = [(k, rt, st, rs) for k in (1, 3, 8, 9, 16) for rt in (0, 1) for st, rs in ((1, 1), (0, 0))]


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    hipcc = _hipcc()
    if hipcc is None:
        pytest.skip("hipcc not available")
    tmp = tmp_path_factory.mktemp("isa_last")
    src, out = tmp / "last.hip", tmp / "last.s"
    src.write_text('#include "int8_kernels.hpp"\nnamespace autoloco {\n' + "".join(
        f"template __global__ void int8_round_kernel<{k}, {('RT_F32', 'RT_BF16')[rt]}, {('false', 'true')[st]}, "
        f"{('false', 'true')[rs]}>(Int8Args);\n" for k, rt, st, rs in KERNELS) + "}\n")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", f"-I{INCLUDE}", f"-I{CSRC}", "--cuda-device-only", "-S", str(src), "-o", str(out)]
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-3000:]
    return out.read_text()


@pytest.mark.parametrize("k,rt,st,rs", KERNELS)
def test_last_block_is_not_read_again(asm, k, rt, st, rs):
    _, path = _loop_path(asm, f"_ZN8autoloco17int8_round_kernelILi{k}ELi{rt}ELb{st}ELb{rs}EEEvNS_8Int8ArgsE")
    select = re.compile(r"v_cndmask_b32\S* (v\d+), 0, v\d+")
    checked = 0
    for i, line in enumerate(path):
        # the next block's loads at a scalar base (the momentum's, of this block, is no
        # direct load; workers 9 and up come through registers behind theta's second part)
        m = re.match(r"global_load_lds_dwordx4 (v\d+), s\[", line)
        if not m:
            continue
        reg = m.group(1)
        write = re.compile(rf"v_\S+ {reg},|v_\S+ v\[{reg[1:]}:")
        last = next(l for l in reversed(path[:i]) if write.match(l))
        assert select.match(last) and select.match(last).group(1) == reg, (line, last)
        checked += 1
    assert checked >= min(k, 8), checked
