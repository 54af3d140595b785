"""GPU parity of the INT8 round's block loop at the worker counts where its way
of holding and prefetching a block changes (8 | 9: fp32 workers through registers
as well as LDS, theta read back from LDS; 16: the most), several blocks per
workgroup, a ragged last one, every flag subset."""
import pytest
import torch

import paper_2609_36662_amd as al
from tests.gpu_common import cpu_inputs, to_device
from tests.test_gpu_int8 import COEFFS, EPS, _check, ctx  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [1, 3])
@pytest.mark.parametrize("dtype,k", [(torch.float32, 7), (torch.float32, 9), (torch.float32, 13), (torch.float32, 16),
                                     (torch.bfloat16, 3), (torch.bfloat16, 9), (torch.bfloat16, 12)])
def test_several_blocks_per_workgroup(ctx, grid, dtype, k):  # noqa: F811
    # codes and scales bit for bit, step and statistics within the round's tolerances
    al.autoloco_set_grid_limit(ctx, grid)
    try:
        _check(ctx, 7 * 4096 + 100, k, dtype=dtype, seed=70 + grid + k, normalize=grid % 2 == 1)
    finally:
        al.autoloco_set_grid_limit(ctx, 0)


@pytest.mark.parametrize("k,dtype", [(1, torch.float32), (8, torch.bfloat16), (9, torch.float32), (12, torch.bfloat16),
                                     (16, torch.float32), (16, torch.bfloat16)])
@pytest.mark.parametrize("flags", [0, al.FUSE_STATS, al.FUSE_RESET])
def test_flag_subsets_agree(ctx, k, dtype, flags):  # noqa: F811
    # every flag subset takes the same step, bit for bit, as the call with both flags
    n = 9 * 4096 + 1001
    inp = cpu_inputs(n, k, seed=90 + k, replica_dtype=dtype)
    c = al.make_coeffs(COEFFS["mu"], COEFFS["eta_out"], COEFFS["rho"], True)
    al.autoloco_set_grid_limit(ctx, 2)
    try:
        a, b = to_device(inp), to_device(inp)
        want = al.autoloco_outer_step_int8(ctx, a.theta, a.momentum, a.replicas, c, al.FUSE_STATS | al.FUSE_RESET, EPS)
        got = al.autoloco_outer_step_int8(ctx, b.theta, b.momentum, b.replicas, c, flags, EPS)
        torch.cuda.synchronize()
    finally:
        al.autoloco_set_grid_limit(ctx, 0)
    assert torch.equal(a.theta, b.theta) and torch.equal(a.momentum, b.momentum)
    for x, y, z in zip(a.replicas, b.replicas, inp.replicas):
        assert torch.equal(y, x if flags & al.FUSE_RESET else z.cuda())
    if flags & al.FUSE_STATS:
        assert bytes(got) == bytes(want)
