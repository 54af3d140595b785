"""GPU parity of the round's main loop where it changes its way: workgroups with no
whole window, fewer than it keeps in flight, exactly as many, and several times as
many, with a short last window and a ragged tail; every mode.  The statistics of
every mode with them must be the same bits (same grid, same order)."""
import numpy as np
import pytest
import torch

import paper_2609_36662_amd as al
from tests.gpu_common import (assert_bf16_reset_close, assert_close_elementwise, assert_stats_close, bits16,
                              cpu_inputs, to_device)
from tests.test_gpu_parity import EPS, _oracle_round, _tiny_coeffs, ctx  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu
WINDOW = {torch.float32: 1024, torch.bfloat16: 2048}   # parameters of a workgroup's window


@pytest.mark.parametrize("windows", [0.4, 1, 2.6, 8, 16, 37.3])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("k", [1, 2, 4, 5, 6, 8, 16])
def test_every_mode(ctx, dtype, k, windows):  # noqa: F811
    grid = 3
    n = int(WINDOW[dtype] * windows * grid) // 4 * 4 + (3 if windows % 1 else 0)
    inp = cpu_inputs(n, k, seed=int(windows * 10) + k, replica_dtype=dtype)
    c = _tiny_coeffs(True)
    ref = _oracle_round(inp, c)
    al.autoloco_set_grid_limit(ctx, grid)
    try:
        dev = to_device(inp)
        first = al.autoloco_round_stats(ctx, dev.theta, dev.replicas, EPS)
        assert_stats_close(first, ref.stats, floor=1e-9 * max(ref.stats.D, 1e-30))
        for flags in (0, al.FUSE_STATS, al.FUSE_RESET, al.FUSE_STATS | al.FUSE_RESET):
            dev = to_device(inp)
            st = al.autoloco_outer_step(ctx, dev.theta, dev.momentum, dev.replicas, c, flags, EPS)
            torch.cuda.synchronize()
            if flags & al.FUSE_STATS:
                assert bytes(st) == bytes(first), flags
            th = dev.theta.cpu().numpy()
            assert_close_elementwise(th, ref.theta, what=f"theta' {flags}")
            assert_close_elementwise(dev.momentum.cpu().numpy(), ref.momentum, what=f"v' {flags}")
            for r, before in zip(dev.replicas, inp.replicas):
                if not flags & al.FUSE_RESET:
                    assert torch.equal(r.cpu(), before)
                elif dtype == torch.float32:
                    assert torch.equal(r, dev.theta)
                else:
                    assert np.array_equal(bits16(r), bits16(dev.theta.to(torch.bfloat16)))
                    assert_bf16_reset_close(bits16(r), ref.theta)
    finally:
        al.autoloco_set_grid_limit(ctx, 0)
