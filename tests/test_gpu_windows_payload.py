"""GPU parity of the BF16-payload round's main loop over the window counts where
it changes its way (no whole window, one, fewer than in flight, several times as
many, a short last window and a ragged tail), every mode: the received mean bit
for bit, the step and the statistics within the round's tolerances.  The worker
counts are those where a window's loads or the mean's store are ordered
differently, or where two windows are in flight (up to 4 fp32 replicas, update
with statistics)."""
import numpy as np
import pytest
import torch

import paper_2609_36662_amd as al
from oracle import bf16_payload as bp
from tests.gpu_common import (assert_bf16_reset_close, assert_close_elementwise, assert_stats_close, bits16,
                              cpu_inputs, host_array, to_device)
from tests.test_gpu_bf16_payload import EPS, ETA, MU, RHO, ctx  # noqa: F401 (a fixture)
from tests.test_gpu_windows import WINDOW

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("windows", [0.4, 1, 2.6, 8, 13.3])
@pytest.mark.parametrize("dtype,k", [(torch.float32, k) for k in (1, 2, 4, 5, 8, 9, 12, 15, 16)] +
                         [(torch.bfloat16, k) for k in (1, 4, 6, 7, 16)])
def test_every_payload_mode(ctx, dtype, k, windows):  # noqa: F811
    grid = 3
    n = int(WINDOW[dtype] * windows * grid) // 4 * 4 + (3 if windows % 1 else 0)
    inp = cpu_inputs(n, k, seed=int(windows * 10) + k, replica_dtype=dtype)
    c = al.make_coeffs(MU, ETA, RHO, True)
    ref = bp.bf16_round(inp.theta.numpy(), inp.momentum.numpy(), [host_array(r) for r in inp.replicas],
                        c.mu, c.eta_out, c.rho, True, EPS)
    al.autoloco_set_grid_limit(ctx, grid)
    try:
        for flags in (0, al.FUSE_STATS, al.FUSE_RESET, al.FUSE_STATS | al.FUSE_RESET):
            dev = to_device(inp)
            mean = torch.zeros(n + 64, dtype=torch.bfloat16, device="cuda")
            st = al.autoloco_outer_step_bf16(ctx, dev.theta, dev.momentum, dev.replicas, c, flags, EPS,
                                             mean_bf16=mean[:n])
            torch.cuda.synchronize()
            assert np.array_equal(bits16(mean)[:n], ref.mean_bits), flags
            assert not mean[n:].any()
            if flags & al.FUSE_STATS:
                assert_stats_close(st, ref.stats, floor=1e-9 * max(ref.stats.D, 1e-30))
            assert_close_elementwise(dev.theta.cpu().numpy(), ref.theta, what=f"theta' {flags}")
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
