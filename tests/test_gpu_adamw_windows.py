"""GPU parity of both loops of the inner AdamW update and of the norm pass in
front of it, element by element against the oracle.

From 16 windows (of 1,024 parameters) a workgroup on, the update loads the next
window before it works on this one; it walks from the last window, which may be
short, down to the first.  A capped grid puts the window counts just below, at
and above that line, for one and three workgroups a worker, with short last
windows and ragged tails, with and without the BF16 copy; the same cap takes the
norm pass (four windows at once for one worker, two for two) through its
unrolled loop and its remainder.  Guard bands catch a write past n."""
import numpy as np
import pytest
import torch

import paper_2609_36662_amd as al
from oracle import adamw as oa
from tests.gpu_common import assert_bf16_reset_close, assert_close_elementwise, bits16
from tests.test_gpu_adamw import C4, _check_stats, _coeffs, _np, ctx  # noqa: F401 (a fixture)
from workloads import inner

pytestmark = pytest.mark.gpu
GUARD = 4100


def _guarded(t, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.cat([t, torch.randn(GUARD, generator=g).to(t.dtype)]).cuda()


@pytest.mark.parametrize("copy", [False, True])
@pytest.mark.parametrize("per", [1, 3])
@pytest.mark.parametrize("k", [1, 2, 4])
@pytest.mark.parametrize("windows,tail", [(15, 0), (15.6, 3), (16, 0), (16.3, 1), (17, 2), (33.7, 3)])
def test_every_element(ctx, windows, tail, k, per, copy):  # noqa: F811
    n = int(windows * per * 1024) // 4 * 4 + tail
    lr, step = 3e-4, 1 + k
    host = inner.make_state(n, k, seed=int(10 * windows) + k)
    ref = oa.inner_step(_np(host.params), _np(host.exp_avg), _np(host.exp_avg_sq), _np(host.grads), lr, step, C4)
    groups = [[_guarded(t, 7 * i + j) for i, t in enumerate(group)]
              for j, group in enumerate((host.params, host.exp_avg, host.exp_avg_sq, host.grads))]
    cp = [_guarded(torch.zeros(n, dtype=torch.bfloat16), 90 + i) for i in range(k)] if copy else None
    every = [t for group in groups for t in group] + (cp or [])
    bands = [t[n:].clone() for t in every]
    al.autoloco_set_grid_limit(ctx, per * k)
    try:
        st = al.autoloco_inner_adamw(ctx, *groups, _coeffs(C4, lr, step), model_bf16=cp, n=n)
        torch.cuda.synchronize()
    finally:
        al.autoloco_set_grid_limit(ctx, 0)
    _check_stats(st, ref, k)
    for i in range(k):
        for name, got, want in zip(("params", "m", "v"), groups, (ref.params, ref.exp_avg, ref.exp_avg_sq)):
            assert_close_elementwise(got[i][:n].cpu().numpy(), want[i], what=f"{name}[{i}]")
        assert torch.equal(groups[3][i][:n].cpu(), host.grads[i])
        if copy:
            assert np.array_equal(bits16(cp[i][:n]), bits16(groups[0][i][:n].to(torch.bfloat16)))
            assert_bf16_reset_close(bits16(cp[i][:n]), ref.params[i], what=f"bf16 copy {i}")
    for t, band in zip(every, bands):
        assert torch.equal(t[n:].view(torch.int16), band.view(torch.int16))
