"""GPU test of the calls whose way changes with a grid cap above the default
(three workgroups per compute unit, 768): AdamW's norms are added up by a kernel
between the passes from 1,025 workgroups on.  State and norms against the oracle on
both sides of that line, and the norms equal bit for bit with and without clipping."""
import pytest
import torch

import paper_2609_36662_amd as al
from oracle import adamw as oa
from tests.gpu_common import assert_close_elementwise
from tests.test_gpu_adamw import C4, _check_stats, _coeffs, _np, ctx  # noqa: F401 (a fixture)
from workloads import inner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [1024, 1025, 16384])
@pytest.mark.parametrize("k", [1, 3])
def test_adamw_norms_above_the_default_grid(ctx, k, cap):  # noqa: F811
    n = 1100 * 1024 + 5          # 1,101 workgroups of the norm pass, if the cap lets them
    host = inner.make_state(n, k, seed=k)
    ref = oa.inner_step(_np(host.params), _np(host.exp_avg), _np(host.exp_avg_sq), _np(host.grads), 3e-4, 2, C4)
    groups = [[t.cuda() for t in g] for g in (host.params, host.exp_avg, host.exp_avg_sq, host.grads)]
    other = [[t.clone() for t in g] for g in groups]
    al.autoloco_set_grid_limit(ctx, cap)
    try:
        st = al.autoloco_inner_adamw(ctx, *groups, _coeffs(C4, 3e-4, 2))
        free = al.autoloco_inner_adamw(ctx, *other, al.make_adamw_coeffs(3e-4, 2, max_grad_norm=0.0))
        torch.cuda.synchronize()
    finally:
        al.autoloco_set_grid_limit(ctx, 0)
    _check_stats(st, ref, k)
    assert list(st.grad_norm[:k]) == list(free.grad_norm[:k])
    for i in range(k):
        for name, got, want in zip(("params", "m", "v"), groups, (ref.params, ref.exp_avg, ref.exp_avg_sq)):
            assert_close_elementwise(got[i].cpu().numpy(), want[i], what=f"{name}[{i}]")
