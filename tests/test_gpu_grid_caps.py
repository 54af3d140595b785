"""GPU test of the calls whose way changes with a grid cap above the default.

AdamW's norms are added up by a kernel between the passes from 1,025 workgroups on:
state and norms against the oracle on both sides of that line, and the norms equal
bit for bit with and without clipping.  The round's statistics keep several windows
in flight up to 768 workgroups, their update up to 256: against the oracle on both
sides, the standalone and the fused statistics with the same bits."""
import pytest
import torch

import paper_2609_36662_amd as al
from oracle import adamw as oa
from tests.gpu_common import assert_close_elementwise, assert_stats_close, cpu_inputs, to_device
from tests.test_gpu_adamw import C4, _check_stats, _coeffs, _np, ctx  # noqa: F401 (a fixture)
from tests.test_gpu_parity import EPS, _oracle_round, _tiny_coeffs
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


@pytest.mark.parametrize("cap", [256, 257, 768, 769])
@pytest.mark.parametrize("k,dtype", [(1, torch.float32), (3, torch.float32), (2, torch.bfloat16)])
def test_round_statistics_above_the_default_grid(ctx, k, dtype, cap):  # noqa: F811
    window = 1024 if dtype == torch.float32 else 2048
    n = 2 * 769 * window + 5 * window // 2 + 3      # two windows a workgroup at the largest cap, and a short last one
    inp = cpu_inputs(n, k, seed=cap + k, replica_dtype=dtype)
    c = _tiny_coeffs(True)
    ref = _oracle_round(inp, c)
    al.autoloco_set_grid_limit(ctx, cap)
    try:
        dev = to_device(inp)
        first = al.autoloco_round_stats(ctx, dev.theta, dev.replicas, EPS)
        st = al.autoloco_outer_step(ctx, dev.theta, dev.momentum, dev.replicas, c, al.FUSE_STATS, EPS)
        torch.cuda.synchronize()
    finally:
        al.autoloco_set_grid_limit(ctx, 0)
    assert_stats_close(first, ref.stats, floor=1e-9 * max(ref.stats.D, 1e-30))
    assert bytes(st) == bytes(first)
    assert_close_elementwise(dev.theta.cpu().numpy(), ref.theta, what="theta'")
    assert_close_elementwise(dev.momentum.cpu().numpy(), ref.momentum, what="v'")
