"""GPU test of the two reduction stages: every sum ends in its own place for every
worker count (2K + 1 sums of the round and the INT8 round, K of AdamW's norms, one of
the payload kernel), for grids of one workgroup, fewer than a finishing
workgroup's threads, and more.  The inputs make every sum exact in any order:
worker k's pseudo-gradient is the same power of two everywhere, so the sums are n
times its square and the GPU's must equal that bit for bit."""
import pytest
import torch

import paper_2609_36662_amd as al

pytestmark = pytest.mark.gpu
N = 700 * 1024 + 3      # more windows than the largest grid below, and a ragged tail


@pytest.fixture(scope="module")
def ctx():
    c = al.autoloco_create(0)
    yield c
    c.close()


@pytest.mark.parametrize("grid", [1, 3, 600])
@pytest.mark.parametrize("k", range(1, 17))
def test_every_sum_in_its_place(ctx, k, grid):
    theta = torch.zeros(N, device="cuda")
    momentum = torch.zeros(N, device="cuda")
    reps = [torch.full((N,), 2.0 ** (i - 8), device="cuda") for i in range(k)]
    grads = [torch.full((N,), 2.0 ** (i - 8), device="cuda") for i in range(k)]
    want = [N * 4.0 ** (i - 8) for i in range(k)]
    al.autoloco_set_grid_limit(ctx, grid)
    try:
        st = al.autoloco_round_stats(ctx, theta, reps)
        assert list(st.sq_norm[:k]) == want
        q = al.autoloco_outer_step_int8(ctx, theta, momentum, reps, al.make_coeffs(0.9, 0.7), al.FUSE_STATS)
        assert list(q.sq_norm[:k]) == want
        # the deviations belong to their workers: for a constant mean m, n (d_k - m)^2
        m = sum(2.0 ** (i - 8) for i in range(k)) / k
        for i in range(k):
            assert st.sq_dev[i] == pytest.approx(N * (2.0 ** (i - 8) - m) ** 2, rel=1e-5, abs=N * m * m * 1e-10)
            # a constant block decodes to its value times 1 + e, |e| <= 5 roundings of 2^-24 (two scales, two products,
            # the mean), so the square is off by 2 |e| m |d_k - m| at most: never more than this sum of a relative 1e-5
            # and (e m)^2 / 1e-5
            assert q.sq_dev[i] == pytest.approx(N * (2.0 ** (i - 8) - m) ** 2, rel=1e-5, abs=N * m * m * 1e-8)
        assert st.sq_mean == pytest.approx(N * m * m, rel=1e-6)
        zeros = [[torch.zeros(N, device="cuda") for _ in range(k)] for _ in range(3)]
        norms = al.autoloco_inner_adamw(ctx, *zeros, grads, al.make_adamw_coeffs(1e-3, 1, max_grad_norm=0.0))
        assert [x * x for x in norms.grad_norm[:k]] == pytest.approx(want, rel=1e-12)
    finally:
        al.autoloco_set_grid_limit(ctx, 0)
    payload = torch.empty(N, dtype=torch.bfloat16, device="cuda")
    assert al.autoloco_rank_payload(ctx, torch.zeros(N, device="cuda"), reps[k - 1], payload) == want[k - 1]


# Up to 1,024 partial sums the host adds them up in the second stage's order; the call
# without a context always launches that stage: equal bits on random inputs at one
# workgroup, below a wavefront's 64, and on both sides of 1,024 (1,024 parameters a
# workgroup, 2K + 1 sums; with one worker the default grid ends at 256 workgroups, 768
# sums, so all its sizes are on the host's side).
@pytest.mark.parametrize("k", [1, 2, 8, 16])
def test_host_and_kernel_second_stage_agree(ctx, k):
    most = 1024 // (2 * k + 1)
    coeffs = al.make_coeffs(0.9, 0.7)
    for blocks in sorted({1, 2, 31, 65, 129, most - 1, most, most + 1}):
        n = blocks * 1024 - 5
        g = torch.Generator(device="cuda").manual_seed(blocks)
        theta = torch.randn(n, device="cuda", generator=g)
        reps = [theta + torch.randn(n, device="cuda", generator=g) * 10.0 ** (i % 5 - 4) for i in range(k)]
        momentum = torch.zeros(n, device="cuda")
        want = al.autoloco_outer_step_static(theta.clone(), momentum.clone(), reps, coeffs, al.FUSE_STATS)
        got = al.autoloco_outer_step(ctx, theta.clone(), momentum.clone(), reps, coeffs, al.FUSE_STATS)
        assert got.as_dict() == want.as_dict(), blocks
        assert al.autoloco_round_stats(ctx, theta, reps).as_dict() == want.as_dict(), blocks
