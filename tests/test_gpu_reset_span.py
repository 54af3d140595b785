"""GPU test of the standalone reset on both sides of the sizes where its launch
changes: four windows a span into one fp32 replica from 4M parameters on (two
replicas keep one window), and fewer workgroups for one or two bf16 replicas
from 100M on.  Bit for bit against theta, with guard bands, at the default grid
and at three workgroups, whose last spans are short."""
import pytest
import torch

import paper_2609_36662_amd as al

pytestmark = pytest.mark.gpu
GUARD = 8200
SPAN4 = 4 << 20          # parameters
BF16_FEWER = 100_000_000


@pytest.fixture(scope="module")
def ctx():
    c = al.autoloco_create(0)
    yield c
    c.close()


@pytest.mark.parametrize("grid", [0, 3])
@pytest.mark.parametrize("n,k,dtype", [
    (SPAN4 - 1, 1, torch.float32), (SPAN4, 1, torch.float32), (SPAN4 + 2 * 1024 + 515, 1, torch.float32),
    (SPAN4 + 4 * 1024 * 3 + 3, 1, torch.float32), (SPAN4 - 1, 2, torch.float32), (SPAN4 + 2 * 1024 + 515, 2, torch.float32),
    (BF16_FEWER - 1, 1, torch.bfloat16), (BF16_FEWER + 2051, 1, torch.bfloat16), (BF16_FEWER + 2051, 2, torch.bfloat16)])
def test_reset_is_the_copy_and_no_more(ctx, n, k, dtype, grid):
    g = torch.Generator(device="cuda").manual_seed(n % 1000 + k)
    theta = torch.randn(n + GUARD, device="cuda", generator=g)
    reps = [torch.randn(n + GUARD, device="cuda", generator=g).to(dtype) for _ in range(k)]
    bits = torch.int32 if dtype == torch.float32 else torch.int16
    bands = [r[n:].clone() for r in reps]
    before = theta.clone()
    al.autoloco_set_grid_limit(ctx, grid)
    try:
        al.autoloco_broadcast_reset(ctx, theta[:n], [r[:n] for r in reps])
        torch.cuda.synchronize()
    finally:
        al.autoloco_set_grid_limit(ctx, 0)
    want = theta[:n].to(dtype).view(bits)
    for r, band in zip(reps, bands):
        assert torch.equal(r[:n].view(bits), want)
        assert torch.equal(r[n:].view(bits), band.view(bits))
    assert torch.equal(theta.view(torch.int32), before.view(torch.int32))
