"""The public normal operator on both sides of the size from which it runs in one pass, with
groups of vectors that divide the batch and that do not, with the workspace of two passes and
with the least: M of M^dagger bit for bit (mu2 = 0), and the workspace that it takes.
"""
import numpy as np
import pytest
import torch

from paper_1804_07195_amd import binding as hb
from tests.gpu_helpers import dev, lattices

pytestmark = pytest.mark.gpu

# 30x30x128: 230,400 sites; 32x32x256: 524,288, two vectors are the million; 32x32x43: 88,064,
# six vectors are half of it and more
CASES = [((30, 30, 128), b) for b in (2, 3, 4, 5, 7, 8, 15)] + [((32, 32, 256), 2), ((31, 33, 256), 2), ((32, 32, 43), 5),
                                                               ((32, 32, 43), 6), ((5, 7, 9), 64)]


@pytest.mark.parametrize("shape,batch", CASES, ids=["x".join(map(str, s)) + "-%d" % b for s, b in CASES])
def test_groups(shape, batch):
    hl, ol = lattices(*shape, 0.2, 0.04)
    rng = np.random.default_rng(6)
    pd = dev(rng.normal(0.0, 1.0, size=ol.shape))
    xd = dev(rng.standard_normal((batch, *ol.shape)) + 1j * rng.standard_normal((batch, *ol.shape)))
    step = 2 << 20  # budgets in whole blocks of the pool
    for budget in (0, (ol.n * 16 + step) // step * step):
        ctx = hb.Context(0, hbm_budget_bytes=budget)
        try:
            want = hb.hub_apply_M(ctx, hl, pd, hb.hub_apply_Mdag(ctx, hl, pd, xd))
            assert torch.equal(hb.hub_apply_normal(ctx, hl, pd, [0.0] * batch, xd), want)
            y = torch.empty_like(xd)
            if batch * ol.n * 16 <= hb.HUB_NOALLOC_SCRATCH_BYTES:
                hb.hub_apply_normal_noalloc(ctx, hl, pd, [0.0] * batch, xd, y)
                assert torch.equal(y, want)
        finally:
            ctx.close()
