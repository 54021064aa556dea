"""The public normal operator, in two passes and in one (k_normal_pub), where its neighbours
coincide or wrap and where its grid has a remainder: equal, bit for bit, to M applied to M^dagger x by the
public calls at mu2 = 0 (the same products and sums in the same order), and to the oracle with
mu2 at the bar of the other operator tests (1e-13 of the largest entry).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1804_07195_amd import binding as hb
from tests.gpu_helpers import dev, host, lattices, rel_max

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hub():
    ctx = hb.Context(0)
    yield ctx
    ctx.close()


# one vector per workgroup (two passes), and groups (one pass): 2 for the four vectors, 4 to 8
CASES = [(s, b) for s in [(3, 2, 1), (1, 1, 2), (1, 2, 3), (2, 1, 64), (2, 2, 2), (16, 16, 4)] for b in (1, 3, 64)] + [
    ((1, 1, 9000), 64), ((1, 2, 5001), 64), ((2, 1, 5000), 64), ((130, 70, 1), 64), ((25, 23, 30), 64), ((32, 33, 64), 4)]


@pytest.mark.parametrize("shape,batch", CASES, ids=["x".join(map(str, s)) + "-%d" % b for s, b in CASES])
def test_normal_is_M_of_Mdagger(hub, shape, batch):
    hl, ol = lattices(*shape, 0.2, 0.04)
    rng = np.random.default_rng(5)
    phi = rng.normal(0.0, 1.0, size=ol.shape)
    x = rng.standard_normal((batch, *ol.shape)) + 1j * rng.standard_normal((batch, *ol.shape))
    pd, xd = dev(phi), dev(x)
    y = hb.hub_apply_normal(hub, hl, pd, [0.0] * batch, xd)
    assert torch.equal(y, hb.hub_apply_M(hub, hl, pd, hb.hub_apply_Mdag(hub, hl, pd, xd)))
    mu2 = [0.1 * b for b in range(batch)]
    y = host(hb.hub_apply_normal(hub, hl, pd, mu2, xd))
    for b in {0, batch - 1}:
        assert rel_max(y[b], oracle.normal_apply(ol, phi, mu2[b], x[b])) <= 1e-13
