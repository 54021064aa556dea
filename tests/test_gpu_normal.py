"""The one-pass public normal operator (k_normal_pub) where its neighbours coincide or wrap
and where its grid has a remainder: equal, bit for bit, to M applied to M^dagger x by the
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


@pytest.mark.parametrize("shape", [(3, 2, 1), (1, 1, 2), (1, 2, 3), (2, 1, 64), (2, 2, 2), (3, 4, 11), (16, 16, 4)])
@pytest.mark.parametrize("batch", [1, 3, 64])
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
    for b in range(batch):
        assert rel_max(y[b], oracle.normal_apply(ol, phi, mu2[b], x[b])) <= 1e-13
