"""The one-pass force and actions of the Hasenbusch terms (k_terms) and the applies of a
kick group in one launch (k_apply_jobs) against the same quantities composed from the
public single-vector calls, at a lattice below one workgroup, exactly one, one and a
remainder, and many; 1, 2 and 17 terms; adding to a given force or not.

With the solutions eta given back by the call: xi_i = M_den^dagger eta_i and the force of
eta_i with xi_i - chi_i.  Both sides hold the same products in FP64 and differ by the
rounding of at most 17 additions of terms of one size: 17 * 2^-53 < 1e-14, with the
differences xi - chi of at most ten times the size of their result, 1e-13 in the 2-norm.
The actions are sums over N products, pairwise on both sides: 1e-13.
"""
import numpy as np
import pytest
import torch

from paper_1804_07195_amd import binding as hb
from tests.gpu_helpers import dev, host, rel2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hub():
    ctx = hb.Context(0)
    yield ctx
    ctx.close()


@pytest.mark.parametrize("shape", [(1, 1, 2), (2, 1, 64), (5, 3, 9), (12, 12, 32)])
@pytest.mark.parametrize("nmass", [0, 1, 16])
@pytest.mark.parametrize("accumulate", [False, True])
def test_terms_match_single_calls(hub, shape, nmass, accumulate):
    L1, L2, Nt = shape
    rng = np.random.default_rng(7)
    mts = [0.15 * (k + 1) for k in range(nmass)]
    lat = [hb.lattice(L1, L2, Nt, 0.2, m) for m in [0.02] + mts]  # lat[i + 1]: mass of operator i
    full = (nmass + 1, Nt, 2, L1, L2)
    phi = dev(rng.normal(0.0, 0.7, size=full[1:]))
    rho = dev(rng.standard_normal(full) + 1j * rng.standard_normal(full))
    start = rng.normal(size=full[1:])
    chi, _, _ = hb.hub_hasenbusch_heatbath(hub, lat[0], phi, mts, rho)
    out = dev(start.copy())
    F, S, eta, _, _ = hb.hub_hasenbusch_force(hub, lat[0], phi, mts, chi, scale=0.75, accumulate=accumulate, out=out)
    ref = dev(start.copy()) if accumulate else dev(np.zeros(full[1:]))
    for i in range(nmass + 1):
        last = i == nmass
        den = lat[nmass] if last else lat[i]
        rhs = chi[i] if last else hb.hub_apply_M(hub, lat[i + 1], phi, chi[i].contiguous())
        xi = hb.hub_apply_Mdag(hub, den, phi, eta[i].contiguous())
        z = xi if last else xi - chi[i]
        hb.hub_force(hub, den, phi, eta[i].contiguous(), xi=z.contiguous(), scale=0.75, accumulate=True, out=ref)
        s = float(np.vdot(host(rhs).ravel(), host(eta[i]).ravel()).real)
        assert abs(S[i] - s) <= 1e-13 * float(torch.linalg.vector_norm(rhs) * torch.linalg.vector_norm(eta[i]))
    assert rel2(host(F), host(ref)) <= 1e-13
