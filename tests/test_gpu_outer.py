"""The FGMRES outer kernels (k_arnoldi_dots, k_cgs and the reductions that their last
workgroups finish) and the warm starts, where a path changes: one workgroup per system, 32
and just past 32 (they count in groups from there), many; restart lengths at which the sums
of a tile are laid out 8, 32 and 64 wide; systems of several sizes of the two tile classes
in one call.  The solution's true residual, evaluated by the oracle in FP64, has to meet the
tolerance that the solver was given (1e-10 of |b|), as the solver itself claims.
"""
import numpy as np
import pytest

import oracle
from paper_1804_07195_amd import binding as hb
from tests.gpu_helpers import dev, host, lattices

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hub():
    ctx = hb.Context(0)
    yield ctx
    ctx.close()


@pytest.mark.parametrize("shape", [(1, 1, 3), (2, 3, 16), (3, 2, 17), (25, 23, 30)])
@pytest.mark.parametrize("solver,warm,restart", [("fgmres", w, m) for w in (False, True) for m in (1, 4, 15, 20)] +
                         [("cg", True, 10)])
def test_residual(hub, shape, solver, warm, restart):
    hl, ol = lattices(*shape, 0.2, 0.03)
    rng = np.random.default_rng(11)
    phi = rng.normal(0.0, 0.8, size=ol.shape)
    b, x0 = (rng.standard_normal((3, *ol.shape)) + 1j * rng.standard_normal((3, *ol.shape)) for _ in range(2))
    mu2 = [0.02, 0.2, 1.5]
    opts = hb.default_opts(solver=solver, restart_m=restart, tol=1e-10, use_x0=1 if warm else 0)
    x, info, _ = hb.hub_solve(hub, hl, dev(phi), mu2, dev(b), x=dev(x0.copy()), opts=opts)
    for k, m in enumerate(mu2):
        assert info[k]["converged"] == 1
        r = b[k] - oracle.normal_apply(ol, phi, m, host(x)[k])
        assert np.linalg.norm(r) <= 1e-10 * (1 + 1e-3) * np.linalg.norm(b[k])
