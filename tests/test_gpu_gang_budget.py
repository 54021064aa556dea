"""A request's bits do not depend on what else is served, whatever the budget (GPU).

Budgets from one request's workspace up: with the smallest the tiled kernels iterate, with
the others the gang, and never one alone and the other in company.
"""
import time

import numpy as np
import pytest
import torch

from paper_1804_07195_amd import binding as hb
from tests.gpu_helpers import dev, lattices

pytestmark = pytest.mark.gpu


def _served(budget, hl, jobs, opts):
    """x of every job, all in flight together on a context of their own; None: never fits."""
    ctx = hb.Context(0, hbm_budget_bytes=budget)
    try:
        try:
            wait = pend = [hb.hub_submit(ctx, hl, mu2, phi, b, opts=opts) for mu2, phi, b in jobs]
        except hb.HubError as e:
            assert e.status == hb.HUB_ERR_BUSY
            return None
        end = time.time() + 60
        while wait:
            assert time.time() < end
            polled = [(p, hb.hub_poll(ctx, p)) for p in wait]
            assert all(info["status"] == hb.HUB_OK for _, (done, info) in polled if done)
            wait = [p for p, (done, _) in polled if not done]
        return [p.x.clone() for p in pend]
    finally:
        ctx.close()


@pytest.mark.parametrize("solver", ["cg", "fgmres"])
def test_alone_and_in_company(solver):
    hl, ol = lattices(12, 12, 32, 0.2)
    rng = np.random.default_rng(5)
    jobs = [(mu2, dev(rng.normal(0.0, 0.8, size=ol.shape)),
             dev(rng.standard_normal((1,) + ol.shape) + 1j * rng.standard_normal((1,) + ol.shape)))
            for mu2 in (0.0, 0.01, 0.05, 0.1)]
    opts = hb.default_opts(solver=solver, tol=1e-11)
    torch.cuda.synchronize()
    # the smallest budget that is not refused: one workspace, to 64 KiB
    lo, hi = 0, 64 << 20
    while hi - lo > 65536:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if _served(mid, hl, jobs[:1], opts) is not None else (mid, hi)
    kinds = []
    for part in (1.0, 1.3, 1.7, 2.2, 3.0, 4.0, 6.0, 20.0):
        alone = [_served(int(hi * part), hl, [j], opts)[0] for j in jobs]
        both = _served(int(hi * part), hl, jobs, opts)
        for a, b in zip(alone, both):
            assert torch.equal(a, b), part
        if not any(torch.equal(alone[0], k) for k in kinds):
            kinds.append(alone[0])
    assert len(kinds) == 2
