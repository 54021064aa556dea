"""A gang that does not meet goes on in steps, with the bits of the whole launch (GPU).

Launches are refused on the host's word (a mask over their number), so that a solve runs
whole, in steps from its start, or changes between the two after the first launch, for
blocks cut in time, in space and in both, for every body (sites per thread, the solution in
registers or in memory) and both precisions.  Everything is compared bit for bit with the
solve whose gangs all meet.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_1804_07195_amd import binding as hb
from tests.gpu_helpers import dev, lattices

pytestmark = pytest.mark.gpu

ALWAYS, FIRST, LATER = 0xffffffff, 0x1f, 0x3e
CASES = [((4, 3, 27), "cg"), ((6, 6, 64), "cg"), ((6, 6, 64), "fgmres"), ((12, 12, 32), "cg"), ((12, 12, 32), "fgmres"),
         ((13, 22, 18), "fgmres"), ((33, 17, 6), "cg"), ((25, 23, 30), "fgmres"), ((40, 32, 16), "cg"),
         ((48, 48, 32), "fgmres"), ((102, 77, 24), "cg"), ((102, 77, 48), "fgmres"), ((102, 77, 64), "fgmres")]


@pytest.mark.parametrize("shape,solver", CASES, ids=["x".join(map(str, s)) + "-" + v for s, v in CASES])
def test_steps_have_the_same_bits(shape, solver):
    hl, ol = lattices(*shape, 0.2, 0.03)
    rng = np.random.default_rng(17)
    phi = dev(rng.normal(0.0, 0.8, size=ol.shape))
    b = dev(rng.standard_normal((2,) + ol.shape) + 1j * rng.standard_normal((2,) + ol.shape))
    # the FP64 CG also cut off, at odd and even counts and beyond the first launch
    caps = [1, 2, 17, 150, 20000] if solver == "cg" else [20]
    lib = hb.load()
    lib.hub_test_deny_meetings.argtypes = [ctypes.c_void_p, ctypes.c_uint32]
    ctx = hb.Context(0)
    try:
        for cap in caps:
            opts = hb.default_opts(solver=solver, tol=1e-12, max_iter=cap)
            want = None
            for mask in (0, ALWAYS, FIRST, LATER):
                assert lib.hub_test_deny_meetings(ctx.handle, mask) == hb.HUB_OK
                x, info, st = hb.hub_solve(ctx, hl, phi, [0.0, 0.05], b, opts=opts, allow_noconv=True)
                assert st == (hb.HUB_ERR_NOCONV if solver == "cg" and cap < 20000 and
                              any(not i["converged"] for i in info) else hb.HUB_OK)
                if want is None:
                    want = (x.clone(), info)
                assert info == want[1], (cap, hex(mask))
                assert torch.equal(x, want[0]), (cap, hex(mask))
    finally:
        ctx.close()
