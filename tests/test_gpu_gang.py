"""The gang CG (csrc/hub_gang.hip) where its cut or its body changes.

* FP64: the k-th iterate against the oracle's textbook CG (1e-12, as for the other CG
  kernels) for one workgroup, cuts in time, in space and in both, partly filled bodies,
  and iterations past the end of a launch (the state kept between launches).
* Mixed solves over the same range and solves with the bodies of the largest blocks,
  judged by the oracle's true residual.
* Gangs of several contexts that do not fit on the device together, at once: every
  solve is what it is alone.
"""
import threading

import numpy as np
import pytest
import torch

import oracle
from oracle.operator import NormalOperator
from oracle.solve import cg as oracle_cg
from paper_1804_07195_amd import binding as hb
from tests.gpu_helpers import dev, host, lattices, rel2

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 3), (2, 1, 16), (4, 3, 27), (6, 6, 16), (6, 6, 64), (9, 9, 40), (11, 11, 42), (12, 12, 32),
          (13, 22, 18), (33, 17, 6), (25, 23, 30), (40, 32, 16)]


@pytest.fixture(scope="module")
def hub():
    ctx = hb.Context(0)
    yield ctx
    ctx.close()


def _field(shape, seed, ms=0.0):
    hl, ol = lattices(*shape, 0.2, ms)
    rng = np.random.default_rng(seed)
    phi = rng.normal(0.0, 0.8, size=ol.shape)
    b = rng.standard_normal(ol.shape) + 1j * rng.standard_normal(ol.shape)
    return hl, ol, phi, b


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_fp64_iterates(hub, shape):
    hl, ol, phi, b = _field(shape, 7, ms=0.03)
    mu2 = 0.05
    op = NormalOperator(ol, phi, mu2)
    for k in (1, 2, 6, 129, 259):
        want, its, rel = oracle_cg(op, b.ravel(), tol=1e-13, maxiter=k)
        # alone, and with another: the launches are longer for one
        for rhs in ([b], [b, 2 * b]):
            x, info, st = hb.hub_solve(hub, hl, dev(phi), [mu2] * len(rhs), dev(np.stack(rhs)),
                                       opts=hb.default_opts(solver="cg", max_iter=k, tol=1e-13), allow_noconv=True)
            if its == k:
                assert info[0]["inner_iters"] == k
            assert rel2(host(x)[0].ravel(), want) <= 1e-12, k
        if its < k:
            break


# with the bodies of the largest blocks: eight and eleven sites per thread, four in FP64
LARGE = [((48, 48, 32), "fgmres"), ((102, 77, 48), "fgmres"), ((102, 77, 64), "fgmres"), ((102, 77, 24), "cg")]
SOLVES = [(s, "fgmres") for s in SHAPES + [(10, 9, 12), (10, 4, 20)]] + LARGE


@pytest.mark.parametrize("shape,solver", SOLVES, ids=["x".join(map(str, s)) + "-" + v for s, v in SOLVES])
def test_residual(hub, shape, solver):
    hl, ol, phi, b = _field(shape, 8, ms=0.03)
    mu2 = [0.01, 0.3]
    x, info, _ = hb.hub_solve(hub, hl, dev(phi), mu2, dev(np.stack([b, b])), opts=hb.default_opts(solver=solver))
    for k, m in enumerate(mu2):
        r = b - oracle.normal_apply(ol, phi, m, host(x)[k])
        assert np.linalg.norm(r) <= 1e-10 * np.linalg.norm(b)


def test_gangs_of_several_contexts():
    jobs = []
    for seed, (shape, solver) in enumerate([((102, 102, 16), "cg"), ((102, 102, 32), "fgmres"), ((48, 48, 64), "cg"),
                                            ((24, 24, 64), "fgmres")]):
        lat = hb.lattice(*shape, 0.1875)
        gen = torch.Generator(device="cuda").manual_seed(seed)
        phi = torch.randn((shape[2], 2) + shape[:2], generator=gen, dtype=torch.float64, device="cuda") * 0.7
        b = torch.randn((2, shape[2], 2) + shape[:2], generator=gen, dtype=torch.complex128, device="cuda")
        jobs.append((hb.Context(0), lat, phi, b, hb.default_opts(solver=solver)))
    torch.cuda.synchronize()

    def solve(job, stream):
        ctx, lat, phi, b, opts = job
        x, _, _ = hb.hub_solve(ctx, lat, phi, [0.1, 0.02], b, opts=opts, stream=stream)
        stream.synchronize()
        return x.cpu()

    alone = [solve(j, torch.cuda.Stream()) for j in jobs]
    got, errors = {}, []

    def work(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                got[k] = [solve(jobs[k], s) for _ in range(4)]
        except Exception as e:  # reported below
            errors.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join(timeout=100)
    assert not errors and len(got) == len(jobs), errors
    for k in range(len(jobs)):
        for x in got[k]:
            assert torch.equal(x, alone[k]), k
    for j in jobs:
        j[0].close()
