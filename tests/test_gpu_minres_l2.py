"""MINRES with the second Lanczos update inside the element kernel (box meshes of
up to 1024 workgroups) against the oracle's MINRES: every hex class that has
it, ragged last workgroups, fixed DoFs by boundary, by mask and none, and the
sizes at which it ends (1024 workgroups; above, the general path).  Tolerance
as in the test of the general path, 1e-9 of dx after 8 iterations; the FP32
action against the general path (three-term form), whose entries may differ by
one FP32 rounding: 1e-4.
"""
import numpy as np
import pytest

import oracle
from oracle import solver
from tests.gpu_common import log, make_case, rel, to_dev, to_host

pytestmark = pytest.mark.gpu

CLASSES = [(1, 2), (1, 3), (1, 4), (2, 3), (2, 4), (2, 5), (3, 4), (3, 5), (3, 6), (4, 5), (4, 6)]


def _case(dim, ns, p, nq, ess, storage, precision="fp64"):
    import torch
    from paper_2205_12721_amd.tmop import Context
    pb, x = make_case(dim, ns, p, nq, "interior_jitter", 0.02, seed=81,
                      constrain="boundary" if ess == "boundary" else None)
    kw = {}
    if ess == "mask":
        mask = np.random.default_rng(82).uniform(size=pb.ndof) < 0.2
        pb = oracle.Problem(dim, p, nq, pb.e2n, pb.nx, ess=mask)
        kw = dict(ess=torch.as_tensor(mask.astype(np.uint8)).cuda())
    x = x + 1e-3 / max(ns) * np.random.default_rng(83).standard_normal(x.size)
    ctx = Context(dim, ns, p, nq, storage=storage, precision=precision, **kw)
    ctx.hessian_setup(to_dev(x))
    return pb, x, ctx


def _check(dim, ns, p, nq, ess, storage, jacobi, its=8):
    log("case", dim, ns, p, nq, ess, storage, jacobi)
    pb, x, ctx = _case(dim, ns, p, nq, ess, storage)
    g = pb.gradient(x)
    minv = solver.jacobi_inverse(pb.diag(x), pb.ess)
    pre = (lambda r: minv * r) if jacobi else None
    for n in (its, 1):
        xo, ito, _ = solver.minres(lambda v: pb.hvp(x, v), g, pre, rtol=1e-9, maxit=n)
        dx, itg = ctx.minres(to_dev(g), max_its=n, rtol=1e-9, jacobi=jacobi)
        assert itg == ito
        assert rel(to_host(dx), xo) <= 1e-9
    ctx.close()


@pytest.mark.parametrize("storage", ["tensor", "compact"])
@pytest.mark.parametrize("p,nq", CLASSES)
def test_classes(p, nq, storage):
    _check(3, (5, 3, 3), p, nq, "mask", storage, True)


@pytest.mark.parametrize("dim,ns,p,nq,ess", [
    (3, (4, 3, 5), 3, 5, "boundary"), (2, (17, 19), 2, 4, "boundary"), (2, (23, 9), 3, 5, "mask"),
    (3, (16, 8, 8), 3, 6, "boundary"), (3, (43, 6, 4), 3, 6, "boundary"),
    (2, (64, 80), 4, 7, "boundary"), (2, (569, 9), 4, 7, "mask")])
def test_edges(dim, ns, p, nq, ess):
    _check(dim, ns, p, nq, ess, "compact", False)


@pytest.mark.parametrize("storage", ["tensor", "compact"])
@pytest.mark.parametrize("dim,ns,p,nq", [(3, (4, 4, 3), 2, 4), (3, (3, 3, 3), 4, 6), (2, (17, 12), 3, 5)])
def test_mixed(dim, ns, p, nq, storage):
    log("case", dim, ns, p, nq, storage)
    pb, x, ctx = _case(dim, ns, p, nq, "boundary", storage, "mixed")
    g = to_dev(pb.gradient(x))
    a, ia = ctx.minres(g, max_its=8, rtol=0.0)
    a = to_host(a)
    ctx.set_lanczos_bank_limit(0)
    b, ib = ctx.minres(g, max_its=8, rtol=0.0)
    assert ia == ib == 8
    assert rel(a, to_host(b)) <= 1e-4
    ctx.close()
