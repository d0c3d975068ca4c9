"""MINRES in one launch (small quad meshes) against the oracle's MINRES, for every
class and at the edges of its blocks of elements (p = 2, n_q = 4: 64 elements
a pass, at most 128; the next larger mesh takes the general path) and of its
nodes (1024 lanes, two nodes each at most).  Tolerance as in the test of the
general path: 1e-9 of dx after at most 12 iterations.  The FP32 action is
compared with the general path's: its entries may differ by one FP32 rounding
(6e-8), which 12 iterations of a system conditioned up to some 1e3 leave
below 1e-4.
"""
import numpy as np
import pytest

from oracle import solver
from paper_2205_12721_amd import inputs
from tests.gpu_common import log, make_case, rel, to_dev, to_host

pytestmark = pytest.mark.gpu

CLASSES = [(1, 2), (1, 3), (1, 4), (2, 3), (2, 4), (2, 5), (3, 4), (3, 5), (3, 6), (4, 5), (4, 6), (4, 7)]
EDGES = [((8, 8), 2, 4), ((13, 5), 2, 4), ((16, 8), 2, 4), ((43, 3), 2, 4), ((32, 16), 1, 2),
         ((27, 19), 1, 2), ((128, 1), 3, 4), ((12, 9), 3, 4), ((8, 5), 4, 5), ((41, 1), 4, 5)]


def _setup(ns, p, nq, storage, precision="fp64", general=False):
    import torch
    from paper_2205_12721_amd.tmop import Context
    pb, x = make_case(2, ns, p, nq, "interior_jitter", 0.02, seed=71, constrain=None)
    # a fixed corner component pair keeps the translations out
    ess = np.zeros(pb.ndof, dtype=bool)
    ess[[0, pb.nx - 1, pb.nx, 2 * pb.nx - 1]] = True
    import oracle
    pb = oracle.Problem(2, p, nq, pb.e2n, pb.nx, ess=ess)
    x = x + 1e-3 / max(ns) * np.random.default_rng(72).standard_normal(x.size)
    mask = torch.as_tensor(ess.astype(np.uint8)).cuda()
    kw = dict(storage=storage, precision=precision, ess=mask)
    if general:
        ctx = Context(2, None, p, nq, elem_to_node=torch.as_tensor(pb.e2n).cuda(), num_nodes=pb.nx, **kw)
    else:
        ctx = Context(2, ns, p, nq, **kw)
    ctx.hessian_setup(to_dev(x))
    return pb, x, ctx


def _check(ns, p, nq, storage, jacobi, general, its=12):
    log("case", ns, p, nq, storage, jacobi, general)
    pb, x, ctx = _setup(ns, p, nq, storage, general=general)
    g = pb.gradient(x)
    minv = solver.jacobi_inverse(pb.diag(x), pb.ess)
    pre = (lambda r: minv * r) if jacobi else None
    for rtol in (1e-5, 0.3):
        xo, ito, _ = solver.minres(lambda v: pb.hvp(x, v), g, pre, rtol=rtol, maxit=its)
        dx, itg = ctx.minres(to_dev(g), max_its=its, rtol=rtol, jacobi=jacobi)
        log("iterations", ito, itg)
        assert itg == ito
        assert rel(to_host(dx), xo) <= 1e-9
    d0, i0 = ctx.minres(to_dev(g), max_its=0, rtol=1e-5, jacobi=jacobi)
    assert i0 == 0 and not np.any(to_host(d0))
    d0, i0 = ctx.minres(to_dev(0.0 * g), max_its=5, rtol=1e-5, jacobi=jacobi)
    assert i0 == 0 and not np.any(to_host(d0))
    ctx.close()


@pytest.mark.parametrize("storage", ["tensor", "compact"])
@pytest.mark.parametrize("p,nq", CLASSES)
def test_classes(p, nq, storage):
    _check((3, 2), p, nq, storage, True, False)


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("ns,p,nq", EDGES)
def test_edges(ns, p, nq, general):
    _check(ns, p, nq, "tensor", not general, general)


@pytest.mark.parametrize("storage", ["tensor", "compact"])
@pytest.mark.parametrize("ns,p,nq", [((8, 8), 2, 4), ((5, 4), 3, 5)])
def test_mixed(ns, p, nq, storage):
    log("case", ns, p, nq, storage)
    pb, x, ctx = _setup(ns, p, nq, storage, "mixed")
    g = to_dev(pb.gradient(x))
    a, ia = ctx.minres(g, max_its=12, rtol=0.0)
    a = to_host(a)
    ctx.set_lanczos_bank_limit(0)
    b, ib = ctx.minres(g, max_its=12, rtol=0.0)
    assert ia == ib == 12
    assert rel(a, to_host(b)) <= 1e-4
    ctx.close()
