"""MINRES with the second Lanczos update inside the element kernel, where it stops before its cap, on
meshes of several workgroups with a ragged last one: iterations and solution are the oracle's, a repeated
call gives the same bits, nothing is left over for a zero right-hand side or for no iterations.
Tolerance as in the test of its capped solves: 1e-9 of dx.
"""
import numpy as np
import pytest

from oracle import solver
from tests.gpu_common import log, make_case, rel, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("jacobi", [True, False])
@pytest.mark.parametrize("storage", ["tensor", "compact"])
@pytest.mark.parametrize("dim,ns,p,nq", [(3, (5, 3, 3), 2, 4), (3, (4, 3, 5), 3, 5), (3, (5, 3, 3), 4, 6),
                                         (3, (9, 7, 8), 1, 3), (2, (17, 19), 2, 4), (2, (23, 9), 3, 5)])
def test_stops_as_the_oracle(dim, ns, p, nq, storage, jacobi):
    from paper_2205_12721_amd.tmop import Context
    log("case", dim, ns, p, nq, storage, jacobi)
    pb, x = make_case(dim, ns, p, nq, "interior_jitter", 0.02, seed=84)
    ctx = Context(dim, ns, p, nq, storage=storage)
    ctx.hessian_setup(to_dev(x))
    g = pb.gradient(x)
    gd = to_dev(g)
    minv = solver.jacobi_inverse(pb.diag(x), pb.ess)
    pre = (lambda r: minv * r) if jacobi else None
    for rtol in (0.3, 1e-3):
        xo, ito, _ = solver.minres(lambda v: pb.hvp(x, v), g, pre, rtol=rtol, maxit=60)
        assert 0 < ito < 60
        dx, itg = ctx.minres(gd, max_its=60, rtol=rtol, jacobi=jacobi)
        log("iterations", ito, itg)
        assert itg == ito
        a = to_host(dx)
        assert rel(a, xo) <= 1e-9
        # a capped solve in between, then the same again
        _, itc = ctx.minres(gd, max_its=2, rtol=0.0, jacobi=jacobi)
        assert itc == 2
        dx, itg = ctx.minres(gd, max_its=60, rtol=rtol, jacobi=jacobi)
        assert itg == ito and np.array_equal(a, to_host(dx))
    for b, cap in ((gd, 0), (to_dev(0.0 * g), 5)):
        d0, i0 = ctx.minres(b, max_its=cap, rtol=1e-5, jacobi=jacobi)
        assert i0 == 0 and not np.any(to_host(d0))
    ctx.close()
