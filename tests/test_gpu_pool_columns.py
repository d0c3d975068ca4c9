"""A pool takes the column form of the compact setup and action for a class by the
elements resident together, so a mesh's form depends on its neighbours: its
gradient, energy, action and diagonal are to be bitwise the same alone (pencil
form) and beside a mesh large enough to put the class in column form.
"""
import numpy as np
import pytest

from oracle import basis
from paper_2205_12721_amd import inputs
from tests.gpu_common import log, make_case, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("p,nq,big", [(1, 4, (26, 26, 25)), (2, 4, (26, 26, 25)), (3, 4, (26, 26, 25)),
                                      (3, 5, (26, 26, 25)), (3, 6, (21, 20, 20)), (4, 7, (21, 20, 20))])
def test_alone_equals_beside_large(p, nq, big, precision):
    from paper_2205_12721_amd.tmop import Pool, request, request_bytes, solve_params
    log("case", p, nq, big, precision)
    ns = (3, 4, 3)
    pb, x = make_case(3, ns, p, nq, seed=61, amp=0.03)
    xb, _ = inputs.perturbed_box(3, big, p, basis.gll_nodes(p), 62, recipe="interior_jitter", amp=0.01)
    v = to_dev(inputs.gaussian_vector(pb.ndof, 63))
    xd, xbd = to_dev(x), to_dev(xb)
    small, large = (request(3, n, p, nq, precision=precision, storage="compact") for n in (ns, big))
    pool = Pool(request_bytes(*small) + request_bytes(*large), 2)
    slot = pool.admit(*small, solve_params(), xd)

    def results():
        pool.hessian_setup(slot, xd)
        return [np.array(pool.energy_mindet(slot, xd)), to_host(pool.gradient(slot, xd)),
                to_host(pool.hessian_apply(slot, v)), to_host(pool.hessian_diag(slot, v))]

    alone = results()
    pool.admit(*large, solve_params(), xbd)
    for a, b in zip(alone, results()):
        assert np.array_equal(a, b)
    pool.close()
