"""Quad energy and gradient in column form (640 workgroups of the pencil form and
more) against the oracle, for every class at a size just above that line with a
ragged last workgroup, and just below it, as a box and as an element list,
with an ideal and with a sheared target.

The coordinates are of size 1 and the elements of size 1/n, n up to 203, so A
has a relative error of up to some n eps sum|G| < 1e-12: min det A within 1e-11;
F and the gradient, whose values are of the size of the deformation (2% of an
element and more) times that of A, within 1e-10.
"""
import numpy as np
import pytest

from tests.gpu_common import log, make_case, rel, to_dev, to_host

pytestmark = pytest.mark.gpu

CASES = [(1, 2, (203, 203)), (1, 3, (135, 133)), (1, 4, (103, 101)), (2, 3, (135, 133)),
         (2, 4, (103, 101)), (2, 5, (81, 80)), (3, 4, (103, 101)), (3, 5, (81, 80)), (3, 6, (68, 67)),
         (4, 5, (81, 80)), (4, 6, (68, 67)), (4, 7, (58, 57)),
         (2, 4, (101, 101)), (3, 5, (79, 81))]  # the last two: below the line

AMP = {1: 0.1, 2: 0.1, 3: 0.05, 4: 0.025}  # of the element size; every det stays positive


@pytest.mark.parametrize("target", ["ideal", "sheared"])
@pytest.mark.parametrize("p,nq,ns", CASES)
def test_against_oracle(p, nq, ns, target):
    import torch
    from paper_2205_12721_amd.tmop import Context
    log("case", p, nq, ns, target)
    W = None if target == "ideal" else np.array([[1.1, 0.2], [-0.1, 0.9]])
    pb, x = make_case(2, ns, p, nq, "interior_jitter", AMP[p], seed=91, W=W)
    F0, md0, g0 = pb.energy(x), pb.min_det(x), pb.gradient(x)
    xd = to_dev(x)
    box = Context(2, ns, p, nq, W=W)
    gen = Context(2, None, p, nq, W=W, elem_to_node=torch.as_tensor(pb.e2n).cuda(), num_nodes=pb.nx,
                  ess=torch.as_tensor(pb.ess.astype(np.uint8)).cuda())
    for ctx in (box, gen):
        F, md, g, g2 = ctx.energy_gradient(xd)
        g = to_host(g)
        assert (F, md) == ctx.energy_mindet(xd)
        assert np.array_equal(g, to_host(ctx.gradient(xd)))
        assert abs(F - F0) <= 1e-10 * F0
        assert abs(md - md0) <= 1e-11 * md0
        assert rel(g, g0) <= 1e-10
        assert abs(g2 - float(g @ g)) <= 1e-13 * float(g @ g)
        ctx.close()


@pytest.mark.parametrize("p,nq,ns", [(2, 4, (103, 101)), (3, 5, (81, 80))])
def test_inverted(p, nq, ns):
    from paper_2205_12721_amd.tmop import Context
    log("case", p, nq, ns)
    pb, x = make_case(2, ns, p, nq, "interior_jitter", AMP[p], seed=92)
    x = x.copy()
    mid = pb.nx // 2
    x[mid] += 3.0 / ns[0]  # one node past its neighbours
    ctx = Context(2, ns, p, nq)
    F, md = ctx.energy_mindet(to_dev(x))
    F1, md1, _, _ = ctx.energy_gradient(to_dev(x))
    assert F == F1 == float("inf") and md == md1
    assert md < 0 and abs(md - pb.min_det(x)) <= 1e-11 * abs(pb.min_det(x))
    ctx.close()
