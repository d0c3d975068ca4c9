"""The end of the energy and of the one-pass energy + gradient: the reduction
of the workgroups' partial sums, which takes one slice up to 1024 of them, and
the gather of g with |g|^2, which one workgroup does together with it up to
4096 nodes.  Quads of one node and 16 points per element side put either line
at a small mesh; sizes are the last below and the first above each.

F and min det A of the two calls are the same sums, so bitwise equal; |g|^2
against numpy: n terms added in any order differ by at most n eps relative,
and by far less in a tree: 1e-13.
"""
import numpy as np
import pytest

from tests.gpu_common import TOL64, log, make_case, rel, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("ns,nq", [((1, 2), 4), ((63, 63), 2), ((63, 64), 2), ((128, 128), 4),
                                   ((129, 128), 4), ((181, 181), 4), ((300, 257), 3)])
def test_energy_gradient_end(ns, nq, general):
    import torch
    from paper_2205_12721_amd.tmop import Context
    log("case", ns, nq, general)
    pb, x = make_case(2, ns, 1, nq, "interior_jitter", 0.002, seed=51, constrain=None)
    x = x + 1e-4 * np.random.default_rng(52).standard_normal(x.size)
    if general:
        ctx = Context(2, None, 1, nq, elem_to_node=torch.as_tensor(pb.e2n).cuda(), num_nodes=pb.nx,
                      ess="none")
    else:
        ctx = Context(2, ns, 1, nq, ess="none")
    xd = to_dev(x)
    for _ in range(2):
        F, md, gd, g2 = ctx.energy_gradient(xd)
        assert (F, md) == ctx.energy_mindet(xd)
        g = to_host(gd)
        assert abs(F - pb.energy(x)) <= TOL64 * abs(pb.energy(x))
        assert abs(md - pb.min_det(x)) <= 1e-12 * abs(pb.min_det(x))
        assert rel(g, pb.gradient(x)) <= TOL64
        assert abs(g2 - float(g @ g)) <= 1e-13 * float(g @ g)
    ctx.close()
