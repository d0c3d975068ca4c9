"""Hex kernels in column form (energy, gradient, compact setup and action)
against the oracle where their workgroups end: a single element, a mesh with
every kind of remainder of the elements per workgroup (2 to 32 by class), a
sheared constant target, general connectivity with a mask.  Tolerances as in
the parity tests: 1e-11 in FP64, 2e-6 for the FP32 action.
"""
import numpy as np
import pytest

import oracle
from paper_2205_12721_amd import inputs
from tests.gpu_common import TOL64, log, make_case, rel, to_dev, to_host

pytestmark = pytest.mark.gpu

CLASSES = [(1, 2), (1, 3), (1, 4), (1, 9), (2, 3), (2, 4), (2, 5), (2, 9), (3, 4), (3, 5), (3, 6),
           (3, 9), (4, 5), (4, 6), (4, 7), (4, 9)]


def _check(ctx, pb, x, seed, mixed=False):
    xd = to_dev(x)
    F, md, gd, _ = ctx.energy_gradient(xd)
    assert (F, md) == ctx.energy_mindet(xd)
    assert abs(F - pb.energy(x)) <= TOL64 * abs(pb.energy(x))
    assert abs(md - pb.min_det(x)) <= 1e-12 * abs(pb.min_det(x))
    assert rel(to_host(gd), pb.gradient(x)) <= TOL64
    v = inputs.gaussian_vector(pb.ndof, seed)
    ctx.hessian_setup(xd)
    assert rel(to_host(ctx.hessian_apply(to_dev(v))), pb.hvp(x, v)) <= (2e-6 if mixed else TOL64)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("ns", [(1, 1, 1), (5, 3, 1), (3, 3, 3)])
@pytest.mark.parametrize("p,nq", CLASSES)
def test_remainders(p, nq, ns, precision):
    from paper_2205_12721_amd.tmop import Context
    log("case", p, nq, ns, precision)
    if p == 1 and ns == (1, 1, 1):
        ns = (1, 1, 2)  # the recipe moves no corner: one Q1 element stays a cube, its gradient 0
    # no node fixed: these meshes have few or no interior nodes
    # (the smooth recipe's displacement inverts a single element of high order)
    recipe = "interior_jitter" if ns == (1, 1, 1) else "smooth"
    pb, x = make_case(3, ns, p, nq, recipe, 0.03, seed=31, constrain=None)
    ctx = Context(3, ns, p, nq, storage="compact", precision=precision, ess="none")
    _check(ctx, pb, x, 32, precision == "mixed")
    ctx.close()


@pytest.mark.parametrize("p,nq", [(1, 2), (2, 4), (3, 4), (2, 5)])
def test_sheared_target_and_general_mesh(p, nq):
    import torch
    from paper_2205_12721_amd.tmop import Context
    log("case", p, nq)
    ns = (4, 3, 2)
    W = np.eye(3) + 0.2 * np.random.default_rng(33).standard_normal((3, 3))
    pb, x = make_case(3, ns, p, nq, seed=34, W=W)
    ctx = Context(3, ns, p, nq, storage="compact", W=W)
    _check(ctx, pb, x, 35)
    ctx.close()
    mask = np.random.default_rng(36).uniform(size=pb.ndof) < 0.3
    pbm = oracle.Problem(3, p, nq, pb.e2n, pb.nx, ess=mask)
    ctx = Context(3, None, p, nq, storage="compact", elem_to_node=torch.as_tensor(pb.e2n).cuda(),
                  num_nodes=pb.nx, ess=torch.as_tensor(mask.astype(np.uint8)).cuda())
    _check(ctx, pbm, x, 37)
    ctx.close()
