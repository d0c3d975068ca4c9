"""The FP64 tensor setup on both sides of the element counts from which a point's entries are stored
together: the stored tensors give bitwise the action and the diagonal of those of the other route, the
one-pass setup with diagonal, on a mesh with inverted points too (whose entries are zero).
"""
import pytest

from oracle import basis
from paper_2205_12721_amd import inputs
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu


# bytes per element 45 * 8 * (n_q^3 rounded up to 16 points): n_q = 3 from 29128 elements on, n_q = 4 from
# 46604, n_q = 5 from 7282
@pytest.mark.parametrize("inverted", [False, True])
@pytest.mark.parametrize("p,nq,ns", [(1, 3, (61, 2, 238)), (1, 3, (61, 2, 239)), (2, 3, (61, 2, 238)),
                                     (2, 3, (61, 2, 239)), (1, 4, (31, 37, 40)), (1, 4, (31, 37, 41)),
                                     (2, 4, (31, 37, 41)), (2, 5, (28, 10, 26)), (2, 5, (28, 10, 27)),
                                     (3, 5, (28, 10, 27)), (4, 5, (28, 10, 27))])
def test_both_routes(p, nq, ns, inverted):
    import torch
    from paper_2205_12721_amd.tmop import Context
    log("case", p, nq, ns, inverted)
    x, _ = inputs.perturbed_box(3, ns, p, basis.gll_nodes(p), 97, recipe="interior_jitter", amp=0.02)
    xd = to_dev(x)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(98)
    if inverted:
        xd += 0.5 / max(ns) * torch.randn(x.size, dtype=torch.float64, device="cuda", generator=gen)
    v = torch.randn(x.size, dtype=torch.float64, device="cuda", generator=gen)
    ctx = Context(3, ns, p, nq, ess="none")
    assert (ctx.min_det(xd) < 0) == inverted
    ctx.hessian_setup(xd)
    a, da = ctx.hessian_apply(v), ctx.hessian_diag()
    db = ctx.hessian_setup_diag(xd)
    b = ctx.hessian_apply(v)
    assert torch.isfinite(a).all() and torch.equal(a, b) and torch.equal(da, db)
    ctx.close()
