"""The compact action's choice of form on hex meshes, on both sides of the element counts between which
the base tile shape runs in column form: the action is bitwise that of another tile shape, which always
runs in pencil form.
"""
import pytest

from oracle import basis
from paper_2205_12721_amd import inputs
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu


# (1, 3) FP64 9216 .. 80659, FP32 .. 161319; (2, 3) FP64 9216 .. 80659; (1, 4) FP64 4096 .. 40329;
# (2, 5) FP64 4096 .. 20164, FP32 from 16384 on; epb: elements per workgroup of another shape
@pytest.mark.parametrize("p,nq,precision,epb,ns", [
    (1, 3, "fp64", 4, (96, 96, 1)), (1, 3, "fp64", 4, (43, 43, 43)), (1, 3, "fp64", 4, (44, 43, 43)),
    (1, 3, "mixed", 18, (54, 54, 55)), (1, 3, "mixed", 18, (54, 55, 55)),
    (2, 3, "fp64", 4, (43, 43, 43)), (2, 3, "fp64", 4, (44, 43, 43)),
    (1, 4, "fp64", 2, (34, 34, 34)), (1, 4, "fp64", 2, (34, 34, 35)),
    (2, 5, "fp64", 1, (27, 27, 27)), (2, 5, "fp64", 4, (27, 27, 28)),
    (2, 5, "mixed", 1, (25, 25, 26)), (2, 5, "mixed", 1, (25, 26, 26))])
def test_limits(p, nq, precision, epb, ns):
    import torch
    from paper_2205_12721_amd.tmop import Context
    log("case", p, nq, precision, epb, ns)
    x, _ = inputs.perturbed_box(3, ns, p, basis.gll_nodes(p), 93, recipe="interior_jitter", amp=0.02)
    ctx, xd = Context(3, ns, p, nq, precision=precision, storage="compact"), to_dev(x)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(94)
    v = torch.randn(x.size, dtype=torch.float64, device="cuda", generator=gen)
    ctx.hessian_setup(xd)
    ctx.set_tile({2: 32, 3: 9, 4: 4, 5: 2}[nq])  # the base shape (another may have been tuned before)
    a = ctx.hessian_apply(v)
    ctx.set_tile(epb)
    b = ctx.hessian_apply(v)
    assert torch.isfinite(a).all() and torch.equal(a, b)
    ctx.close()
