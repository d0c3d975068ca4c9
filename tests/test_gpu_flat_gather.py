"""The tensor action at n_q = 5 on both sides of the 4096 workgroups (two elements each) from which
its gather runs over components as well: bitwise the action in another tile shape, which gathers by node,
with the boundary, a mask and no DoF fixed, on the box and on the same mesh as an element list.
"""
import pytest

from oracle import basis, mesh
from paper_2205_12721_amd import inputs
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ess", ["boundary", "mask", "none"])
@pytest.mark.parametrize("p,precision", [(2, "fp64"), (3, "fp64"), (3, "mixed")])
@pytest.mark.parametrize("ns", [(30, 13, 21), (32, 32, 8), (27, 19, 17)])  # 4095, 4096, 4361 (one ragged)
def test_limit(p, precision, ns, ess):
    import torch
    from paper_2205_12721_amd.tmop import Context
    log("case", p, precision, ns, ess)
    e2n, nx = mesh.box_topology(3, ns, p)
    x, _ = inputs.perturbed_box(3, ns, p, basis.gll_nodes(p), 95, recipe="interior_jitter", amp=0.02)
    xd = to_dev(x)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(96)
    v = torch.randn(x.size, dtype=torch.float64, device="cuda", generator=gen)
    if ess == "mask":
        ess = (torch.rand(x.size, device="cuda", generator=gen) < 0.2).to(torch.uint8)
    ways = [dict(n=ns)]
    if not isinstance(ess, str) or ess == "none":
        ways.append(dict(elem_to_node=torch.as_tensor(e2n).to(torch.int32).cuda(), num_nodes=nx))
    for kw in ways:
        ctx = Context(3, p=p, nq1d=5, ess=ess, precision=precision, **kw)
        ctx.hessian_setup(xd)
        ctx.set_tile(2)  # the base shape (another may have been tuned before)
        a = ctx.hessian_apply(v)
        ctx.set_tile(1)
        b = ctx.hessian_apply(v)
        assert torch.isfinite(a).all() and torch.equal(a, b)
        ctx.close()
