"""The compact setup's choice of form on large hex meshes.

Rate: the setup's time per element does not grow once its data passes the 256 MB last-level cache by
more than memory asks for.  In column form, whose stores then reach memory in parts, it grew by 1.56
to 1.81 (n_q = 2 and 3 in FP64); in pencil form by 0.97 to 1.29.  The bound is 1.45.

Limits: on both sides of the sizes between which the column form is used, the stored data gives
bitwise the action of the data that the one-pass setup with diagonal (always in pencil form) stores.
"""
import time

import pytest

from oracle import basis
from paper_2205_12721_amd import inputs
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu


def _context(ns, p, nq, precision):
    from paper_2205_12721_amd.tmop import Context
    x, _ = inputs.perturbed_box(3, ns, p, basis.gll_nodes(p), 91, recipe="interior_jitter", amp=0.02)
    return Context(3, ns, p, nq, precision=precision, storage="compact", ess="none"), to_dev(x)


@pytest.mark.parametrize("p,nq,mid,large", [(1, 2, 60, 112), (1, 3, 42, 80), (2, 3, 41, 56)])
def test_rate_of_large_setups(p, nq, mid, large):
    import torch

    def per_element(n):
        ctx, x = _context((n, n, n), p, nq, "fp64")
        best = 1e9
        for k in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(20):
                ctx.hessian_setup(x)
            torch.cuda.synchronize()
            if k:
                best = min(best, time.perf_counter() - t)
        ctx.close()
        return best / 20 / n ** 3

    a, b = per_element(mid), per_element(large)
    log("case", p, nq, "ns per element: %d^3 %.3f, %d^3 %.3f" % (mid, a * 1e9, large, b * 1e9))
    assert b <= 1.45 * a


# element counts around the limits: (1, 4) FP64 16384 .. 40329; (3, 5) FP64 8192 .. 20164;
# (4, 6) FP64 from 16384 on; (1, 2) FP32 131072 .. 655360
@pytest.mark.parametrize("p,nq,precision,ns", [
    (1, 4, "fp64", (16, 32, 32)), (1, 4, "fp64", (34, 34, 34)), (1, 4, "fp64", (34, 34, 35)),
    (3, 5, "fp64", (16, 16, 32)), (3, 5, "fp64", (27, 27, 27)), (3, 5, "fp64", (27, 27, 28)),
    (4, 6, "fp64", (25, 26, 25)), (4, 6, "fp64", (25, 26, 26)),
    (1, 2, "mixed", (64, 64, 32)), (1, 2, "mixed", (64, 128, 80)), (1, 2, "mixed", (64, 128, 81))])
def test_limits(p, nq, precision, ns):
    import torch
    log("case", p, nq, precision, ns)
    ctx, x = _context(ns, p, nq, precision)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(92)
    v = torch.randn(x.numel(), dtype=torch.float64, device="cuda", generator=gen)
    ctx.hessian_setup(x)
    a = ctx.hessian_apply(v)
    ctx.hessian_setup_diag(x)
    b = ctx.hessian_apply(v)
    assert torch.isfinite(a).all() and torch.equal(a, b)
    ctx.close()
