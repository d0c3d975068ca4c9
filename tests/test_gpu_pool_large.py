"""Pool slots with more than three DoFs per lane of a vector tile (above 786432 DoFs), and the
largest with three: the first Newton step of the slot against a context's on the same mesh.  Both
run the same recurrences on the same element kernels and differ in the order of their sums, so the
bounds are those of the step's parity with the oracle: 1e-9 of the step in FP64, 1e-4 in mixed
precision, the energies within 1e-10 and 1e-6 of the initial one.
"""
import pytest

from oracle import basis
from paper_2205_12721_amd import inputs
from tests.gpu_common import log, rel, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,bank", [("fp64", False), ("fp64", True), ("mixed", False)])
@pytest.mark.parametrize("dim,ns,p,nq", [(3, (63, 63, 63), 1, 2), (3, (63, 63, 64), 1, 2),
                                         (3, (18, 18, 17), 4, 6), (2, (640, 641), 1, 3)])
def test_first_step(dim, ns, p, nq, precision, bank):
    from paper_2205_12721_amd.tmop import Context, Pool, request, request_bytes, solve_params
    log("case", dim, ns, p, nq, precision, bank)
    x, _ = inputs.perturbed_box(dim, ns, p, basis.gll_nodes(p), 71, recipe="interior_jitter", amp=0.02)
    kw = dict(precision=precision, storage="compact")
    ctx = Context(dim, ns, p, nq, **kw)
    xc = to_dev(x)
    ref = ctx.solve(xc, max_newton=1, max_minres=8)
    ctx.close()
    req = request(dim, ns, p, nq, **kw)
    pool = Pool(request_bytes(*req) + (16 * x.size * 8 + (1 << 20) if bank else 0), 1, lanczos_bank=bank)
    xp = to_dev(x)
    slot = pool.admit(*req, solve_params(max_newton=1, max_minres=8), xp)
    while pool.step():
        pass
    done, rep = pool.poll(slot)
    pool.result(slot, xp)
    pool.close()
    assert done and rep["status_name"] == ref["status_name"] == "ERR_NOT_CONVERGED"
    assert rep["minres_its_total"] == ref["minres_its_total"] == 8
    assert rep["halvings_total"] == ref["halvings_total"]
    step, step_ref = to_host(xp) - x, to_host(xc) - x
    assert rel(step, step_ref) <= (1e-9 if precision == "fp64" else 1e-4)
    assert abs(rep["F"] - ref["F"]) <= (1e-10 if precision == "fp64" else 1e-6) * ref["F0"]
