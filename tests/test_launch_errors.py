"""Kernel launches that fail, on the CPU: a stand-in for the HIP runtime (host memory, launches that do
nothing and one of which can be told to fail) takes the runtime's place before the library is loaded.
Every launch of an evaluation fails in turn: the call has to say so (TMOP_ERR_HIP), since the results
it would return are those of the call before, and the next call, whose launches succeed, is accepted.
A MINRES call has to wait, before it returns with the error, for what it did launch: those kernels
report their progress to the word that the context's next solve reads.
"""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stdlib.h>
#include <string.h>
#include <stddef.h>
static long launches, fail_at, syncs, syncs_at_fail;
static int last;
void fake_fail_at(long k) { launches = 0; fail_at = k; last = 0; syncs_at_fail = -1; }
long fake_launches(void) { return launches; }
// synchronisations since the launch that failed (-1: none failed)
long fake_syncs_after_failure(void) { return syncs_at_fail < 0 ? -1 : syncs - syncs_at_fail; }
int __hipPushCallConfiguration(unsigned long long gx, unsigned gz, unsigned long long bx, unsigned bz,
                               size_t lds, void *s) { return 0; }
int __hipPopCallConfiguration(void *g, void *b, size_t *lds, void **s) { *lds = 0; *s = 0; return 0; }
int hipLaunchKernel(const void *f, unsigned long long gx, unsigned gz, unsigned long long bx, unsigned bz,
                    void **a, size_t lds, void *s)
{
    if (++launches == fail_at) { syncs_at_fail = syncs; return last = 9; }
    return 0;
}
int hipMalloc(void **p, size_t n) { *p = calloc(1, n ? n : 1); return *p ? 0 : 2; }
int hipHostMalloc(void **p, size_t n, unsigned f) { return hipMalloc(p, n); }
int hipHostGetDevicePointer(void **d, void *h, unsigned f) { *d = h; return 0; }
int hipFree(void *p) { free(p); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { memcpy(d, s, n); return 0; }
int hipStreamSynchronize(void *s) { ++syncs; return 0; }
int hipStreamQuery(void *s) { return 0; }
int hipPeekAtLastError(void) { return last; }
int hipGetLastError(void) { int e = last; last = 0; return e; }
int hipEventDestroy(void *e) { return 0; }
"""

DRIVER = r"""
import ctypes, sys
import numpy as np
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # before the library: its calls go here
rt.fake_fail_at.argtypes = [ctypes.c_long]
rt.fake_launches.restype = rt.fake_syncs_after_failure.restype = ctypes.c_long
from paper_2205_12721_amd import tmop
L = ctypes.CDLL(tmop.LIB_PATH)
for k, a in tmop.SIGNATURES.items():
    getattr(L, k).argtypes = a
HIP, OK, INVERTED = 10, 0, 3

def context(dim, ns, p, nq, storage=0):
    md = tmop.MeshDesc()
    md.dim, md.order_p, md.nx, md.ny, md.nz = dim, p, ns[0], ns[1], ns[2] if dim == 3 else 0
    prm = tmop.Params()
    prm.metric, prm.nq1d, prm.hess_storage = 2 if dim == 2 else 303, nq, storage
    h = ctypes.c_void_p()
    rt.fake_fail_at(0)
    assert L.tmop_create(ctypes.byref(h), ctypes.byref(md), ctypes.byref(prm), None) == OK
    n = dim * int(np.prod([v * p + 1 for v in ns]))
    return h, np.zeros(n), np.zeros(n)

def every_launch(name, call, accepted=(OK,), after=lambda: True):
    rt.fake_fail_at(0)
    assert call() in accepted
    n = rt.fake_launches()
    assert n >= 1, name
    for k in range(1, n + 1):
        rt.fake_fail_at(k)
        assert call() == HIP, "%s: launch %d of %d failed unnoticed" % (name, k, n)
        assert after(), "%s: launch %d of %d" % (name, k, n)
        rt.fake_fail_at(0)
        assert call() in accepted, "%s after a failure" % name
    print("checked", name, n)

P = lambda a: a.ctypes.data_as(ctypes.c_void_p)
"""

EVALUATIONS = DRIVER + r"""
for dim, ns, p, nq in [(2, (3, 3), 2, 4), (2, (90, 90), 1, 3), (3, (2, 3, 2), 2, 4), (3, (24, 24, 24), 2, 4)]:
    for limited in (False, True):
        h, x, g = context(dim, ns, p, nq)
        if limited:
            assert L.tmop_set_limiting(h, P(x), 1.0, 1.0) == OK
        F, m, g2 = ctypes.c_double(), ctypes.c_double(), ctypes.c_double()
        tag = " %s %s" % (ns, limited)
        every_launch("energy" + tag, lambda: L.tmop_energy(h, P(x), F))
        every_launch("min_det" + tag, lambda: L.tmop_min_det(h, P(x), m))
        every_launch("energy_mindet" + tag, lambda: L.tmop_energy_mindet(h, P(x), F, m))
        every_launch("gradient" + tag, lambda: L.tmop_gradient(h, P(x), P(g)))
        every_launch("energy_gradient" + tag, lambda: L.tmop_energy_gradient(h, P(x), F, m, P(g), g2))
        # (nothing runs here, so the initial mesh has min det 0)
        sp, rep = tmop.SolveParams(1e-8, 3, 5, 1e-12, 3, 1, 0.0), tmop.SolveReport()
        every_launch("solve" + tag, lambda: L.tmop_solve(h, P(x), sp, rep), (INVERTED,))
        L.tmop_destroy(h)
print("done")
"""


MINRES = DRIVER + r"""
for dim, ns, p, nq, bank in [(2, (3, 3), 2, 4, None), (2, (90, 90), 1, 3, None), (2, (90, 90), 1, 3, 0),
                             (3, (4, 3, 2), 2, 4, None), (3, (24, 24, 24), 1, 3, None),
                             (3, (17, 17, 17), 2, 5, None)]:
    h, b, dx = context(dim, ns, p, nq, storage=1)
    assert L.tmop_hessian_setup(h, P(b)) == OK
    if bank is not None:
        assert L.tmop_set_lanczos_bank_limit(h, bank) == OK
    every_launch("minres %s" % (ns,), lambda: L.tmop_minres(h, P(b), P(dx), 12, 1e-9, 0, None),
                 after=lambda: rt.fake_syncs_after_failure() >= 1)
    L.tmop_destroy(h)
print("done")
"""


def _run(tmp_path, script):
    from paper_2205_12721_amd import tmop
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("gcc is not installed")
    if not os.path.exists(tmop.LIB_PATH):
        pytest.fail("libtmop_hip.so is not built (run __graft_entry__.build())")
    (tmp_path / "rt.c").write_text(RUNTIME)
    rt = str(tmp_path / "librt_fake.so")
    r = subprocess.run([cc, "-O1", "-w", "-shared", "-fPIC", str(tmp_path / "rt.c"), "-o", rt],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([sys.executable, "-c", script, rt], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("done\n"), r.stdout[-2000:] + r.stderr[-2000:]


def test_failed_launch_of_an_evaluation_is_reported(tmp_path):
    _run(tmp_path, EVALUATIONS)


def test_failed_minres_waits_for_what_it_launched(tmp_path):
    _run(tmp_path, MINRES)
