"""CPU check of the pool's vector tiles: the header's own rule is compiled into a host program.
Every workgroup of a slot's MINRES vector kernels sums one partial per tile of the slot, so
whatever the slot's size there are at most 1024 tiles; a tile is a whole number of entries per
lane (256 lanes), at least three, and no more than the limit asks for.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2205_12721_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "vec.hpp"
#include <cstdio>

int main()
{
    long bad = 0, checked = 0;
    auto check = [&](long n) {
        if (n < 1 || n > 0x7fffffffL) return;
        const long t = tmop::vtile_dofs((int)n), tiles = (n + t - 1) / t;
        const bool ok = t >= 768 && t % 256 == 0 && tiles <= 1024 &&
                        (t == 768 || (n + t - 256 - 1) / (t - 256) > 1024);
        ++checked;
        if (!ok && ++bad <= 5) std::printf("ndof %ld: tiles of %ld, %ld of them\n", n, t, tiles);
    };
    for (long n = 1; n < 3000000; ++n) check(n);
    for (long k = 1; k <= 8192; ++k)
        for (long d = -2; d <= 2; ++d) check(k * 262144 + d);
    for (long n = 1; n < 0x7fffffffL; n += 9973) check(n);
    std::printf("checked %ld bad %ld\n", checked, bad);
    return bad == 0 ? 0 : 1;
}
"""


def test_tiles_of_a_slot(tmp_path):
    cc = HIPCC if os.path.exists(HIPCC) else shutil.which("hipcc")
    if cc is None:
        pytest.skip("hipcc is not installed")
    src = tmp_path / "tiles.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "tiles"
    r = subprocess.run([cc, "-std=c++17", "-O2", "-I" + CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and " bad 0" in r.stdout, r.stdout + r.stderr
