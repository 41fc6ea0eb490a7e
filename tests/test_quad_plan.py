"""Plans of the quadrature Dirichlet data, on the CPU: which meshes they take, the work space they ask for, and
that the split of a source's sum follows the mesh alone.  The meshes are all that a context can be made for (its
coarsest level has at most 16 nodes per axis: 1 to 8 elements an axis, halved together)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2510_21213_amd")
LIB = os.path.join(PKG, "libdgpoisson.so")

SOURCE = r"""
#include <cstdio>
#include "dg_internal.h"
#include "dg_kernels.h"
int main() {
    using namespace dg;
    const long long cap = 8LL << 20;  // doubles of the fixed work space
    long long meshes = 0, bad = 0;
    for (int k = 0; k <= 9; ++k)
        for (int p = 1; p <= 7; ++p)
            for (int a = 1; a <= 8; ++a)
                for (int b = 1; b <= a; ++b)
                    for (int c = 1; c <= b; ++c) {
                        LevelHost L;
                        L.n = p + 1;
                        L.p = p;
                        L.E[0] = a << k, L.E[1] = b << k, L.E[2] = c << k;
                        const long long N[3] = {1LL * L.E[0] * L.n, 1LL * L.E[1] * L.n, 1LL * L.E[2] * L.n};
                        L.ndof = N[0] * N[1] * N[2];
                        if (L.ndof > 5000000000LL) continue;  // level tables and vectors of more exceed the memory
                        ++meshes;
                        const long long nface = 2 * (N[0] * N[1] + N[0] * N[2] + N[1] * N[2]);
                        bool ok = quad_indices_fit(L) == (nface <= (1LL << 30));
                        if (!quad_indices_fit(L)) continue;
                        long long parts = 0;
                        for (int n : {1, 2, 3, 4, 5, 8, 9, 12, 13, 16, 17, 20, 28, 31, 32, 33, 36, 48, 49, 64, 96}) {
                            const QuadPlan P = quad_plan(L, n);
                            // records of at most 8 GiB, or of the sources in fours up to 48
                            const long long fields = n < 4 ? n : n > 48 ? 48 : (n + 3) / 4 * 4;
                            ok &= P.rmax >= 1 && P.nface == nface && P.rec_len >= L.ndof * (n < 4 ? n : 4) &&
                                  (P.rec_len <= (1LL << 30) || P.rec_len <= L.ndof * fields);
                            // the same parts for every source
                            const int widest = n < P.rmax ? n : P.rmax;
                            ok &= P.part_len % (widest * nface) == 0 && (!parts || parts == P.part_len / (widest * nface));
                            parts = P.part_len / (widest * nface);
                            // the fixed work space takes every mesh whose field fits it
                            const QuadPlan B = quad_plan_bounded(L, n, cap);
                            ok &= (B.rmax >= 1) == (L.ndof <= cap) && (!B.rmax || B.rec_len + B.part_len <= cap);
                        }
                        if (!ok && ++bad < 10) std::printf("E %d %d %d p %d\n", L.E[0], L.E[1], L.E[2], p);
                    }
    std::printf("%lld meshes, %lld wrong\n", meshes, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
def test_plans_over_every_mesh(tmp_path):
    src, exe = tmp_path / "plans.cpp", tmp_path / "plans"
    src.write_text(SOURCE)
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + PKG + "/csrc", str(src),
                    LIB, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + PKG + ":/opt/rocm/lib", "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stdout
