"""Gather coordinates (csrc/gather_point.h, compiled for the host) against extended
precision: floor and fraction of the radius index, and the fraction of the angle
step, over the grids, radius scales and angle counts that plans take. The bounds
are the roundings of the results, derived beside each."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1704_08364_amd", "csrc")
LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")
U = 2.0 ** -24

SOURCE = """
#include "gather_point.h"
extern "C" void points(double rscale, int V, int count, const int* x, const int* y, const int* guess,
                       const float* ri, int* m, float* g, float* f) {
    const bst::RadiusScale s = bst::radius_scale(rscale);
    const double vpi = V / M_PI;
    const float2 v = bst::split_float(vpi);
    for (int i = 0; i < count; ++i) {
        const bst::RadialIndex r = bst::radial_index(x[i] * x[i] + y[i] * y[i], ri[i], s);
        const double th = guess[i] * M_PI / V;
        const float4 d = bst::split_direction(std::cos(th), std::sin(th));
        m[i] = r.m;
        g[i] = r.g;
        f[i] = bst::angle_offset((float)x[i], (float)y[i], d, r, v.x, v.y);
    }
}
"""


@pytest.fixture(scope="module")
def points(tmp_path_factory):
    gxx = os.environ.get("BST_HOST_CXX", "g++")
    if shutil.which(gxx) is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("points")
    src, lib = d / "points.cpp", d / "points.so"
    src.write_text(SOURCE)
    subprocess.run([gxx, "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", f"-I{CSRC}", str(src), "-o", str(lib)], check=True)
    fn = C.CDLL(str(lib)).points
    fn.restype = None
    fn.argtypes = [C.c_double, C.c_int, C.c_int] + [C.c_void_p] * 7
    return fn


@pytest.mark.parametrize("G,rscale,V", [
    (16, 1.0, 16), (16, 0.25, 17), (64, 4.0, 40), (512, 1.0, 256), (1024, 2.0, 100), (1024, 0.5, 500),
    (2048, 1.0, 1001), (2048, 4.0, 2000), (4096, 1.0, 3001), (4096, 2.0, 4096), (8192, 1.0, 8192),
    (8192, 0.25, 6001), (8192, 1.0, 16384), (128, 1.0, 16384),
])
def test_point_index(points, G, rscale, V):
    rng = np.random.default_rng(G + V)
    k = 100000
    x = rng.integers(-G // 2 + 1, G // 2, k)
    y = rng.integers(0, G // 2 + 1, k)
    ok = (x * x + y * y > 0) & (x * x + y * y < (G // 2) ** 2) & ~((y == 0) & (x < 0))
    x, y = x[ok].astype(np.int32), y[ok].astype(np.int32)
    n = x.astype(np.int64) ** 2 + y.astype(np.int64) ** 2
    r = np.sqrt(n.astype(LD)) * LD(rscale)
    q = np.arctan2(y.astype(LD), x.astype(LD)) * LD(V) / PI
    # the angle at or below the point, or the next one where that is near (a coarse first guess)
    guess = np.minimum(np.floor(q), V - 1)
    guess = np.where((q - guess > 0.9) & (guess < V - 1), guess + 1, guess).astype(np.int32)
    # an inverse root as the hardware's: one ulp off either way
    ri = (1.0 / np.sqrt(n.astype(np.float32).astype(np.float64)))
    ri = (ri * (1.0 + rng.choice([-1, 0, 1], n.size) * 2.0 ** -24)).astype(np.float32)
    m = np.empty(n.size, np.int32)
    g = np.empty(n.size, np.float32)
    f = np.empty(n.size, np.float32)
    points(rscale, V, n.size, x.ctypes.data, y.ctypes.data, guess.ctypes.data, ri.ctypes.data, m.ctypes.data,
           g.ctypes.data, f.ctypes.data)

    assert np.array_equal(m, np.floor(r).astype(np.int32))
    assert not np.signbit(g).any()
    # the rounding of g < 1, and that of the residual 2 m g + g^2 < 1 over 2 r
    eg = np.abs(r - m - g.astype(LD)).astype(np.float64)
    assert np.all(eg <= 2.0 ** -25 * (1.0 + 0.5 / r)), eg.max()
    # the cross product's rounding, 1 - r rinv's (at most g / r before it), the
    # series' missing term (s^11 at s <= pi / V), and the last rounding
    off = q - guess
    ef = np.abs(off - f.astype(LD)).astype(np.float64)
    size = np.abs(off).astype(np.float64)
    bound = size * (U * (1.05 + 1.0 / r) + 0.0224 * (np.pi / V) ** 10) + np.where(size < 1.0, U / 2, U)
    assert np.all(ef <= bound), (ef / bound).max()
    print(f"G={G} P_r/P_c={rscale} V={V}: g {eg.max():.2e}, f {ef.max():.2e}")
