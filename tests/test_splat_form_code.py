"""The rasterizers' decisions about a splat's quadratic form, as raster_common.h
takes them: the header is compiled for the host (contraction off and on, the
reciprocal exact and an ulp off either way) and its own functions are called.  A
splat walked without the tests on the power's sign and on the clamp needs neither,
and a splat culled for a rectangle of pixels reaches 1/255 at none of them."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

F = np.float32
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_08743_amd", "csrc")

# what the header needs of the HIP headers, for a host compiler
SHIM = r"""
#pragma once
#include <cmath>
#include <cstdint>
#define __device__
#define __host__
#define __forceinline__ inline
struct uint2 { uint32_t x, y; };
struct float4 { float x, y, z, w; };
struct double2 { double x, y; };
typedef void *hipStream_t;
typedef int hipError_t;
inline int rcp_ulps = 0;
inline float rcp_shim(float x) {
    float r = 1.f / x;
    for (int k = 0; k < rcp_ulps; k++) r = std::nextafterf(r, INFINITY);
    for (int k = 0; k > rcp_ulps; k--) r = std::nextafterf(r, -INFINITY);
    return r;
}
#define __builtin_amdgcn_rcpf rcp_shim
#define __builtin_amdgcn_exp2f exp2f
#define __builtin_amdgcn_mbcnt_lo(m, x) (x)
#define __builtin_amdgcn_mbcnt_hi(m, x) (x)
#define __fmaf_rn fmaf
using std::fabs; using std::fmax; using std::fmin;
"""
CODE = r"""
#include "raster_common.h"
using namespace gsp;
extern "C" {
void set_rcp(int ulps) { rcp_ulps = ulps; }
float lo_no_clamp(void) { return kLoNoClamp; }
void plain(int n, const float *A, const float *B, const float *C, const float *lo, uint8_t *out) {
    for (int k = 0; k < n; k++) out[k] = plain_splat(A[k], B[k], C[k], lo[k]);
}
// p2 at offsets (dx, dy), and the alpha before the clamp
void power(int n, const float *A, const float *B, const float *C, const float *lo, const float *dx, const float *dy,
           float *p2, float *alpha) {
    for (int k = 0; k < n; k++) {
        const ColTerms t = col_terms(StagedA{dx[k], 0.f, A[k], B[k]}, 0.f);
        p2[k] = splat_p2(t, C[k], dy[k]);
        alpha[k] = splat_alpha_pre(p2[k], lo[k]);
    }
}
// over a w x h rectangle of pixels with the centre at (u, v): kept by the
// bound; blended at some pixel
void rect(int n, int w, int h, const float *A, const float *B, const float *C, const float *lo, const float *u,
          const float *v, uint8_t *keep, uint8_t *hit) {
    for (int k = 0; k < n; k++) {
        keep[k] = SplatForm(A[k], B[k], C[k], lo[k]).reaches(u[k] - (float)(w - 1), u[k], v[k] - (float)(h - 1), v[k]);
        hit[k] = 0;
        for (int x = 0; x < w; x++) {
            const ColTerms t = col_terms(StagedA{u[k], v[k], A[k], B[k]}, (float)x);
            for (int y = 0; y < h; y++) {
                const float p2 = splat_p2(t, C[k], v[k] - (float)y);
                hit[k] |= p2 <= 0.f && fminf(kAlphaMax, splat_alpha_pre(p2, lo[k])) >= kAlphaMin;
            }
        }
    }
}
void bands(int n, const float *A, const float *B, const float *C, const float *lo, const float *u, const float *v,
           uint32_t *out) {
    for (int k = 0; k < n; k++) out[k] = band_mask(u[k], v[k], A[k], B[k], C[k], lo[k]);
}
}
"""


@pytest.fixture(scope="module", params=["off", "fast"])
def code(request, tmp_path_factory):
    d = tmp_path_factory.mktemp("form")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(SHIM)
    (d / "form.cpp").write_text(CODE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-mfma", f"-ffp-contract={request.param}", "-w", "-shared", "-fPIC",
                    f"-I{d}", f"-I{CSRC}", "-o", str(d / "form.so"), str(d / "form.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "form.so"))
    lib.lo_no_clamp.restype = ctypes.c_float
    return lib


def _call(fn, ints, arrays, outs):
    n = len(arrays[0])
    res = [np.zeros(n, t) for t in outs]
    arrays = [np.ascontiguousarray(a, F) for a in arrays]
    fn(ctypes.c_int(n), *[ctypes.c_int(i) for i in ints], *[a.ctypes.data_as(ctypes.c_void_p) for a in arrays + res])
    return res


def _forms(rng, n, slack, lo_exp):
    """Base-2 conics with B^2 = 4 A C (1 - slack), both signs of B."""
    A = -np.exp2(rng.uniform(lo_exp, 1.3, n)).astype(F)
    C = -np.exp2(rng.uniform(lo_exp, 1.3, n)).astype(F)
    B = (np.sqrt(4.0 * A.astype(np.float64) * C * (1 - slack)) * rng.choice([-1, 1], n)).astype(F)
    return A, B, C


# extents from a fraction of a pixel to thousands, and (where A C leaves the
# normal numbers) to 1e20 pixels
@pytest.mark.parametrize("lo_exp", [-24, -140])
@pytest.mark.parametrize("slack", [-1e-6, 0.0, 1e-7, 1e-4, 1.01e-4, 1e-3, 0.1, 1.0])
def test_plain_splats_have_no_positive_power(code, slack, lo_exp):
    rng = np.random.default_rng(5)
    n = 200_000
    A, B, C = _forms(rng, n, slack, lo_exp)
    lo = np.full(n, -1.0, F)
    plain = _call(code.plain, [], [A, B, C, lo], [np.uint8])[0].astype(bool)
    if lo_exp == -24 and slack >= 1.01e-4:
        assert plain.mean() > 0.99
    # offsets along the form's long axis, where it is closest to zero, and off it
    dy = (rng.uniform(-1, 1, n) * np.exp2(rng.uniform(-12, 17, n))).astype(F)
    along = -0.5 * B.astype(np.float64) * dy / A
    dx = along * (1 + rng.choice([0, 1e-7, 1e-5, 1e-3, 0.5], n) * rng.standard_normal(n))
    inside = np.abs(dx) < 2 ** 17
    p2, _ = _call(code.power, [], [A, B, C, lo, np.where(inside, dx, 0.0), dy], [F, F])
    assert (p2[plain & inside] <= 0).all()


def test_plain_splats_stay_below_the_clamp(code):
    n = 100_000
    lo = np.concatenate([np.linspace(-0.0155 - 1e-4, -0.0155 + 1e-4, n // 2), np.linspace(-8, 0, n // 2)]).astype(F)
    A = np.full(n, -1.0, F)
    B = np.zeros(n, F)
    plain = _call(code.plain, [], [A, B, A, lo], [np.uint8])[0].astype(bool)
    assert np.array_equal(plain, lo <= F(code.lo_no_clamp()))
    _, alpha = _call(code.power, [], [A, B, A, lo, B, B], [F, F])
    # below 0.99 by 2^-11 of it, for an exponential that is an ulp (2^-23) off
    assert plain.any() and (alpha[plain] < 0.99 * (1 - 2.0 ** -11)).all()


@pytest.mark.parametrize("ulps", [-1, 0, 1])
@pytest.mark.parametrize("w,h", [(8, 8), (16, 4)])
@pytest.mark.parametrize("slack", [-1e-6, 0.0, 1e-4, 0.05, 1.0])
def test_culled_splats_reach_no_pixel(code, w, h, slack, ulps):
    rng = np.random.default_rng(6)
    n = 40_000
    A, B, C = _forms(rng, n, slack, -24)
    lo = np.log2(rng.uniform(1 / 255, 1, n)).astype(F)
    # centres from inside the rectangle to some extents away from it
    ext = np.sqrt(8.0 / np.minimum(-A, -C).astype(np.float64))
    far = rng.choice([0, 1], n) * np.minimum(ext, 4000)
    u = rng.uniform(-1, w, n) + rng.uniform(-1, 1, n) * far
    v = rng.uniform(-1, h, n) + rng.uniform(-1, 1, n) * far
    code.set_rcp(ulps)
    keep, hit = _call(code.rect, [w, h], [A, B, C, lo, u, v], [np.uint8, np.uint8])
    assert 0.02 < keep.mean() < 0.98 and hit.any()
    assert not (hit & ~keep & 1).any()
    if (w, h) == (16, 4):   # the backward's bands are this rectangle at rows 0, 4, 8, 12
        mask = _call(code.bands, [], [A, B, C, lo, u, v], [np.uint32])[0]
        for q in range(4):
            kq = _call(code.rect, [w, h], [A, B, C, lo, u, v.astype(F) - F(4 * q)], [np.uint8, np.uint8])[0]
            same = (mask >> q & 1) == kq
            # (v - 4 q is rounded before the rectangle's edges here, behind them there)
            assert same.mean() > 0.999
    code.set_rcp(0)
