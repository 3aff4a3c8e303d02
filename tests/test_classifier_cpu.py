"""The FP32 pixel classifier with its guard band against the FP64 one, over the
offsets of the angular-weight table, on the CPU: the device functions of
kernels.h are compiled for the host, with the hardware's approximate
reciprocal, square root and their product off by up to an ulp either way.
Every sub-point outside the guard band must get the FP64 classifier's pixel
(inside it the kernels take that one)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# what kernels.h needs of the HIP runtime; the wave helpers are not called
STUB = r"""
#pragma once
#include <cmath>
#include <cstring>
#include <cstdint>
#define __device__
#define __global__
#define __host__
extern int u_rcp, u_rsq, u_sqrt;
inline float off_by(float v, int n) { return n == 0 ? v : std::nextafterf(v, n > 0 ? INFINITY : -INFINITY); }
inline float __builtin_amdgcn_rcpf(float x) { return off_by((float)(1.0 / (double)x), u_rcp); }
inline float __builtin_amdgcn_rsqf(float x) { return off_by((float)(1.0 / std::sqrt((double)x)), u_rsq); }
inline float __builtin_amdgcn_sqrtf(float x) { return x > 0.0f ? off_by(std::sqrt(x), u_sqrt) : 0.0f; }
inline double __dsqrt_rn(double x) { return std::sqrt(x); }
inline float __int_as_float(int v) { float f; std::memcpy(&f, &v, 4); return f; }
inline int __float_as_int(float f) { int v; std::memcpy(&v, &f, 4); return v; }
inline int __double2loint(double d) { int64_t v; std::memcpy(&v, &d, 8); return (int)v; }
inline int __double2hiint(double d) { int64_t v; std::memcpy(&v, &d, 8); return (int)(v >> 32); }
inline double __hiloint2double(int h, int l) { int64_t v = ((int64_t)h << 32) | (uint32_t)l; double d; std::memcpy(&d, &v, 8); return d; }
inline int __popc(unsigned v) { return __builtin_popcount(v); }
inline unsigned __lane_id() { return 0; }
inline int __builtin_amdgcn_readfirstlane(int v) { return v; }
inline int __builtin_amdgcn_readlane(int v, int) { return v; }
inline int __builtin_amdgcn_update_dpp(int, int v, int, int, int, bool) { return v; }
inline unsigned __builtin_amdgcn_mbcnt_lo(unsigned, unsigned) { return 0; }
inline unsigned __builtin_amdgcn_mbcnt_hi(unsigned, unsigned) { return 0; }
template <typename T> T max(T a, T b) { return a > b ? a : b; }
using std::fabs; using std::floor; using std::sqrt; using std::atan2;
"""

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include <random>
#include "kernels.h"
int u_rcp, u_rsq, u_sqrt;
// argv: N_side, s, 2 / theta, offsets of a ratio at most; prints sub-points, doubtful ones, wrong ones
int main(int, char **v)
{
    const int ns = atoi(v[1]), s = atoi(v[2]), reach = atoi(v[3]);
    const long most = atol(v[4]);
    const float tol = 1e-5f * (ns > 2 ? (float)ns : 2.0f);   // the sweep's guard band
    long n = 0, doubt = 0, wrong = 0;
    std::mt19937 rng(5);
    for (int ri = 0; ri < 6; ++ri) {
        const int r = 1 << ri, w = (reach + 1) * r, nw = 2 * w + 1;
        const long all = (long)nw * nw * nw, take = all < most ? all : most;
        for (long q = 0; q < take; ++q) {
            const long k = take == all ? q : (long)(((unsigned long)rng() << 20 ^ rng()) % (unsigned long)all);
            const int b[3] = {(int)(k / ((long)nw * nw)) - w, (int)(k / nw % nw) - w, (int)(k % nw) - w};
            if (b[0] <= 0 && b[0] + r > 0 && b[1] <= 0 && b[1] + r > 0 && b[2] <= 0 && b[2] + r > 0) continue;   // holds the target
            const float step = (float)r * (1.0f / (float)s);
            for (int l = 0; l < s * s * s; ++l) {
                const int ia = l / (s * s), ib = (l / s) % s, ic = l % s;
                const float x = fmaf(((float)ia + 0.5f) + (float)tr::kJit0, step, 0.5f * (float)(2 * b[0] - 1));
                const float y = fmaf(((float)ib + 0.5f) + (float)tr::kJit1, step, 0.5f * (float)(2 * b[1] - 1));
                const float z = fmaf(((float)ic + 0.5f) + (float)tr::kJit2, step, 0.5f * (float)(2 * b[2] - 1));
                const int pd = tr::subpoint_pix_d(ns, s, b[0], b[1], b[2], r, r, r, 1, 1, 1, ia, ib, ic);
                for (int c = 0; c < 9; ++c) {
                    u_rcp = c == 8 ? 0 : c & 1 ? 1 : -1;
                    u_rsq = c == 8 ? 0 : c & 2 ? 1 : -1;
                    u_sqrt = c == 8 ? 0 : c & 4 ? 1 : -1;
                    bool unsure = false;
                    const int pf = tr::ang2pix_f(ns, x, y, z, tol, unsure);
                    ++n;
                    doubt += unsure;
                    wrong += !unsure && pf != pd;
                }
            }
        }
    }
    printf("%ld %ld %ld\n", n, doubt, wrong);
}
"""


@pytest.fixture(scope="module")
def progs(tmp_path_factory):
    d = tmp_path_factory.mktemp("classifier")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "m.cpp").write_text(SRC)
    out = {}
    # the compiler may fuse multiply-adds of the FP32 form (here then of the FP64 form too, which the
    # kernels never fuse: far inside the guard band)
    for name, flags in (("separate", ["-ffp-contract=off"]), ("fused", ["-ffp-contract=fast", "-mfma"])):
        out[name] = str(d / name)
        subprocess.run(["g++", "-O2", "-std=c++17", "-w", *flags, "-I", str(d), "-I",
                        os.path.join(ROOT, "paper_2105_09644_amd", "csrc"), "-o", out[name], str(d / "m.cpp")], check=True)
    return out


@pytest.mark.parametrize("form", ["separate", "fused"])
@pytest.mark.parametrize("nside,s,reach", [(1, 2, 4), (2, 4, 4), (4, 4, 4), (8, 3, 8), (64, 4, 4)])
def test_fp32_pixels_are_the_fp64_ones(progs, form, nside, s, reach):
    n, doubt, wrong = map(int, subprocess.run([progs[form], str(nside), str(s), str(reach), "6000"], capture_output=True,
                                              text=True, check=True).stdout.split())
    print(f"{form} N_side {nside}: {n} classifications, {doubt / n:.2e} in the guard band")
    assert n > 10 ** 6 and wrong == 0
    assert doubt < 0.05 * n
