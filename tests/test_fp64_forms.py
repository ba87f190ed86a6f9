"""The shading's FP64 forms (FMAs, Newton steps from the hardware's reciprocal and root
estimates) are no further from the exact values than the plain sequence of correctly rounded
operations: the device code's own header compiled for the host, with estimates that are off by
up to 2^-23, against the same formulas in 128 bits (CPU only).

What is compared is the root mean square of the error over the inputs, relative to the value
(to the vector for the normal derivatives); 2 % is left for the finite sample."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"

HIP_RUNTIME = r'''
#pragma once
#include <stdint.h>
#include <math.h>
#include <string.h>
#include <stddef.h>
#define __device__
#define __host__
#define __forceinline__ inline
#define __global__
using std_size = size_t;
struct float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
struct double2 { double x, y; };
inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
inline float2 make_float2(float a, float b) { return {a, b}; }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
// uniform numbers, and the estimates of the hardware (relative error up to 2^-23)
inline double uni() {
    static uint64_t s = 0x9E3779B97F4A7C15ull;
    s ^= s << 13, s ^= s >> 7, s ^= s << 17;
    return (double)(s >> 11) * 0x1p-53;
}
inline double est(double e) { return e * (1.0 + (2.0 * uni() - 1.0) * 0x1p-23); }
inline double est_rcp(double x) { return est(1.0 / x); }
inline double est_rsq(double x) { return est(1.0 / sqrt(x)); }
#define __builtin_amdgcn_rcp est_rcp
#define __builtin_amdgcn_rsq est_rsq
'''

MAIN = r'''
#include "common.hpp"
#include <stdio.h>
#include <type_traits>
using namespace dpcs;
// 128-bit root: Newton steps from the FP64 one
static __float128 sq(__float128 x) {
    __float128 r = sqrt((double)x);
    r = (r + x / r) / 2;
    return (r + x / r) / 2;
}
static double sq(double x) { return sqrt(x); }
template <class T> struct V { T x, y, z; };
template <class T> T dt(V<T> a, V<T> b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
template <class T> V<T> cr(V<T> a, V<T> b) { return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x}; }
template <class T> V<T> ad(V<T> a, V<T> b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
template <class T> V<T> mu(V<T> a, T s) { return {a.x * s, a.y * s, a.z * s}; }
template <class T> V<T> to(D3 a) { return {(T)a.x, (T)a.y, (T)a.z}; }
constexpr int NV = 30;
static const char* NAME[NV] = {"f", "d_rough", "d_spec", "density", "pf", "pf_albedo", "pf_rough", "pf_spec", "pf_metal",
                               "dn0", "dn1", "dn2", "dn3", "dn4", "dn5", "dn6", "dn7", "dn8", "throughput", "lambert",
                               "distance", "direction", "falloff"};
constexpr int USED = 23;
// every value in plain operations of type T
template <class T>
void plain(D3 n_, D3 wo_, D3 wi_, D3 al_, double r_, double sp_, double mt_, D3 xp_, D3 tow_, T* o) {
    const V<T> n = to<T>(n_), wo = to<T>(wo_), wi = to<T>(wi_), al = to<T>(al_);
    const T r = r_, sp = sp_, mt = mt_, pi = PI, ipi = (T)(1.0 / PI), c08 = 0.08, one = 1, two = 2, half = 0.5;
    const T ci = dt(n, wi), co = dt(n, wo);
    const V<T> v = ad(wi, wo), nxv = cr(n, v);
    const T vv = dt(v, v), nv = dt(n, v), c2v = nv * nv, s2v = dt(nxv, nxv);
    const T a = r * r > (T)ALPHA_MIN ? r * r : (T)ALPHA_MIN, a2 = a * a, kv = a2 * c2v + s2v;
    const T qi = sq(a2 + (one - a2) * ci * ci), qo = sq(a2 + (one - a2) * co * co);
    const T m = one - half * sq(vv), m5 = m * m * m * m * m;
    const T F0 = c08 * sp, F = F0 + (one - F0) * m5;
    const T G = a2 * vv * vv / (pi * kv * kv * (ci + qi) * (co + qo));
    const T dD = two / a * (one - two * a2 * c2v / kv);
    const T dG = -a * ((one - ci * ci) / (qi * (ci + qi)) + (one - co * co) / (qo * (co + qo)));
    const T da = two * r;
    o[0] = al.x * ipi + F * G;
    o[1] = F * G * (dD + dG) * da;
    o[2] = c08 * (one - m5) * G;
    const T an = nv < 0 ? -nv : nv, ov = dt(wo, v);
    const T kp = a2 * an * an + s2v;
    o[3] = (T)(1.0 - P_SPEC) * (ci * ipi) + (T)P_SPEC * (a2 * vv * vv * an / (4 * pi * kp * kp * ov));
    const T kd = one - mt;
    const T f0 = kd * (c08 * sp) + mt * al.x, Fx = f0 + (one - f0) * m5;
    o[4] = al.x * (kd / pi) + Fx * G;
    o[5] = kd / pi + mt * (one - m5) * G;
    o[6] = Fx * (G * (dD + dG) * da);
    o[7] = kd * c08 * (one - m5) * G;
    o[8] = al.x * (T)(-1.0 / PI) + (al.x - c08 * sp) * ((one - m5) * G);
    const T iv = one / sq(vv), ch = nv * iv, k = kv / vv, D = a2 / (pi * k * k);
    const T Gi = two * ci / (ci + qi), Go = two * co / (co + qo);
    const T Dd = -4 * a2 * ch * (a2 - one) / (pi * k * k * k);
    const T gi = two * a2 / (qi * (ci + qi) * (ci + qi)), go = two * a2 / (qo * (co + qo) * (co + qo));
    const T S = G * ci, i4 = one / (4 * co);
    const V<T> dS = ad(ad(mu(v, Dd * Gi * Go * i4 * iv), mu(wi, D * gi * Go * i4)), mu(wo, D * Gi * go * i4 - S / co));
    const T ac[3] = {al.x, al.y, al.z};
    for (int c = 0; c < 3; ++c) {
        const T fc = kd * (c08 * sp) + mt * ac[c], Fc = fc + (one - fc) * m5;
        const V<T> q = ad(mu(wi, kd * ac[c] / pi), mu(dS, Fc));
        o[9 + 3 * c] = q.x, o[10 + 3 * c] = q.y, o[11 + 3 * c] = q.z;
    }
    o[18] = o[0] * (ci / o[3]);
    o[19] = al.x * ipi * (ci / (ci * ipi));
    const V<T> xp = to<T>(xp_), tow = to<T>(tow_);
    const T d = sq(dt(tow, tow)), ca = xp.z / sq(dt(xp, xp));
    o[20] = d;
    o[21] = tow.x * (one / d);
    o[22] = one / (ca * ca * ca * d * d);
}
static void ours(D3 n, D3 wo, D3 wi, D3 al, double r, double sp, double mt, D3 xp, D3 tow, double* o) {
    const Brdf b = brdf_eval<true>(1, n, wo, wi, al, r, sp);
    o[0] = b.f.x, o[1] = b.ds_dr, o[2] = b.ds_dsp, o[3] = bounce_pdf(1, n, wo, wi, r);
    const BrdfX x = brdf_x<true>(1, n, n, wo, wi, al, r, sp, mt);
    o[4] = x.f.x, o[5] = x.dfa, o[6] = x.dfr.x, o[7] = x.dfs, o[8] = x.dfm.x;
    for (int c = 0; c < 3; ++c) o[9 + 3 * c] = x.dn[c].x, o[10 + 3 * c] = x.dn[c].y, o[11 + 3 * c] = x.dn[c].z;
    o[18] = bounce_weight(b.f, dot(n, wi), o[3]).x;
    o[19] = bounce_weight(brdf_eval<false>(0, n, wo, wi, al, r, sp).f, dot(n, wi), bounce_pdf(0, n, wo, wi, r)).x;
    D3 wp;
    double dist;
    o[22] = projector_falloff(xp, tow, wp, dist);
    o[20] = dist, o[21] = wp.x;
}
static D3 unit(double x, double y, double z) {
    const double l = 1.0 / sqrt(x * x + y * y + z * z);
    return d3(x * l, y * l, z * l);
}
static D3 any() {
    for (;;) {
        const double x = 2 * uni() - 1, y = 2 * uni() - 1, z = 2 * uni() - 1, l = x * x + y * y + z * z;
        if (l < 1 && l > 0.01) return unit(x, y, z);
    }
}
int main() {
    double s[2][USED] = {}, d[2][3] = {};
    int cnt = 0;
    for (int it = 0; cnt < 400000; ++it) {
        const D3 n = any(), wo = any(), al = d3(0.05 + 0.9 * uni(), 0.05 + 0.9 * uni(), 0.05 + 0.9 * uni());
        const double r = 0.1 + 0.85 * uni(), sp = uni(), mt = uni(), co = dot(n, wo);
        D3 wi = any();
        if (it & 1) {   // about the mirror direction
            const D3 e = any();
            const double w = 0.1 * r;
            wi = unit(2 * co * n.x - wo.x + w * e.x, 2 * co * n.y - wo.y + w * e.y, 2 * co * n.z - wo.z + w * e.z);
        }
        if (co < 0.02 || dot(n, wi) < 0.02) continue;
        // a point 0.3 to 1.5 in front of the projector, and the same vector as the world has it
        const double z = 0.3 + 1.2 * uni(), dd = sqrt(1.0 + 0.16 * uni());
        const D3 xp = d3(0.8 * (uni() - 0.5) * z, 0.8 * (uni() - 0.5) * z, z);
        const D3 tow = any() * (z * dd);
        __float128 e[NV];
        double p[NV], q[NV];
        plain<__float128>(n, wo, wi, al, r, sp, mt, xp, tow, e);
        plain<double>(n, wo, wi, al, r, sp, mt, xp, tow, p);
        ours(n, wo, wi, al, r, sp, mt, xp, tow, q);
        for (int j = 0; j < USED; ++j) {
            double scale = fabs((double)e[j]);
            if (j >= 9 && j < 18) {   // a vector's component: against its length
                const int b = 9 + (j - 9) / 3 * 3;
                scale = sqrt((double)(e[b] * e[b] + e[b + 1] * e[b + 1] + e[b + 2] * e[b + 2]));
            }
            if (j == 21) scale = 1.0;
            // derivatives of either sign cancel: beyond 2^-45 one sample would decide the mean
            auto err = [&](double v) { return fmin(fabs((double)((__float128)v - e[j])) / scale, 0x1p-45); };
            s[0][j] += err(p[j]) * err(p[j]);
            s[1][j] += err(q[j]) * err(q[j]);
        }
        {   // the camera-pose gradient's differences: of the falloff over a step of the point, of
            // the reflectances over a turn of the outgoing direction
            const double h = 1e-8 * z, w = 1e-7;
            const D3 e1 = any(), e2 = any();
            const D3 X[2] = {xp, d3(xp.x + e1.x * h, xp.y + e1.y * h, xp.z + e1.z * h)};
            const D3 Y[2] = {tow, d3(tow.x + e2.x * h, tow.y + e2.y * h, tow.z + e2.z * h)};
            const D3 O[2] = {wo, unit(wo.x + e1.x * w, wo.y + e1.y * w, wo.z + e1.z * w)};
            __float128 E[2][NV];
            double P[2][NV], R[2][NV];
            for (int k = 0; k < 2; ++k) {
                plain<__float128>(n, O[k], wi, al, r, sp, mt, X[k], Y[k], E[k]);
                plain<double>(n, O[k], wi, al, r, sp, mt, X[k], Y[k], P[k]);
                ours(n, O[k], wi, al, r, sp, mt, X[k], Y[k], R[k]);
            }
            const int id[3] = {22, 0, 4};
            for (int v = 0; v < 3; ++v) {
                const int j = id[v];
                const double st = v == 0 ? h : w, scale = fabs((double)E[0][j]) / (v == 0 ? z : 1.0);
                const __float128 x = (E[1][j] - E[0][j]) / (__float128)st;
                auto err = [&](double f0, double f1) { return fmin(fabs((double)((f1 - f0) / st - x)) / scale, 1e-6); };
                const double a = err(P[0][j], P[1][j]), b = err(R[0][j], R[1][j]);
                d[0][v] += a * a, d[1][v] += b * b;
            }
        }
        ++cnt;
    }
    for (int j = 0; j < USED; ++j)
        printf("%s %.4f %.4f\n", NAME[j], sqrt(s[0][j] / cnt) * 0x1p53, sqrt(s[1][j] / cnt) * 0x1p53);
    const char* nd[3] = {"slope_falloff", "slope_f", "slope_pf"};
    for (int v = 0; v < 3; ++v) printf("%s %.4f %.4f\n", nd[v], sqrt(d[0][v] / cnt) * 1e8, sqrt(d[1][v] / cnt) * 1e8);
    return 0;
}
'''


@pytest.fixture(scope="module")
def errors(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(HIP_RUNTIME)
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "forms")
    subprocess.check_call([CLANG, "-std=c++17", "-O2", "-mfma", "-ffp-contract=off", "-Wno-unknown-pragmas", "-w", "-I", str(d),
                           "-I", os.path.join(ROOT, "paper_2503_12174_amd", "csrc"), str(d / "main.cpp"), "-o", exe])
    lines = subprocess.check_output([exe], text=True).split("\n")
    return {k: (float(a), float(b)) for k, a, b in (ln.split() for ln in lines if ln)}


@pytest.mark.parametrize("value", ["f", "d_rough", "d_spec", "density", "pf", "pf_albedo", "pf_rough", "pf_spec", "pf_metal",
                                   "dn0", "dn1", "dn2", "dn3", "dn4", "dn5", "dn6", "dn7", "dn8", "throughput", "lambert",
                                   "distance", "direction", "falloff", "slope_falloff", "slope_f", "slope_pf"])
def test_error_is_no_larger_than_the_plain_sequences(errors, value):
    plain, ours = errors[value]
    assert ours <= 1.02 * plain
