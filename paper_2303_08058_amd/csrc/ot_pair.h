// ot_pair.h -- the arithmetic of one (target cell, source cell) pair: what is
// staged of a source and how it adds into a target's accumulators. Device
// code only; included by ot_interact.h.
//
// The contraction is arranged around the separation vector r = X_i - X_j
// instead of around the derivatives of G = -1/r. With the radial factors D_p
// (D_0 = G, D_{p+1} = -(2p+1) D_p / r^2, so grad D_p = r D_{p+1}) and a source
// whose second and third moments are made trace-free (which changes no
// result: derivatives of 1/r are trace-free),
//   phi(r) = q D_0 + e D_1 + s D_2 + u D_3,
//   e = d.r,  s = r.Q.r,  u = O:rrr,
// and every output is a derivative of phi by the product rule: with
// v = Q r, w = O:rr, M = O r
//   c_p = q D_p + e D_{p+1} + s D_{p+2} + u D_{p+3},
//   y_p = d D_p + 2 v D_{p+1} + 3 w D_{p+2},   Z_p = 2 Q D_p + 6 M D_{p+1}:
//   L_0 = c_0,  L_i = r_i c_1 + y_1,  L_ij = delta c_1 + c_2 r r + sym(r y_2) + Z_2, ...
// A total-order truncation leaves out the terms of too high an order. The
// vectors and small tensors are shared by all outputs. FP64 instructions a
// pair (pair loop of the compiled kernels, contraction with the derivatives
// of G before): forward 95 (113 before), orders 0..3 and exact order 4 202
// (226), target role 171 (210), full truncation's forward 197 (438), its
// orders 0..4 302 (about 760). The kernels are bound by the FP64 issue rate:
// with nothing else changed the forward of 4096 sub-grids fell from 15.7 to
// 13.5 ms, the two-launch step of 32768 from 474 to 436 ms and the full
// truncation's two-launch step of 720 from 30.8 to 15.0 ms (same box); the
// error against a 64-bit reference halved (fewer roundings).
//
// Outputs whose z exponent is 2 or more are not accumulated: they follow from
// two others (Laplace's equation). Symmetric tensors are kept as the
// coefficients of homogeneous polynomials in a formal vector t, modulo t_z^2:
// multiplying by (r.t) or (t.t) never lowers a z exponent, so the kept
// coefficients of each step need only kept ones of the step before.
#pragma once

#include <hip/hip_runtime.h>

#include "ot_common.h"

using namespace otfmm;

namespace {

// The output sums a pair adds into, in kept graded-lex order (acc index):
enum Sums : int {
    SUMS_MONO = 0,  // orders 0..3 of a mass                                    (16)
    SUMS_F3 = 1,    // orders 0..3, total order |a| + |b| <= 3                   (16)
    SUMS_FE = 2,    // the same, then orders 1..4 with |a| + |b| = 4 exactly     (16 + 24)
    SUMS_T4 = 3,    // orders 1..4, |a| + |b| <= 4                               (24)
    SUMS_X3 = 4,    // orders 0..3, every |b| <= 3                               (16)
    SUMS_X4 = 5,    // orders 0..4, every |b| <= 3                               (25)
    SUMS_X4T = 6    // orders 1..4, every |b| <= 3                               (24)
};

__host__ __device__ constexpr int sums_count(int s)
{
    return s == SUMS_FE ? 40 : (s == SUMS_T4 || s == SUMS_X4T) ? 24 : s == SUMS_X4 ? 25 : 16;
}

// ---------------------------------------------------------------------------
// Staged source record: centre, q, then (not for a mass) d, Q and O -- a
// multiple of 16 bytes, read with 16-byte LDS loads.
//   rec[0..2] centre, [3] q, [4..6] d,
//   [7..12]  Q xx, xy, xz, yy, yz, zz (trace-free; doubled for the X sums),
//   [13..19] O xxx, xxy, xxz, xyy, xyz, yyy, yyz (trace-free; tripled for the
//            X sums). F3 needs only u and takes O reduced by its trace
//            partners instead (xxx - xzz, xxy - yzz, xxz - zzz, xyy - xzz,
//            xyz, yyy - yzz, yyz - zzz), contracted with the trace-free
//            polynomials of r.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int record_size(int sums) { return sums == SUMS_MONO ? 4 : 20; }

// factor of raw component b: the forward's sources carry (-1)^{|b|}/b!, the
// adjoint's (-1)^{|b|}
template <bool REV>
__host__ __device__ constexpr double source_factor(int b)
{
    return REV ? parity_sign(b) : parity_sign(b) * inv_multi_factorial(b);
}

// k1 raw[b1] + k2 raw[b2] + k3 raw[b3], each with its source factor
template <bool REV, int B1, int B2, int B3>
__device__ __forceinline__ double mix3(const double* raw, double k1, double k2, double k3)
{
    constexpr double f1 = source_factor<REV>(B1), f2 = source_factor<REV>(B2), f3 = source_factor<REV>(B3);
    return __builtin_fma(k3 * f3, raw[B3], __builtin_fma(k2 * f2, raw[B2], k1 * f1 * raw[B1]));
}

// The record's entries 3.. of a source with raw components raw[20] (raw[1]
// for a mass). Second moments: with T_xx = c_xx, T_xy = c_xy / 2 (c: raw
// times its factor) the contraction with G_ij is sum_ij T_ij G_ij, and Q is T
// less a third of its trace, formed from the differences of the diagonal.
// Third moments: T_xxx = c_xxx, T_xxy = c_xxy / 3, T_xyz = c_xyz / 6, and
// O_ijk = T_ijk - (delta_ij t_k + delta_ik t_j + delta_jk t_i) / 5, t_k = T_iik.
template <int SUMS, bool REV>
__device__ __forceinline__ void stage_record(const double* raw, double* rec)
{
    constexpr double fq = (SUMS == SUMS_X3 || SUMS == SUMS_X4 || SUMS == SUMS_X4T) ? 2.0 : 1.0;
    constexpr double fo = (SUMS == SUMS_X3 || SUMS == SUMS_X4 || SUMS == SUMS_X4T) ? 3.0 : 1.0;
    rec[3] = raw[0] * source_factor<REV>(0);
    if constexpr (SUMS != SUMS_MONO) {
#pragma unroll
        for (int k = 1; k < 4; ++k) rec[3 + k] = raw[k] * source_factor<REV>(1);
        constexpr double f2 = source_factor<REV>(4), f11 = 0.5 * source_factor<REV>(5);
        const double xx_yy = raw[4] - raw[7], xx_zz = raw[4] - raw[9], yy_zz = raw[7] - raw[9];
        rec[7] = (fq * f2 / 3.0) * (xx_yy + xx_zz);
        rec[8] = (fq * f11) * raw[5];
        rec[9] = (fq * f11) * raw[6];
        rec[10] = (fq * f2 / 3.0) * (yy_zz - xx_yy);
        rec[11] = (fq * f11) * raw[8];
        rec[12] = (-fq * f2 / 3.0) * (xx_zz + yy_zz);
        if constexpr (SUMS == SUMS_F3) {
            rec[13] = mix3<REV, 10, 15, 15>(raw, 1.0, -1.0, 0.0);
            rec[14] = mix3<REV, 11, 18, 18>(raw, 1.0, -1.0, 0.0);
            rec[15] = mix3<REV, 12, 19, 19>(raw, 1.0, -1.0, 0.0);
            rec[16] = mix3<REV, 13, 15, 15>(raw, 1.0, -1.0, 0.0);
            rec[17] = source_factor<REV>(14) * raw[14];
            rec[18] = mix3<REV, 16, 18, 18>(raw, 1.0, -1.0, 0.0);
            rec[19] = mix3<REV, 17, 19, 19>(raw, 1.0, -1.0, 0.0);
        } else {
            // 10 xxx, 11 xxy, 12 xxz, 13 xyy, 14 xyz, 15 xzz, 16 yyy, 17 yyz, 18 yzz, 19 zzz
            rec[13] = mix3<REV, 10, 13, 15>(raw, fo * 0.4, fo * -0.2, fo * -0.2);
            rec[14] = mix3<REV, 11, 16, 18>(raw, fo * 4.0 / 15.0, fo * -0.2, fo / -15.0);
            rec[15] = mix3<REV, 12, 17, 19>(raw, fo * 4.0 / 15.0, fo / -15.0, fo * -0.2);
            rec[16] = mix3<REV, 13, 10, 15>(raw, fo * 4.0 / 15.0, fo * -0.2, fo / -15.0);
            rec[17] = (fo * source_factor<REV>(14) / 6.0) * raw[14];
            rec[18] = mix3<REV, 16, 11, 18>(raw, fo * 0.4, fo * -0.2, fo * -0.2);
            rec[19] = mix3<REV, 17, 12, 19>(raw, fo * 4.0 / 15.0, fo / -15.0, fo * -0.2);
        }
    }
}

// ---------------------------------------------------------------------------
// Pair step
// ---------------------------------------------------------------------------
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

__device__ __forceinline__ double rsqrt_fp64(double a)
{
    // hardware estimate, then y (1 + e/2 + 3e^2/8) with e = 1 - a y^2
    double y = __builtin_amdgcn_rsq(a);
    const double e = __builtin_fma(-a * y, y, 1.0);
    y = __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
    return y;
}

// Sum of the order-3 outputs c H_ijk(r), H the trace-free part of r r r
// (kept: xxx, xxy, xxz, xyy, xyz, yyy, yyz), from cr = c r.
struct Cubic {
    double a1, b1, a3, b3, yz;  // xx - r2/5, yy - r2/5, xx - 3 r2/5, yy - 3 r2/5, yz
};
__device__ __forceinline__ Cubic cubic(double xx, double yy, double yz, double r2)
{
    return {fma_(-0.2, r2, xx), fma_(-0.2, r2, yy), fma_(-0.6, r2, xx), fma_(-0.6, r2, yy), yz};
}
__device__ __forceinline__ void add_cubic(double* a, const Cubic& h, double cx, double cy, double cz)
{
    a[0] = fma_(cx, h.a3, a[0]);
    a[1] = fma_(cy, h.a1, a[1]);
    a[2] = fma_(cz, h.a1, a[2]);
    a[3] = fma_(cx, h.b1, a[3]);
    a[4] = fma_(cx, h.yz, a[4]);
    a[5] = fma_(cy, h.b3, a[5]);
    a[6] = fma_(cz, h.b1, a[6]);
}

// Sum of the order-4 outputs c H_ijkl(r), H the trace-free part of r r r r
// (kept: xxxx, xxxy, xxxz, xxyy, xxyz, xyyy, xyyz, yyyy, yyyz).
__device__ __forceinline__ void add_quartic(double* a, double c, double xx, double yy, double xy, double xz,
                                            double yz, double r2)
{
    constexpr double k7 = 1.0 / 7.0;
    const double a1 = fma_(-k7, r2, xx), b1 = fma_(-k7, r2, yy);
    const double a3 = fma_(-3.0 * k7, r2, xx), b3 = fma_(-3.0 * k7, r2, yy);
    const double a6 = fma_(-6.0 * k7, r2, xx), b6 = fma_(-6.0 * k7, r2, yy);
    const double r4 = r2 * r2;
    const double t4 = (3.0 / 35.0) * r4;
    const double cxy = c * xy, cxz = c * xz, cyz = c * yz;
    a[0] = fma_(c, fma_(xx, a6, t4), a[0]);
    a[1] = fma_(cxy, a3, a[1]);
    a[2] = fma_(cxz, a3, a[2]);
    a[3] = fma_(c, fma_(a1, b1, (2.0 / 245.0) * r4), a[3]);
    a[4] = fma_(cyz, a1, a[4]);
    a[5] = fma_(cxy, b3, a[5]);
    a[6] = fma_(cxz, b1, a[6]);
    a[7] = fma_(c, fma_(yy, b6, t4), a[7]);
    a[8] = fma_(cyz, b3, a[8]);
}

// Products of kept polynomials with the linear form p = (px, py, pz).t, added
// to `a`: order 1 x 1 -> 2 (xx, xy, xz, yy, yz), 1 x 2 -> 3, 1 x 3 -> 4.
__device__ __forceinline__ void mul11(double* a, double px, double py, double pz, const double* l)
{
    a[0] = fma_(px, l[0], a[0]);
    a[1] = fma_(px, l[1], fma_(py, l[0], a[1]));
    a[2] = fma_(px, l[2], fma_(pz, l[0], a[2]));
    a[3] = fma_(py, l[1], a[3]);
    a[4] = fma_(py, l[2], fma_(pz, l[1], a[4]));
}
__device__ __forceinline__ void mul12(double* a, double px, double py, double pz, const double* q)
{
    a[0] = fma_(px, q[0], a[0]);
    a[1] = fma_(px, q[1], fma_(py, q[0], a[1]));
    a[2] = fma_(px, q[2], fma_(pz, q[0], a[2]));
    a[3] = fma_(px, q[3], fma_(py, q[1], a[3]));
    a[4] = fma_(px, q[4], fma_(py, q[2], fma_(pz, q[1], a[4])));
    a[5] = fma_(py, q[3], a[5]);
    a[6] = fma_(py, q[4], fma_(pz, q[3], a[6]));
}
__device__ __forceinline__ void mul13(double* a, double px, double py, double pz, const double* c)
{
    a[0] = fma_(px, c[0], a[0]);
    a[1] = fma_(px, c[1], fma_(py, c[0], a[1]));
    a[2] = fma_(px, c[2], fma_(pz, c[0], a[2]));
    a[3] = fma_(px, c[3], fma_(py, c[1], a[3]));
    a[4] = fma_(px, c[4], fma_(py, c[2], fma_(pz, c[1], a[4])));
    a[5] = fma_(px, c[5], fma_(py, c[3], a[5]));
    a[6] = fma_(px, c[6], fma_(py, c[4], fma_(pz, c[3], a[6])));
    a[7] = fma_(py, c[5], a[7]);
    a[8] = fma_(py, c[6], fma_(pz, c[5], a[8]));
}

// Adds the source in `rec` at separation (x, y, z) from the target into acc.
// Some entries of acc are kept scaled (sums_scale gives the factors).
template <int SUMS>
__device__ __forceinline__ void pair_sums(double* acc, const double* rec, double x, double y, double z)
{
    constexpr bool kX = SUMS == SUMS_X3 || SUMS == SUMS_X4 || SUMS == SUMS_X4T;
    constexpr int kTop = SUMS == SUMS_X3 ? 6 : (SUMS == SUMS_X4 || SUMS == SUMS_X4T) ? 7
                       : (SUMS == SUMS_FE || SUMS == SUMS_T4) ? 4 : 3;
    const double xx = x * x, yy = y * y;
    const double r2 = fma_(z, z, xx + yy);
    const double ri = rsqrt_fp64(r2);
    const double ri2 = ri * ri;
    double D[kTop + 1];
    D[0] = -ri;
    D[1] = ri * ri2;
#pragma unroll
    for (int p = 1; p < kTop; ++p) D[p + 1] = ((-(2.0 * p + 1.0)) * ri2) * D[p];
    const double q0 = rec[3];

    if constexpr (SUMS == SUMS_MONO) {
        const double c1 = q0 * D[1], c2 = q0 * D[2], c3 = q0 * D[3];
        const double px = c2 * x, py = c2 * y;
        acc[0] = fma_(q0, D[0], acc[0]);
        acc[1] = fma_(c1, x, acc[1]);
        acc[2] = fma_(c1, y, acc[2]);
        acc[3] = fma_(c1, z, acc[3]);
        acc[4] = fma_(x, px, acc[4]) + c1;
        acc[5] = fma_(x, py, acc[5]);
        acc[6] = fma_(z, px, acc[6]);
        acc[7] = fma_(y, py, acc[7]) + c1;
        acc[8] = fma_(z, py, acc[8]);
        add_cubic(acc + 9, cubic(xx, yy, y * z, r2), c3 * x, c3 * y, c3 * z);
        return;
    } else {
        const double* d = rec + 4;
        const double* Q = rec + 7;
        const double* O = rec + 13;
        const double e = fma_(d[0], x, fma_(d[1], y, d[2] * z));
        const double v[3] = {fma_(Q[0], x, fma_(Q[1], y, Q[2] * z)), fma_(Q[1], x, fma_(Q[3], y, Q[4] * z)),
                             fma_(Q[2], x, fma_(Q[4], y, Q[5] * z))};
        const double vr = fma_(v[0], x, fma_(v[1], y, v[2] * z));

        if constexpr (!kX) {
            const double s = vr;
            const double yz = y * z;
            const Cubic h = cubic(xx, yy, yz, r2);
            const double D2x2 = 2.0 * D[2];
            double u = 0.0, w[3] = {0.0, 0.0, 0.0}, xy = 0.0, xz = 0.0, x2 = 0.0, y2 = 0.0;
            if constexpr (SUMS == SUMS_F3) {
                u = fma_(x, fma_(O[0], h.a3, fma_(O[3], h.b1, O[4] * yz)),
                         fma_(y, fma_(O[1], h.a1, O[5] * h.b3), z * fma_(O[2], h.a1, O[6] * h.b1)));
            } else {
                // w = O:rr in the trace-free basis xx - zz, yy - zz, 2xy, 2xz, 2yz
                x2 = x + x;
                y2 = y + y;
                xy = x * y;
                xz = x * z;
                const double zz = z * z, m1 = xx - zz, m2 = yy - zz;
                const double xy2 = x2 * y, xz2 = x2 * z, yz2 = y2 * z;
                const double Oxzz = -(O[0] + O[3]), Oyzz = -(O[1] + O[5]);
                w[0] = fma_(O[0], m1, fma_(O[3], m2, fma_(O[1], xy2, fma_(O[2], xz2, O[4] * yz2))));
                w[1] = fma_(O[1], m1, fma_(O[5], m2, fma_(O[3], xy2, fma_(O[4], xz2, O[6] * yz2))));
                w[2] = fma_(O[2], m1, fma_(O[6], m2, fma_(O[4], xy2, fma_(Oxzz, xz2, Oyzz * yz2))));
                u = fma_(w[0], x, fma_(w[1], y, w[2] * z));
            }
            const double r[3] = {x, y, z};
            if constexpr (SUMS == SUMS_F3 || SUMS == SUMS_FE) {
                acc[0] = fma_(q0, D[0], fma_(e, D[1], fma_(s, D[2], fma_(u, D[3], acc[0]))));
                const double t1 = fma_(e, D[2], q0 * D[1]);  // also the delta_ij term of order 2
                const double c1 = fma_(s, D[3], t1);
                const double c2 = fma_(e, D[3], q0 * D[2]);
                const double c3 = q0 * D[3];
                double p[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    acc[1 + k] = fma_(r[k], c1, fma_(d[k], D[1], fma_(v[k], D2x2, acc[1 + k])));
                    p[k] = fma_(c2, r[k], D2x2 * d[k]);
                }
                mul11(acc + 4, x, y, z, p);  // off-diagonal coefficients doubled
                acc[4] += t1;
                acc[7] += t1;
                add_cubic(acc + 9, h, c3 * x, c3 * y, c3 * z);
            }
            if constexpr (SUMS == SUMS_FE || SUMS == SUMS_T4) {
                constexpr bool kE = SUMS == SUMS_FE;  // exact order 4: only the terms with |b| = 4 - |a|
                double* a = acc + (kE ? 16 : 0);
                const double D3x3 = 3.0 * D[3], D3x4 = 4.0 * D[3], D2x4 = 4.0 * D[2];
                const double eD3 = e * D[3];
                double c1, c2, c3, t1;
                double p[3], g[3];
                if constexpr (kE) {
                    c1 = u * D[4];
                    t1 = s * D[3];
                    c2 = s * D[4];
                    c3 = e * D[4];
                } else {
                    t1 = fma_(s, D[3], fma_(e, D[2], q0 * D[1]));
                    c1 = fma_(u, D[4], t1);
                    c2 = fma_(s, D[4], fma_(q0, D[2], eD3));
                    c3 = fma_(e, D[4], q0 * D[3]);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    a[k] = fma_(r[k], c1, fma_(w[k], D3x3, a[k]));
                    p[k] = fma_(c2, r[k], D3x4 * v[k]);
                    if constexpr (!kE) {
                        a[k] = fma_(d[k], D[1], fma_(v[k], D2x2, a[k]));
                        p[k] = fma_(d[k], D2x2, p[k]);
                    }
                    g[k] = D[3] * d[k];
                }
                a[3] = fma_(Q[0], D2x2, a[3]);  // + 2 Q D_2
                a[4] = fma_(Q[1], D2x4, a[4]);
                a[5] = fma_(Q[2], D2x4, a[5]);
                a[6] = fma_(Q[3], D2x2, a[6]);
                a[7] = fma_(Q[4], D2x4, a[7]);
                mul11(a + 3, x, y, z, p);  // off-diagonal coefficients doubled
                a[3] += t1;
                a[6] += t1;
                // c_3 H_ijk + D_3 (d.grad) H_ijk; xxx and yyy kept as thirds
                const double f = 0.4 * eD3;
                const double P = fma_(c3, h.a1, fma_(x2, g[0], -f)), R = fma_(c3, h.b1, fma_(y2, g[1], -f));
                const double c3t = c3 * (1.0 / 3.0);
                const double P3 = fma_(c3t, h.a3, -f), R3 = fma_(c3t, h.b3, -f);
                a[8] = fma_(g[0], h.a1, fma_(x, P3, a[8]));
                a[9] = fma_(g[1], h.a1, fma_(y, P, a[9]));
                a[10] = fma_(g[2], h.a1, fma_(z, P, a[10]));
                a[11] = fma_(g[0], h.b1, fma_(x, R, a[11]));
                a[12] = fma_(fma_(c3, x, g[0]), yz, fma_(g[1], xz, fma_(g[2], xy, a[12])));
                a[13] = fma_(g[1], h.b1, fma_(y, R3, a[13]));
                a[14] = fma_(g[2], h.b1, fma_(z, R, a[14]));
                add_quartic(a + 15, q0 * D[4], xx, yy, xy, xz, yz, r2);
            }
        } else {
            // Q holds 2Q, O holds 3 O
            const double s = 0.5 * vr;
            const double Oxzz = -(O[0] + O[3]), Oyzz = -(O[1] + O[5]);
            const double M[5] = {fma_(O[0], x, fma_(O[1], y, O[2] * z)), fma_(O[1], x, fma_(O[3], y, O[4] * z)),
                                 fma_(O[2], x, fma_(O[4], y, Oxzz * z)), fma_(O[3], x, fma_(O[5], y, O[6] * z)),
                                 fma_(O[4], x, fma_(O[6], y, Oyzz * z))};  // 3 M
            const double Mzz = -(M[0] + M[3]);
            const double w[3] = {fma_(M[0], x, fma_(M[1], y, M[2] * z)), fma_(M[1], x, fma_(M[3], y, M[4] * z)),
                                 fma_(M[2], x, fma_(M[4], y, Mzz * z))};  // 3 w
            const double u = (1.0 / 3.0) * fma_(w[0], x, fma_(w[1], y, w[2] * z));
            const double r[3] = {x, y, z};
            double* a = acc + (SUMS == SUMS_X4T ? 0 : 1);
            if constexpr (SUMS != SUMS_X4T)
                acc[0] = fma_(q0, D[0], fma_(e, D[1], fma_(s, D[2], fma_(u, D[3], acc[0]))));
            const double c1 = fma_(q0, D[1], fma_(e, D[2], fma_(s, D[3], u * D[4])));
            const double c2 = fma_(q0, D[2], fma_(e, D[3], fma_(s, D[4], u * D[5])));
            const double c3 = fma_(q0, D[3], fma_(e, D[4], fma_(s, D[5], u * D[6])));
            const double D2x2 = 2.0 * D[2], D3x2 = 2.0 * D[3], D3x4 = 4.0 * D[3], D4x2 = 2.0 * D[4],
                         D4x4 = 4.0 * D[4];
            const double c3t = c3 * (1.0 / 3.0);
            double g[3], p[3], n[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                a[k] = fma_(r[k], c1, fma_(d[k], D[1], fma_(v[k], D[2], fma_(w[k], D[3], a[k]))));
                const double y2 = fma_(d[k], D[2], fma_(v[k], D[3], w[k] * D[4]));
                g[k] = fma_(c2, r[k], y2);
                p[k] = g[k] + y2;
                n[k] = fma_(c3t, r[k], fma_(d[k], D[3], fma_(v[k], D[4], w[k] * D[5])));
            }
            // order 2: c_1 (t.t) + (r.t)(p.t) + t Z_2 t, off-diagonal coefficients doubled
            a[3] = fma_(Q[0], D[2], fma_(M[0], D3x2, a[3]));
            a[4] = fma_(Q[1], D2x2, fma_(M[1], D3x4, a[4]));
            a[5] = fma_(Q[2], D2x2, fma_(M[2], D3x4, a[5]));
            a[6] = fma_(Q[3], D[2], fma_(M[3], D3x2, a[6]));
            a[7] = fma_(Q[4], D2x2, fma_(M[4], D3x4, a[7]));
            mul11(a + 3, x, y, z, p);
            a[3] += c1;
            a[6] += c1;
            // order 3, a third of it: (t.t)(g.t) + (r.t) N(t) + 2 O ttt D_3,
            // N = t Z_3 t + (r.t)(n.t)
            double N[5] = {fma_(Q[0], D[3], M[0] * D4x2), fma_(Q[1], D3x2, M[1] * D4x4),
                           fma_(Q[2], D3x2, M[2] * D4x4), fma_(Q[3], D[3], M[3] * D4x2),
                           fma_(Q[4], D3x2, M[4] * D4x4)};
            mul11(N, x, y, z, n);
            const double o3 = (2.0 / 3.0) * D[3];
            a[8] = fma_(O[0], o3, a[8]) + g[0];
            a[9] = fma_(O[1], D3x2, a[9]) + g[1];
            a[10] = fma_(O[2], D3x2, a[10]) + g[2];
            a[11] = fma_(O[3], D3x2, a[11]) + g[0];
            a[12] = fma_(O[4], D3x4, a[12]);
            a[13] = fma_(O[5], o3, a[13]) + g[1];
            a[14] = fma_(O[6], D3x2, a[14]) + g[2];
            mul12(a + 8, x, y, z, N);
            if constexpr (SUMS == SUMS_X4 || SUMS == SUMS_X4T) {
                // order 4, a sixth of it: (t.t)(c_2/2 (t.t) + B(t)) + (r.t) J(t),
                // B = N + (r.t)((c_3/3 r + n).t),
                // J = (r.t) K(t) + 4 O ttt D_4, K = t Z_4 t + (r.t)(m.t), m = c_4/6 r + 2/3 y_4
                const double c4 = fma_(q0, D[4], fma_(e, D[5], fma_(s, D[6], u * D[7])));
                const double c4s = c4 * (1.0 / 6.0);
                const double E4 = (2.0 / 3.0) * D[4], E5 = (2.0 / 3.0) * D[5], E6 = (2.0 / 3.0) * D[6];
                const double D5x2 = 2.0 * D[5], D5x4 = 4.0 * D[5];
                double l[3], m[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    l[k] = fma_(c3t, r[k], n[k]);
                    m[k] = fma_(c4s, r[k], fma_(d[k], E4, fma_(v[k], E5, w[k] * E6)));
                }
                mul11(N, x, y, z, l);
                N[0] = fma_(0.5, c2, N[0]);
                N[3] = fma_(0.5, c2, N[3]);
                double K[5] = {fma_(Q[0], D[4], M[0] * D5x2), fma_(Q[1], D4x2, M[1] * D5x4),
                               fma_(Q[2], D4x2, M[2] * D5x4), fma_(Q[3], D[4], M[3] * D5x2),
                               fma_(Q[4], D4x2, M[4] * D5x4)};
                mul11(K, x, y, z, m);
                const double o4 = (4.0 / 3.0) * D[4], D4x8 = 8.0 * D[4];
                double J[7] = {O[0] * o4, O[1] * D4x4, O[2] * D4x4, O[3] * D4x4, O[4] * D4x8, O[5] * o4, O[6] * D4x4};
                mul12(J, x, y, z, K);
                double* b = a + 15;
                b[0] += N[0];
                b[1] += N[1];
                b[2] += N[2];
                b[3] += N[0] + N[3];
                b[4] += N[4];
                b[5] += N[1];
                b[6] += N[2];
                b[7] += N[3];
                b[8] += N[4];
                mul13(b, x, y, z, J);
            }
        }
    }
}

// Factor of each accumulator at the end (polynomial coefficients to
// derivatives, and the thirds and sixths above).
__host__ __device__ constexpr double sums_scale(int sums, int k)
{
    constexpr double two[5] = {1.0, 0.5, 0.5, 1.0, 0.5};
    constexpr double thirds[7] = {3.0, 1.0, 1.0, 1.0, 1.0, 3.0, 1.0};
    constexpr double cubes[7] = {3.0, 1.0, 1.0, 1.0, 0.5, 3.0, 1.0};
    constexpr double sixths[9] = {6.0, 1.5, 1.5, 1.0, 0.5, 1.5, 0.5, 6.0, 1.5};
    if (sums == SUMS_MONO) return 1.0;
    if (sums == SUMS_F3) return k >= 4 && k < 9 ? two[k - 4] : 1.0;
    if (sums == SUMS_FE) {
        if (k < 16) return k >= 4 && k < 9 ? two[k - 4] : 1.0;
        k -= 16;
    }
    if (sums == SUMS_FE || sums == SUMS_T4)
        return k < 3 ? 1.0 : k < 8 ? two[k - 3] : k < 15 ? thirds[k - 8] : 1.0;
    if (sums != SUMS_X4T) --k;
    return k < 3 ? 1.0 : k < 8 ? two[k - 3] : k < 15 ? cubes[k - 8] : sixths[k - 15];
}
template <int SUMS, int... K>
__device__ __forceinline__ void scale_sums(double* acc, std::integer_sequence<int, K...>)
{
    ((acc[K] *= sums_scale(SUMS, K)), ...);
}
template <int SUMS>
__device__ __forceinline__ void finish_sums(double* acc)
{
    scale_sums<SUMS>(acc, std::make_integer_sequence<int, sums_count(SUMS)>{});
}

}  // namespace
