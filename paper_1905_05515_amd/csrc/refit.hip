// Calibrated Kalman refit of found tracks and its adjoint.
//
// Forward (one thread per track): calibrate every raw cluster with the 16
// parameters theta, start from the first and third hits, filter outwards and
// sum the chi2 of the updates; the state after every update but the last (in
// large sets after every second hit) is written as a checkpoint (5 parameters
// + 15 covariance entries).
//
// Adjoint (one thread per track): with L = sum_k g_k chi2_k, a reverse sweep
// from the last hit reloads each checkpoint, recomputes the transport and
// update (and the state between two checkpoints), and applies their exact derivatives: of the update (gain, chi2,
// covariance) and of the transport including the dependence of the Jacobian
// on the state and on the step length, which the calibration moves.  The
// symmetric covariance carries a symmetric adjoint G with
// dL = sum_ij G_ij dC_ij.  Hit gradients are written per hit; the theta
// gradient is reduced per block in a fixed order, then over blocks.
//
// What bounds them: few tracks, the serial chain of one track's hits, at 4.3
// cycles per VALU instruction (forward 1.15 us a hit, then 0.9; adjoint 1.9,
// then 1.6, on 400 tracks of up to 152 hits, with the short division and root
// sequences and without waits for hits); many, the checkpoints (80 or 40 bytes
// a hit written and read back) and then the adjoint's instructions.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "exact_fp32.hpp"
#include "tpc_internal.hpp"

namespace tpc {

namespace {

__device__ __forceinline__ int lt(int i, int j) { return i >= j ? i * (i + 1) / 2 + j : j * (j + 1) / 2 + i; }

struct CalibModel {
    float DL, VD, TH, UC, US;
    float iUS, iDL;      // 1 / US, 1 / DL (taken once on the host)
};

inline CalibModel make_calib(const tpc_calib_model& m)
{
    return CalibModel{m.drift_len, m.vd, m.tan_half, m.u_centre, m.u_scale, 1.0f / m.u_scale,
                      1.0f / m.drift_len};
}

struct CalHit {
    float x, y, z;      // calibrated plane, y, z
    float xr, yr, dr;   // raw plane x_r, raw y, raw drift length
    float iv;           // 1 / (x_r tan_half)
    float d, u, v;      // calibrated drift, basis coordinates
};

// Quotient by a row's xr tan_half; iv: its reciprocal.  kIn: those of all
// rows are in the short division's range (a geometry of centimetres lies
// within 2^3 and 2^6).  The kernels branch on it once: with a branch at every
// hit the refit of 16,783 tracks took 135 us for 128.
template <bool kIn>
__device__ __forceinline__ float row_div(float a, float b, float iv)
{
    return kIn ? div_exact_special(a, b, iv) : a / b;
}

// iv, kIn: as for row_div.  (The forward functions write
// their fused multiply-adds out: left to the compiler, the choice of the
// product that is fused changed with the code around, and a low-momentum
// track's gradient with it.  kEnd: a hit that starts a pass or ends the
// reverse sweep, whose drift is rounded once less, as it always was.)
template <bool kEnd, bool kIn>
__device__ __forceinline__ CalHit calibrate(const float* th, float xr, float iv, float yr, float zr,
                                            float sd, const CalibModel& cm)
{
    CalHit h;
    h.xr = xr;
    h.iv = iv;
    h.yr = yr;
    h.dr = fmaf(-sd, zr, cm.DL);
    const float scale = 1.0f + th[0];
    const float drift = kEnd ? fmaf(-cm.VD, th[1], h.dr) : h.dr - cm.VD * th[1];
    h.d = scale * drift;
    h.z = sd * (kEnd ? fmaf(-scale, drift, cm.DL) : cm.DL - h.d);
    h.u = (xr - cm.UC) * cm.iUS;
    h.v = row_div<kIn>(yr, xr * cm.TH, iv);
    const float w = h.d * cm.iDL;
    const float b[7] = {1.0f, h.u, h.v, h.u * h.u, h.u * h.v, h.v * h.v, w};
    float dr = th[2], drphi = th[9];
#pragma unroll
    for (int j = 1; j < 7; ++j) {
        dr = fmaf(th[2 + j], b[j], dr);
        drphi = fmaf(th[9 + j], b[j], drphi);
    }
    h.x = xr + dr;
    h.y = yr + drphi;
    return h;
}

// reverse of calibrate: adjoints (X, Y, Z) of the calibrated point ->
// raw (y, z) adjoints, accumulated theta adjoint
template <bool kIn>
__device__ __forceinline__ void calibrate_adj(const float* th, const CalHit& h, float sd,
                                              const CalibModel& cm, float X, float Y, float Z,
                                              double* gth, float& gyr, float& gzr)
{
    // reverse-mode arithmetic: compared with the float64 adjoint within a
    // tolerance, so products and sums may contract into fused multiply-adds.
    // The theta adjoint is summed in float64 (per lane over its hits, then
    // over lanes and blocks): it is a sum of ~1e8 terms that cancel at the
    // calibration's minimum, where float32 sums would leave a noise floor
    // that stops the fit short of it.
#pragma clang fp contract(fast)
    const float w = h.d * cm.iDL;
    const float b[7] = {1.0f, h.u, h.v, h.u * h.u, h.u * h.v, h.v * h.v, w};
    float bb[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        gth[2 + j] += (double)(X * b[j]);
        gth[9 + j] += (double)(Y * b[j]);
        bb[j] = X * th[2 + j] + Y * th[9 + j];
    }
    const float vb = bb[2] + bb[4] * h.u + 2.0f * bb[5] * h.v;
    gyr = Y + row_div<kIn>(vb, h.xr * cm.TH, h.iv);
    const float db = bb[6] * cm.iDL - Z * sd;
    gth[0] += (double)(db * (h.dr - cm.VD * th[1]));
    gth[1] += (double)(-db * (1.0f + th[0]) * cm.VD);
    gzr = -sd * (1.0f + th[0]) * db;
}

// Per pad row: the plane and the reciprocal of plane times tan_half, in LDS;
// true if all of these are in the short division's range (a barrier: the
// table is whole when it returns).
__device__ __forceinline__ bool load_rows(const float* __restrict__ row_x, int n_rows, float th,
                                          float2* xs)
{
    bool in = true;
    for (int i = threadIdx.x; i < 256; i += blockDim.x) {
        const float x = i < n_rows ? row_x[i] : 0.0f;
        const float b = fabsf(x * th);
        in &= i >= n_rows || (b >= kDivMin && b <= kDivMax);
        xs[i] = make_float2(x, 1.0f / (x * th));
    }
    return __builtin_amdgcn_readfirstlane(__syncthreads_and(in));
}

struct Prop {
    float dx, k, s2, T, q, L, a, a2, g, S, Ts, kdx, Tw, LT, G1, Sk;
    float ic1, ic2, icc, iq;        // reciprocals of c1, c2, c1 + c2 and q
    float e1, e2;                   // s / c1, s2 / c2
    float ys, yw, zs, zt, zw, sw;   // non-trivial Jacobian entries
    float FC[5][5];                 // F C
};

// transport of (p, C) by dx; fills the intermediates; false when |s| at
// either end of the step is not below s_max
__device__ __forceinline__ bool prop_fwd(float* p, float* C, float dx, float curv, float s_max,
                                         Prop& P)
{
    const float s = p[2], t = p[3], w = p[4];
    P.dx = dx;
    P.k = curv * w;
    P.s2 = fmaf(P.k, dx, s);
    if (!(fabsf(s) < s_max) || !(fabsf(P.s2) < s_max)) return false;
    const float u1 = (1.0f - s) * (1.0f + s), u2 = (1.0f - P.s2) * (1.0f + P.s2);
    if (s_max <= 1.0f) {
        // u >= 2^-24: the short sequences are the correctly rounded operations
        const float c1 = sqrt_exact(u1), c2 = sqrt_exact(u2);
        P.icc = rcp_exact(c1 + c2);
        P.ic1 = rcp_exact(c1);
        P.ic2 = rcp_exact(c2);
        P.e1 = div_exact(s, c1, P.ic1);
        P.e2 = div_exact(P.s2, c2, P.ic2);
        P.T = (s + P.s2) * P.icc;
        P.q = sqrt_exact(fmaf(P.T, P.T, 1.0f));
        P.iq = rcp_exact(P.q);
        P.LT = div_exact(dx * P.T, P.q, P.iq);   // 1 <= q <= 2^12
    } else {
        const float c1 = sqrtf(u1), c2 = sqrtf(u2);
        P.icc = 1.0f / (c1 + c2);
        P.ic1 = 1.0f / c1;
        P.ic2 = 1.0f / c2;
        P.e1 = s / c1;
        P.e2 = P.s2 / c2;
        P.T = (s + P.s2) * P.icc;
        P.q = sqrtf(fmaf(P.T, P.T, 1.0f));
        P.iq = 1.0f / P.q;
        P.LT = dx * P.T / P.q;
    }
    P.L = dx * P.q;
    P.a = 0.5f * P.k * P.L;
    P.a2 = P.a * P.a;
    P.g = fmaf(P.a2, fmaf(P.a2, fmaf(P.a2, 5.0f / 112.0f, 3.0f / 40.0f), 1.0f / 6.0f), 1.0f);
    P.S = P.L * P.g;
    P.Ts = fmaf(P.T, P.e1 + P.e2, 2.0f) * P.icc;
    P.kdx = curv * dx;
    P.Tw = P.kdx * fmaf(P.T, P.e2, 1.0f) * P.icc;
    P.G1 = fmaf(P.a2, fmaf(P.a2, fmaf(P.a2, 5.0f / 16.0f, 3.0f / 8.0f), 0.5f), 1.0f);
    P.Sk = P.L * P.L * P.a * fmaf(P.a2, fmaf(P.a2, 15.0f / 112.0f, 3.0f / 20.0f), 1.0f / 6.0f);
    P.ys = dx * P.Ts;
    P.yw = dx * P.Tw;
    const float m1 = P.G1 * P.LT;
    P.zs = t * m1 * P.Ts;
    P.zt = P.S;
    P.zw = t * fmaf(P.Sk, curv, m1 * P.Tw);
    P.sw = P.kdx;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const float cy = C[lt(0, j)], cz = C[lt(1, j)], cs = C[lt(2, j)];
        const float ct = C[lt(3, j)], cw = C[lt(4, j)];
        P.FC[0][j] = fmaf(P.yw, cw, fmaf(P.ys, cs, cy));
        P.FC[1][j] = fmaf(P.zw, cw, fmaf(P.zt, ct, fmaf(P.zs, cs, cz)));
        P.FC[2][j] = fmaf(P.sw, cw, cs);
        P.FC[3][j] = ct;
        P.FC[4][j] = cw;
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const float* B = P.FC[i];
        C[lt(i, 0)] = fmaf(P.yw, B[4], fmaf(P.ys, B[2], B[0]));
        if (i >= 1) C[lt(i, 1)] = fmaf(P.zw, B[4], fmaf(P.zt, B[3], fmaf(P.zs, B[2], B[1])));
        if (i >= 2) C[lt(i, 2)] = fmaf(P.sw, B[4], B[2]);
        if (i >= 3) C[lt(i, 3)] = B[3];
        if (i >= 4) C[lt(i, 4)] = B[4];
    }
    p[0] = fmaf(dx, P.T, p[0]);
    p[1] = fmaf(t, P.S, p[1]);
    p[2] = P.s2;
    return true;
}

struct Upd {
    float r0, r1, B00, B10, B11;
    float A0[5], A1[5], K0[5], K1[5];
};

__device__ __forceinline__ float upd_fwd(float* p, float* C, float my, float mz, float sy2,
                                         float sz2, Upd& U)
{
    U.r0 = my - p[0];
    U.r1 = mz - p[1];
    const float S00 = C[0] + sy2, S10 = C[1], S11 = C[2] + sz2;
    const float idet = rcp_any(fmaf(S00, S11, -(S10 * S10)));
    U.B00 = S11 * idet;
    U.B10 = -S10 * idet;
    U.B11 = S00 * idet;
    const float chi2 = fmaf(U.r0, fmaf(U.B00, U.r0, U.B10 * U.r1),
                            U.r1 * fmaf(U.B10, U.r0, U.B11 * U.r1));
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        U.A0[i] = C[lt(i, 0)];
        U.A1[i] = C[lt(i, 1)];
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        U.K0[i] = fmaf(U.A0[i], U.B00, U.A1[i] * U.B10);
        U.K1[i] = i == 1 ? fmaf(U.A1[i], U.B11, U.A0[i] * U.B10)
                         : fmaf(U.A0[i], U.B10, U.A1[i] * U.B11);
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        p[i] += fmaf(U.K0[i], U.r0, U.K1[i] * U.r1);
#pragma unroll
        for (int j = 0; j <= i; ++j)
            C[lt(i, j)] -= fmaf(U.K0[i], U.A0[j], U.K1[i] * U.A1[j]);
    }
    return chi2;
}

// adjoint of the update: in pb (5), G (15, symmetric adjoint) of the
// updated state; out the same for the predicted state, and the adjoints of
// the measurement
__device__ __forceinline__ void upd_adj(const Upd& U, float cb, float* pb, float* G, float& myb,
                                        float& mzb)
{
    // reverse-mode arithmetic: compared with the float64 adjoint within a
    // tolerance, so products and sums may contract into fused multiply-adds
#pragma clang fp contract(fast)
    float Kb0[5], Kb1[5];
    float rb0 = 0.0f, rb1 = 0.0f;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        Kb0[i] = pb[i] * U.r0;
        Kb1[i] = pb[i] * U.r1;
        rb0 += U.K0[i] * pb[i];
        rb1 += U.K1[i] * pb[i];
    }
    // M = G A (5x2)
    float M0[5], M1[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        float m0 = 0.0f, m1 = 0.0f;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const float gij = G[lt(i, j)];
            m0 += gij * U.A0[j];
            m1 += gij * U.A1[j];
        }
        M0[i] = m0;
        M1[i] = m1;
    }
    // Ab = -2 M B + Kb B ; Bb = -A^T M + A^T Kb + cb r r^T
    float Ab0[5], Ab1[5];
    float Bb00 = cb * U.r0 * U.r0, Bb01 = cb * U.r0 * U.r1, Bb10 = Bb01, Bb11 = cb * U.r1 * U.r1;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const float e0 = Kb0[i] - 2.0f * M0[i], e1 = Kb1[i] - 2.0f * M1[i];
        Ab0[i] = e0 * U.B00 + e1 * U.B10;
        Ab1[i] = e0 * U.B10 + e1 * U.B11;
        const float f0 = Kb0[i] - M0[i], f1 = Kb1[i] - M1[i];
        Bb00 += U.A0[i] * f0;
        Bb01 += U.A0[i] * f1;
        Bb10 += U.A1[i] * f0;
        Bb11 += U.A1[i] * f1;
    }
    // r: chi2 term
    rb0 += 2.0f * cb * (U.B00 * U.r0 + U.B10 * U.r1);
    rb1 += 2.0f * cb * (U.B10 * U.r0 + U.B11 * U.r1);
    // S adjoint: -B sym(Bb) B
    const float s00 = Bb00, s11 = Bb11, s01 = 0.5f * (Bb01 + Bb10);
    const float t00 = U.B00 * s00 + U.B10 * s01, t01 = U.B00 * s01 + U.B10 * s11;
    const float t10 = U.B10 * s00 + U.B11 * s01, t11 = U.B10 * s01 + U.B11 * s11;
    const float Sb00 = -(t00 * U.B00 + t01 * U.B10);
    const float Sb10 = -(t10 * U.B00 + t11 * U.B10);
    const float Sb11 = -(t10 * U.B10 + t11 * U.B11);
    G[0] += Sb00;
    G[1] += Sb10;
    G[2] += Sb11;
    // A = C[:, 0:2], symmetric embedding
    G[0] += Ab0[0];
    G[2] += Ab1[1];
    G[1] += 0.5f * (Ab0[1] + Ab1[0]);
#pragma unroll
    for (int i = 2; i < 5; ++i) {
        G[lt(i, 0)] += 0.5f * Ab0[i];
        G[lt(i, 1)] += 0.5f * Ab1[i];
    }
    myb = rb0;
    mzb = rb1;
    pb[0] -= rb0;
    pb[1] -= rb1;
}

// adjoint of the transport: in pb, G of the transported state; out those of
// the state before it (p0: that state), and the step-length adjoint
__device__ __forceinline__ float prop_adj(const Prop& P, const float* p0, const float* C0,
                                          float curv, float* pb, float* G)
{
    // reverse-mode arithmetic: compared with the float64 adjoint within a
    // tolerance, so products and sums may contract into fused multiply-adds
#pragma clang fp contract(fast)
    const float s = p0[2], t = p0[3];
    // F-bar = 2 G F C for the six free entries
    auto gfc = [&](int a, int b) {
        float v = 0.0f;
#pragma unroll
        for (int j = 0; j < 5; ++j) v += G[lt(a, j)] * P.FC[j][b];
        return 2.0f * v;
    };
    const float Fys = gfc(0, 2), Fyw = gfc(0, 4), Fzs = gfc(1, 2), Fzt = gfc(1, 3),
                Fzw = gfc(1, 4), Fsw = gfc(2, 4);
    // G <- F^T G F
    float E[5][5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const float g0 = G[lt(i, 0)], g1 = G[lt(i, 1)], g2 = G[lt(i, 2)];
        E[i][0] = g0;
        E[i][1] = g1;
        E[i][2] = g2 + g0 * P.ys + g1 * P.zs;
        E[i][3] = G[lt(i, 3)] + g1 * P.zt;
        E[i][4] = G[lt(i, 4)] + g0 * P.yw + g1 * P.zw + g2 * P.sw;
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            float v = E[i][j];
            if (i == 2) v += P.ys * E[0][j] + P.zs * E[1][j];
            if (i == 3) v += P.zt * E[1][j];
            if (i == 4) v += P.yw * E[0][j] + P.zw * E[1][j] + P.sw * E[2][j];
            G[lt(i, j)] = v;
        }
    }
    (void)C0;
    // state part: y' = y + dx T, z' = z + t S, s' = s2, t' = t, w' = w
    float Tb = pb[0] * P.dx, dxb = pb[0] * P.T, Sb = pb[1] * t, s2b = pb[2];
    float tb = pb[3] + pb[1] * P.S, wb = pb[4];
    // Jacobian entries
    const float m1 = P.G1 * P.LT;
    float Tsb = 0.0f, Twb = 0.0f, m1b = 0.0f, Skb = 0.0f, kdxb = 0.0f;
    dxb += Fys * P.Ts;
    Tsb += Fys * P.dx;
    dxb += Fyw * P.Tw;
    Twb += Fyw * P.dx;
    tb += Fzs * m1 * P.Ts;
    m1b += Fzs * t * P.Ts;
    Tsb += Fzs * t * m1;
    Sb += Fzt;
    tb += Fzw * (m1 * P.Tw + P.Sk * curv);
    m1b += Fzw * t * P.Tw;
    Twb += Fzw * t * m1;
    Skb += Fzw * t * curv;
    kdxb += Fsw;
    const float G1b = m1b * P.LT;
    float LTb = m1b * P.G1;
    // Sk = L^2 a h(a2)
    const float h = (1.0f / 6.0f) + P.a2 * ((3.0f / 20.0f) + P.a2 * (15.0f / 112.0f));
    const float hp = (3.0f / 20.0f) + 2.0f * P.a2 * (15.0f / 112.0f);
    float Lb = Skb * 2.0f * P.L * P.a * h;
    float ab = Skb * P.L * P.L * h;
    float a2b = Skb * P.L * P.L * P.a * hp;
    // G1 = 1 + a2 (1/2 + a2 (3/8 + a2 5/16))
    a2b += G1b * (0.5f + P.a2 * (2.0f * (3.0f / 8.0f) + P.a2 * (3.0f * (5.0f / 16.0f))));
    const float iq = P.iq, icc = P.icc, ic1 = P.ic1, ic2 = P.ic2;
    // LT = dx T / q
    dxb += LTb * P.T * iq;
    Tb += LTb * P.dx * iq;
    float qb = -LTb * P.dx * P.T * (iq * iq);
    // Tw = kdx n / cc, n = 1 + T s2 / c2
    const float n = 1.0f + P.T * (P.s2 * ic2);
    kdxb += Twb * n * icc;
    const float nb = Twb * P.kdx * icc;
    float ccb = -Twb * P.Tw * icc;
    Tb += nb * P.s2 * ic2;
    s2b += nb * P.T * ic2;
    float c2b = -nb * P.T * P.s2 * (ic2 * ic2);
    // kdx = curv dx
    dxb += kdxb * curv;
    // Ts = (2 + T e) / cc, e = s/c1 + s2/c2
    const float e = s * ic1 + P.s2 * ic2;
    const float numb = Tsb * icc;
    ccb += -Tsb * P.Ts * icc;
    Tb += numb * e;
    const float eb = numb * P.T;
    float sb = eb * ic1;
    float c1b = -eb * s * (ic1 * ic1);
    s2b += eb * ic2;
    c2b += -eb * P.s2 * (ic2 * ic2);
    // S = L g, g = 1 + a2 (1/6 + a2 (3/40 + a2 5/112))
    Lb += Sb * P.g;
    const float gb = Sb * P.L;
    a2b += gb * ((1.0f / 6.0f) + P.a2 * (2.0f * (3.0f / 40.0f) + P.a2 * (3.0f * (5.0f / 112.0f))));
    // a2 = a^2 ; a = k L / 2
    ab += a2b * 2.0f * P.a;
    float kb = ab * 0.5f * P.L;
    Lb += ab * 0.5f * P.k;
    // L = dx q ; q = sqrt(1 + T^2)
    dxb += Lb * P.q;
    qb += Lb * P.dx;
    Tb += qb * P.T * iq;
    // T = (s + s2) / cc ; cc = c1 + c2
    sb += Tb * icc;
    s2b += Tb * icc;
    ccb += -Tb * P.T * icc;
    c1b += ccb;
    c2b += ccb;
    s2b += c2b * (-P.s2 * ic2);
    sb += c1b * (-s * ic1);
    // s2 = s + k dx ; k = curv w
    sb += s2b;
    kb += s2b * P.dx;
    dxb += s2b * P.k;
    wb += kb * curv;
    pb[0] = pb[0];        // y' = y + ...: dy'/dy = 1
    pb[1] = pb[1];        // z' = z + ...
    pb[2] = sb;
    pb[3] = tb;
    pb[4] = wb;
    return dxb;
}

// Checkpoints are kept in tiles of 64 tracks (one wave): every `stride`-th
// state of the track in lane l of tile g, slot j the state after hit
// j * stride, holds 20 floats (p, C) as five float4 at
// ck4[((g * slots + j) * 5 + q) * 64 + l].  The lanes of a wave that stand
// at the same slot store and load five contiguous 1 KB blocks, and one
// wave's checkpoints are one contiguous block.
__device__ __forceinline__ float4* ck_tile(float* ck, int64_t t, int slots)
{
    return reinterpret_cast<float4*>(ck) + (t / kWave) * (int64_t)slots * 5 * kWave +
           (t & (kWave - 1));
}

__host__ __device__ inline int ck_slots(int n_rows, int stride)
{
    return (n_rows + stride - 1) / stride;
}

__device__ __forceinline__ void store_ck(float4* o, int i, const float* p, const float* C)
{
    o += (int64_t)i * 5 * kWave;
    o[0 * kWave] = make_float4(p[0], p[1], p[2], p[3]);
    o[1 * kWave] = make_float4(p[4], C[0], C[1], C[2]);
    o[2 * kWave] = make_float4(C[3], C[4], C[5], C[6]);
    o[3 * kWave] = make_float4(C[7], C[8], C[9], C[10]);
    o[4 * kWave] = make_float4(C[11], C[12], C[13], C[14]);
}

__device__ __forceinline__ void load_ck(const float4* o, int i, float4* q)
{
    o += (int64_t)i * 5 * kWave;
#pragma unroll
    for (int k = 0; k < 5; ++k) q[k] = o[k * kWave];
}

__device__ __forceinline__ void unpack_ck(const float4* q, float* p, float* C)
{
    p[0] = q[0].x; p[1] = q[0].y; p[2] = q[0].z; p[3] = q[0].w;
    p[4] = q[1].x; C[0] = q[1].y; C[1] = q[1].z; C[2] = q[1].w;
    C[3] = q[2].x; C[4] = q[2].y; C[5] = q[2].z; C[6] = q[2].w;
    C[7] = q[3].x; C[8] = q[3].y; C[9] = q[3].z; C[10] = q[3].w;
    C[11] = q[4].x; C[12] = q[4].y; C[13] = q[4].z; C[14] = q[4].w;
}

__device__ __forceinline__ int wave_max(int v)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const int w = __shfl_xor(v, o, kWave);
        v = w > v ? w : v;
    }
    return v;
}

__device__ __forceinline__ void load_theta(const float* __restrict__ d_theta, float* th)
{
    if (threadIdx.x < 16) th[threadIdx.x] = d_theta[threadIdx.x];
    __syncthreads();
}

// ---- the hits of a wave's tracks, without checkpoints ----------------------
// Read kChunk of every track at a time, a chunk ahead of their use, and put
// into LDS, a column a track, when their chunk begins.
//
// In the order of the track list, a lane reads its own track: its run is
// contiguous, at any alignment of 4 bytes, so these are vector loads.  The
// chunk at slot i0 of a track of n hits holds the hits [base, base + kChunk),
// base = min(i0, n - kChunk), so that the last one reads no entry past the
// track.  Bound by the chain of a track's steps for few tracks, by the lines
// of the list for many, which the tracks in flight push out of the L2s between
// two visits: eight hits a visit, and not four, took 300,000 tracks of 40 to
// 152 hits from 485 to 360 us and a million from 1330 to 950 (16,783: 127 and
// 120).
//
// Through an index, eight lanes read eight hits of one track and the same of
// eight more, the index a chunk further ahead (two loads in a row, each
// waiting for the last, would stand in every chunk's way): bound by a line per
// hit and array for many tracks, where a lane reading its own track's indices
// visits more of their lines.  40 to 152 hits at random places (us; a lane its
// own track, four hits at a time; now): 400 tracks 131, 130; 16,783 179, 162;
// 66,000 392, 375; 131,072 752, 722; 300,000 1780, 1705.
// (Waiting for each instruction's hits of eight tracks took 9000 cycles per 8
// hits, half of the forward kernel's time on 400 tracks.)
constexpr int kChunk = 8;
constexpr int kQuads = kChunk / 4;

typedef float float4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t uint32_u __attribute__((aligned(1)));

struct HitRows {
    const int32_t* __restrict__ idx;
    const uint8_t* __restrict__ row;
    const float* __restrict__ y;
    const float* __restrict__ z;
    const int32_t* __restrict__ off;
};

struct HitChunk {
    float4_u y[kQuads], z[kQuads];
    uint32_t row[kQuads];      // a byte per hit
    int base;
};

// load the chunk at slot i0 of the track of n hits at entry a (past a short
// track the last hit again)
__device__ __forceinline__ void load_chunk(HitChunk& h, const HitRows& in, int a, int n, int i0)
{
    if (n >= kChunk) {
        h.base = i0 < n - kChunk ? i0 : n - kChunk;
        const int e = a + h.base;
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
            h.y[q] = *reinterpret_cast<const float4_u*>(in.y + e + 4 * q);
            h.z[q] = *reinterpret_cast<const float4_u*>(in.z + e + 4 * q);
            h.row[q] = *reinterpret_cast<const uint32_u*>(in.row + e + 4 * q);
        }
        return;
    }
    h.base = 0;
    uint32_t r[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
        const int c = a + (k < n ? k : n - 1);
        h.y[k / 4][k % 4] = in.y[c];
        h.z[k / 4][k % 4] = in.z[c];
        r[k] = in.row[c];
    }
#pragma unroll
    for (int q = 0; q < kQuads; ++q)
        h.row[q] = r[4 * q] | r[4 * q + 1] << 8 | r[4 * q + 2] << 16 | r[4 * q + 3] << 24;
}

// the chunk into the lane's LDS column (plane, y, z, reciprocal of plane
// times tan_half per hit); true if a hit's row is outside the table
__device__ __forceinline__ bool put_chunk(const HitChunk& h, float4* col, const float2* xs,
                                          int n_rows)
{
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
        const int r = (int)(h.row[k / 4] >> (8 * (k % 4))) & 255;
        bad |= r >= n_rows;
        const float2 x = xs[r];
        col[k * kWave] = make_float4(x.x, h.y[k / 4][k % 4], h.z[k / 4][k % 4], x.y);
    }
    return bad;
}

// The same through an index: item j of a lane is hit lane % kChunk of the
// chunk of track lane / kChunk + j * kWave / kChunk of the wave.
constexpr int kItems = kChunk;

struct GatherChunk {
    int c[kItems];                  // clusters of the chunk to load next, -1 past the track
    float y[kItems], z[kItems];
    int r[kItems];                  // -1 past the track
};

__device__ __forceinline__ int gather_track(int j)
{
    return (int)(threadIdx.x & (kWave - 1)) / kChunk + j * (kWave / kChunk);
}

// a, n: entry and hits of the tracks of the lane's items
__device__ __forceinline__ void gather_index(GatherChunk& h, const HitRows& in, const int* a,
                                             const int* n, int i0)
{
    const int i = i0 + (int)(threadIdx.x & (kChunk - 1));
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        h.c[j] = -1;
        if (i < n[j]) h.c[j] = in.idx[a[j] + i];
    }
}

__device__ __forceinline__ void gather_hits(GatherChunk& h, const HitRows& in)
{
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        h.r[j] = -1;
        if (h.c[j] >= 0) {
            h.r[j] = in.row[h.c[j]];
            h.y[j] = in.y[h.c[j]];
            h.z[j] = in.z[h.c[j]];
        }
    }
}

// into the tracks' LDS columns; flags a hit row outside the table in
// bad[track]
__device__ __forceinline__ void put_gather(const GatherChunk& h, float4* hits, int* bad,
                                           const float2* xs, int n_rows)
{
    const int k = threadIdx.x & (kChunk - 1);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        if (h.r[j] < 0) continue;
        const int l = gather_track(j);
        const float2 x = xs[h.r[j]];
        if (h.r[j] >= n_rows) bad[l] = 1;
        hits[k * kWave + l] = make_float4(x.x, h.y[j], h.z[j], x.y);
    }
}

// ---- packed hits, with checkpoints ------------------------------------------
// The checkpoint buffer also holds the hits of the tile's tracks by (slot,
// lane): the forward pass and the adjoint read each slot as whole lines.
// (Read from the CSR a few hits at a time, the 64 tracks of each wave in
// flight keep more lines open than the L2s hold, and every visit fetched its
// line again: 5.5 GB for the 0.86 GB of a million tracks, in each kernel.)
struct PackedHits {
    float2* yz;        // [tile][n_rows][64]
    uint8_t* row;      // [tile][n_rows][64]
    uint8_t* bad;      // [tile][part][64]: a hit's row is outside the table
};

// one lane's hits of a tile
struct PackedCol {
    const float2* yz;
    const uint8_t* row;
};

__device__ __forceinline__ PackedCol packed_col(const PackedHits& h, int64_t q, int n_rows)
{
    const int64_t o = (q / kWave) * (int64_t)n_rows * kWave + (q & (kWave - 1));
    return {h.yz + o, h.row + o};
}

struct RawHit {
    float2 yz;
    int row;
};

__device__ __forceinline__ RawHit raw_at(const PackedCol& c, int i)
{
    return {c.yz[i * kWave], c.row[i * kWave]};
}

}  // namespace

// ---- tile order ---------------------------------------------------------------
// With a checkpoint buffer the tracks are taken in order of decreasing hit
// count (stable: equal counts in track order), so that the 64 tracks of a
// tile have similar lengths: a tile steps to its longest track, storing and
// loading whole checkpoint lines, and tiles of uniformly drawn lengths would
// otherwise move about 1.5 times the checkpoint bytes their tracks need.
// A counting sort by key (n_rows + 1) - min(n, n_rows + 1) in at most
// kOrdRanges runs of tracks, cut from the count on the device: per run the
// key counts (one wave's equal keys found by nine ballots), an exclusive scan
// over (key, run), then every track's position.  What bounds it is the
// launches and the counts: with one run per 256 tracks of the capacity, the
// ordering and its scan took 64 us for the 79,000 tracks that 512 sectors
// leave in buffers many times that size, and now 19; a million tracks take
// 32 either way.
constexpr int kOrdRanges = 512;
constexpr int kOrdBlock = 256;

__device__ __forceinline__ int order_key(const int32_t* __restrict__ off, int64_t t, int n_rows)
{
    const int n = off[t + 1] - off[t];
    const int c = n < 0 ? 0 : n > n_rows + 1 ? n_rows + 1 : n;
    return n_rows + 1 - c;
}

// lanes of the wave holding the same key as this lane (keys below 512)
__device__ __forceinline__ uint64_t same_key(int key)
{
    uint64_t m = ~0ull;
#pragma unroll
    for (int b = 0; b < 9; ++b) {
        const uint64_t v = __ballot((key >> b) & 1);
        m &= ((key >> b) & 1) ? v : ~v;
    }
    return m;
}

// tracks per run: whole blocks, so that a run's chunks are full
__device__ __forceinline__ int64_t order_run(int64_t nt)
{
    const int64_t chunks = (nt + kOrdBlock - 1) / kOrdBlock;
    return (chunks + gridDim.x - 1) / gridDim.x * kOrdBlock;
}

// wc[w][key]: count of the key among wave w's tracks of the chunk at t0 (all
// threads of the block; wc is zero on entry); true where the thread's track
// is below end, key and rank (among the wave's equal keys) are then its own
__device__ __forceinline__ bool order_counts(const int32_t* __restrict__ off, int64_t t0,
                                             int64_t end, int n_rows, int (*wc)[256 + 2],
                                             int& key, int& rank)
{
    const int64_t t = t0 + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    key = t < end ? order_key(off, t, n_rows) : 511;   // 511: no track, no key
    const uint64_t m = same_key(key);
    rank = __popcll(m & ((1ull << lane) - 1ull));
    if (key != 511 && rank == 0) wc[threadIdx.x / kWave][key] = __popcll(m);
    __syncthreads();
    return key != 511;
}

__global__ __launch_bounds__(kOrdBlock) void k_order_count(const int32_t* __restrict__ off,
                                                           const int64_t* __restrict__ d_count,
                                                           int64_t n_tracks, int n_rows,
                                                           int32_t* __restrict__ cnt)
{
    __shared__ int wc[kOrdBlock / kWave][256 + 2], sum[256 + 2];
    const int64_t nt = d_count && *d_count < n_tracks ? *d_count : n_tracks;
    const int nkeys = n_rows + 2;
    for (int k = threadIdx.x; k < nkeys; k += kOrdBlock) {
        sum[k] = 0;
#pragma unroll
        for (int w = 0; w < kOrdBlock / kWave; ++w) wc[w][k] = 0;
    }
    __syncthreads();
    const int64_t run = order_run(nt), t0 = blockIdx.x * run;
    const int64_t end = t0 + run < nt ? t0 + run : nt;
    for (int64_t t = t0; t < end; t += kOrdBlock) {
        int key, rank;
        order_counts(off, t, end, n_rows, wc, key, rank);
        for (int k = threadIdx.x; k < nkeys; k += kOrdBlock) {
#pragma unroll
            for (int w = 0; w < kOrdBlock / kWave; ++w) {
                sum[k] += wc[w][k];
                wc[w][k] = 0;
            }
        }
        __syncthreads();
    }
    for (int k = threadIdx.x; k < nkeys; k += kOrdBlock)
        cnt[(int64_t)k * gridDim.x + blockIdx.x] = sum[k];
}

// after the scan of cnt: position of every track t < nt, order[pos] = t
__global__ __launch_bounds__(kOrdBlock) void k_order_place(const int32_t* __restrict__ off,
                                                           const int64_t* __restrict__ d_count,
                                                           int64_t n_tracks, int n_rows,
                                                           const int32_t* __restrict__ base,
                                                           int32_t* __restrict__ order)
{
    __shared__ int wc[kOrdBlock / kWave][256 + 2], next[256 + 2];
    const int64_t nt = d_count && *d_count < n_tracks ? *d_count : n_tracks;
    const int nkeys = n_rows + 2;
    const int64_t run = order_run(nt), t0 = blockIdx.x * run;
    const int64_t end = t0 + run < nt ? t0 + run : nt;
    if (t0 >= end) return;
    for (int k = threadIdx.x; k < nkeys; k += kOrdBlock) {
        next[k] = base[(int64_t)k * gridDim.x + blockIdx.x];
#pragma unroll
        for (int w = 0; w < kOrdBlock / kWave; ++w) wc[w][k] = 0;
    }
    __syncthreads();
    for (int64_t t = t0; t < end; t += kOrdBlock) {
        int key, rank;
        if (order_counts(off, t, end, n_rows, wc, key, rank)) {
            int pos = next[key] + rank;
            for (int w = 0; w < (int)(threadIdx.x / kWave); ++w) pos += wc[w][key];
            order[pos] = (int32_t)(t + threadIdx.x);
        }
        __syncthreads();
        for (int k = threadIdx.x; k < nkeys; k += kOrdBlock) {
#pragma unroll
            for (int w = 0; w < kOrdBlock / kWave; ++w) {
                next[k] += wc[w][k];
                wc[w][k] = 0;
            }
        }
        __syncthreads();
    }
}

// track of tile position q (q itself past the count, or without an order)
__device__ __forceinline__ int64_t track_at(const int32_t* __restrict__ order, int64_t q,
                                            int64_t nt)
{
    return order && q < nt ? (int64_t)order[q] : q;
}

// The hits of 64 tracks (consecutive in the tile order) into their tile, one
// block per (tile, kPackSlots slots; the last block of a tile also looks at
// the hits past the rows), or per tile where there are enough of them to fill
// the chip: a wave reads kPackRuns tracks' runs at a time, 64 entries of each,
// into LDS, and the block writes the tile slot by slot.
// Streaming: 1M tracks' hits, 0.86 GB read and written.
constexpr int kPackSlots = kWave;
constexpr int kPackRuns = 8;
// tiles from which one block takes a tile: four blocks to a compute unit.
// Blocks of 64 slots find nothing past the longest track of theirs: 300,000
// tracks of 10 hits 66 us and now 53, of 40 hits 97 and 79, a million of 40 to
// 152 600 and 562; 66,000 of 10 hits 21 and 20, 400 tracks need the blocks.
constexpr int64_t kPackWhole = 1024;

__host__ __device__ inline int pack_parts(int n_rows)
{
    return (n_rows + kPackSlots - 1) / kPackSlots;
}

__global__ __launch_bounds__(kBlock) void k_refit_pack(
    HitRows in, const int64_t* __restrict__ d_count, int64_t n_tracks, int n_rows,
    const int32_t* __restrict__ order, PackedHits out)
{
    __shared__ float2 yz[kPackSlots][kWave + 1];
    __shared__ uint8_t rw[kPackSlots][kWave + 4];
    __shared__ int a_[kWave], n_[kWave], bad[kWave], longest;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    constexpr int kWaves = kBlock / kWave;
    const int64_t nt = d_count && *d_count < n_tracks ? *d_count : n_tracks;
    const int parts = pack_parts(n_rows);
    const int64_t tiles = (nt + kWave - 1) / kWave;
    const int split = tiles < kPackWhole ? parts : 1;     // blocks per tile
    for (int64_t u = blockIdx.x; u < tiles * split; u += gridDim.x) {
        const int64_t tile = u / split, tb = tile * kWave;
        const int part = (int)(u % split);
        if (threadIdx.x < kWave) {
            const int64_t t = track_at(order, tb + lane, nt);
            int a = 0, n = 0;
            if (t < nt) {
                a = in.off[t];
                n = in.off[t + 1] - a;
            }
            n = n >= 3 ? n : 0;
            a_[lane] = a;
            n_[lane] = n;
            bad[lane] = 0;
            const int m = wave_max(n);
            if (lane == 0) longest = m;
        }
        __syncthreads();
        const int first = part * kPackSlots;
        const int past = part + 1 < split ? first + kPackSlots : longest;
        for (int i0 = first; i0 < longest && i0 < past; i0 += kPackSlots) {
            const int i = i0 + lane;
            for (int l0 = wid; l0 < kWave; l0 += kWaves * kPackRuns) {
                int c[kPackRuns];
                float y[kPackRuns], z[kPackRuns];
                uint8_t r[kPackRuns];
#pragma unroll
                for (int k = 0; k < kPackRuns; ++k) {
                    const int l = l0 + k * kWaves;
                    c[k] = -1;
                    if (i < n_[l]) c[k] = in.idx ? in.idx[a_[l] + i] : a_[l] + i;
                }
#pragma unroll
                for (int k = 0; k < kPackRuns; ++k)
                    if (c[k] >= 0) {
                        y[k] = in.y[c[k]];
                        z[k] = in.z[c[k]];
                        r[k] = in.row[c[k]];
                    }
#pragma unroll
                for (int k = 0; k < kPackRuns; ++k)
                    if (c[k] >= 0) {
                        const int l = l0 + k * kWaves;
                        yz[lane][l] = make_float2(y[k], z[k]);
                        rw[lane][l] = r[k];
                        if (r[k] >= n_rows) bad[l] = 1;
                    }
            }
            __syncthreads();
            const int n = n_[lane];
            for (int k = wid; k < kPackSlots && i0 + k < n_rows && i0 + k < longest; k += kWaves)
                if (i0 + k < n) {
                    const int64_t o = (tile * n_rows + i0 + k) * kWave + lane;
                    out.yz[o] = yz[k][lane];
                    out.row[o] = rw[k][lane];
                }
            __syncthreads();
        }
        if (threadIdx.x < kWave) {
            uint8_t* b = out.bad + (tile * parts + part) * kWave + lane;
            *b = (uint8_t)bad[lane];
            for (int k = 1; k < parts && split == 1; ++k) b[k * kWave] = 0;
        }
        __syncthreads();
    }
}

constexpr std::true_type kYes{};
constexpr std::false_type kNo{};

// where the forward pass reads its hits
enum { kCsr = 0, kCsrIndex = 1, kPacked = 2 };

// hits, bad: LDS of the readers without checkpoints
template <int kFrom, bool kIn>
__device__ __forceinline__ void refit_fwd(
    const float* th, const float2* xs, float4* hits, int* badl, const HitRows& in,
    const PackedHits& packed, const int8_t* __restrict__ side,
    const int64_t* __restrict__ d_count, int64_t n_tracks, int n_rows, const tpc_params& prm,
    const CalibModel& cm, float* __restrict__ par, float* __restrict__ cov,
    float* __restrict__ chi2_out, int32_t* __restrict__ status, float* __restrict__ ck, int stride,
    const int32_t* __restrict__ order)
{
    constexpr bool kIdx = kFrom == kCsrIndex;
    const int lane = threadIdx.x & (kWave - 1);
    float4* col = hits + lane;
    const int64_t nt = d_count && *d_count < n_tracks ? *d_count : n_tracks;
    // one wave per tile of 64 tracks (consecutive in the tile order)
    for (int64_t tb = blockIdx.x * (int64_t)kWave; tb < nt; tb += (int64_t)gridDim.x * kWave) {
        const int64_t t = track_at(order, tb + lane, nt);
        int a = 0, n = 0;
        if (t < nt) {
            a = in.off[t];
            n = in.off[t + 1] - a;
        }
        // tracks filtered: at least 3 hits, not more hits than rows (a hit
        // row outside the table is found while staging)
        const int ns = n >= 3 ? n : 0;
        const bool fit = n >= 3 && n <= n_rows;
        const int M = wave_max(ns);
        float p[5] = {0, 0, 0, 0, 0}, C[15];
#pragma unroll
        for (int i = 0; i < 15; ++i) C[i] = 0.0f;
        float chi2 = 0.0f, xp = 0.0f;
        bool alive = fit, bad = false;
        int stat = 0;
        const float sd = t < nt && side ? (float)side[t] : 1.0f;
        // every lane of a tile stores every slot up to the wave's longest
        // track (a lane past its own track stores its unchanged state, which
        // nothing reads), so that each store writes whole lines; the tile of
        // the last, partial wave is allocated in full
        float4* ckt =
            kFrom == kPacked ? ck_tile(ck, tb + lane, ck_slots(n_rows, stride)) : nullptr;
        const int M_ck = M < n_rows ? M : n_rows;
        auto start = [&](const CalHit& h0, const CalHit& h2) {
            // state from the first and third hits
            const float dX = h2.x - h0.x;
            const float T0 = (h2.y - h0.y) / dX;
            const float q0 = sqrtf(1.0f + T0 * T0);
            p[0] = h0.y;
            p[1] = h0.z;
            p[2] = T0 / q0;
            p[3] = (h2.z - h0.z) / (dX * q0);
            p[4] = 0.0f;
            C[0] = prm.sigma_y2;
            C[2] = prm.sigma_z2;
            C[5] = prm.c_ss0;
            C[9] = prm.c_tt0;
            C[14] = prm.c_ww0;
            xp = h0.x;
        };
        auto step = [&](const CalHit& h) {
            Prop P;
            if (prop_fwd(p, C, h.x - xp, prm.curv, prm.s_max, P)) {
                Upd U;
                chi2 += upd_fwd(p, C, h.y, h.z, prm.sigma_y2, prm.sigma_z2, U);
                xp = h.x;
            } else {
                stat = 2;
                alive = false;
            }
        };
        if (kFrom == kPacked) {
            const PackedCol hp = packed_col(packed, tb + lane, n_rows);
            auto cal = [&](const RawHit& r, auto end) {
                const float2 x = xs[r.row];
                return calibrate<end(), kIn>(th, x.x, x.y, r.yz.x, r.yz.y, sd, cm);
            };
            // hits of the next two slots, in flight
            RawHit r1{}, r2{};
            if (alive) {
                r1 = raw_at(hp, 1);
                r2 = raw_at(hp, 2);
                start(cal(raw_at(hp, 0), kYes), cal(r2, kYes));
            }
            if (M_ck > 1) store_ck(ckt, 0, p, C);
            for (int i = 1; i < M_ck; ++i) {
                const RawHit r = r1;
                r1 = r2;
                if (alive && i + 2 < n) r2 = raw_at(hp, i + 2);
                if (alive && i < n) step(cal(r, kNo));
                if (i + 1 < M_ck && (stride == 1 || !(i & 1))) store_ck(ckt, i / stride, p, C);
            }
            const int parts = pack_parts(n_rows);
            for (int k = 0; k < parts; ++k)
                bad |= packed.bad[(tb / kWave * parts + k) * kWave + lane] != 0;
        } else {
            int aj[kItems], nj[kItems];
            GatherChunk ng;
            HitChunk nx{};
            if (kIdx) {
#pragma unroll
                for (int j = 0; j < kItems; ++j) {
                    aj[j] = __shfl(a, gather_track(j), kWave);
                    nj[j] = __shfl(ns, gather_track(j), kWave);
                }
                gather_index(ng, in, aj, nj, 0);
                gather_hits(ng, in);
                gather_index(ng, in, aj, nj, kChunk);
                badl[lane] = 0;
                __syncthreads();
            } else if (ns > 0) {
                load_chunk(nx, in, a, n, 0);
            }
            for (int i0 = 0; i0 < M; i0 += kChunk) {
                const int base = kIdx ? i0 : nx.base;
                if (kIdx) {
                    put_gather(ng, hits, badl, xs, n_rows);
                    __syncthreads();
                    if (i0 + kChunk < M) {
                        gather_hits(ng, in);
                        gather_index(ng, in, aj, nj, i0 + 2 * kChunk);
                    }
                } else {
                    if (i0 < ns) bad |= put_chunk(nx, col, xs, n_rows);
                    if (i0 + kChunk < ns) load_chunk(nx, in, a, n, i0 + kChunk);
                }
                auto cal = [&](int k, auto end) {
                    const float4 r = col[k * kWave];
                    return calibrate<end(), kIn>(th, r.x, r.w, r.y, r.z, sd, cm);
                };
                if (i0 == 0 && alive) start(cal(0, kYes), cal(2, kYes));
                const int i_hi = i0 + kChunk < M ? i0 + kChunk : M;
                for (int i = i0 > 1 ? i0 : 1; i < i_hi; ++i)
                    if (alive && i < n) step(cal(i - base, kNo));
                if (kIdx) __syncthreads();       // the next chunk goes to the same place
            }
            if (kIdx) bad = badl[lane] != 0;
        }
        if (t < nt) {
            if (n < 3) stat = 1;
            else if (bad) stat = 3;
            else if (n > n_rows) stat = 4;
            if (stat == 1 || stat == 3 || stat == 4) {
                chi2 = 0.0f;
#pragma unroll
                for (int i = 0; i < 5; ++i) p[i] = 0.0f;
#pragma unroll
                for (int i = 0; i < 15; ++i) C[i] = 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 5; ++i) par[t * 5 + i] = p[i];
#pragma unroll
            for (int i = 0; i < 15; ++i) cov[t * 15 + i] = C[i];
            chi2_out[t] = chi2;
            status[t] = stat;
        }
    }
}

template <int kFrom>
__global__ __launch_bounds__(kWave) void k_refit_fwd(
    HitRows in, PackedHits packed, const int8_t* __restrict__ side, const int64_t* __restrict__ d_count,
    int64_t n_tracks, int n_rows, const float* __restrict__ row_x, tpc_params prm, CalibModel cm,
    const float* __restrict__ d_theta, float* __restrict__ par, float* __restrict__ cov,
    float* __restrict__ chi2_out, int32_t* __restrict__ status, float* __restrict__ ck, int stride,
    const int32_t* __restrict__ order)
{
    __shared__ float th[16];
    __shared__ float2 xs[256];
    __shared__ float4 hits[kFrom == kPacked ? kWave : kChunk * kWave];
    __shared__ int bad[kFrom == kCsrIndex ? kWave : 1];     // by track of the wave
    load_theta(d_theta, th);
    if (load_rows(row_x, n_rows, cm.TH, xs))
        refit_fwd<kFrom, true>(th, xs, hits, bad, in, packed, side, d_count, n_tracks, n_rows, prm,
                               cm, par, cov, chi2_out, status, ck, stride, order);
    else
        refit_fwd<kFrom, false>(th, xs, hits, bad, in, packed, side, d_count, n_tracks, n_rows, prm,
                                cm, par, cov, chi2_out, status, ck, stride, order);
}

// Hit gradients of kGrads slots leave together: 16 lanes write 16 entries of
// one track, so that most of a line is written by one instruction.
constexpr int kGrads = 16;

// grads: the hit gradients of kGrads slots, y then z, by lane
template <int kStride, bool kIn>
__device__ __forceinline__ void refit_adj(
    const float* th, const float2* xs, float (*grads)[kWave][kGrads + 1],
    const int32_t* __restrict__ off, const PackedHits& packed, const int8_t* __restrict__ side,
    const int64_t* __restrict__ d_count, int64_t n_tracks, int n_rows, const tpc_params& prm,
    const CalibModel& cm, const float* __restrict__ ck, const int32_t* __restrict__ status,
    const float* __restrict__ gchi2, const float* __restrict__ seed_p,
    const float* __restrict__ seed_x, float* __restrict__ gy, float* __restrict__ gz,
    double* __restrict__ partials, const int32_t* __restrict__ order)
{
    double gth[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) gth[k] = 0.0;
    const int64_t nt = d_count && *d_count < n_tracks ? *d_count : n_tracks;
    const int lane = threadIdx.x & (kWave - 1);
    // one wave per tile of 64 tracks; the reverse sweep runs over the slots
    // of the tile in lockstep (slot i is active in the lanes whose track has
    // more than i hits), so that hit and checkpoint loads are whole lines
    for (int64_t tb = blockIdx.x * (int64_t)kWave; tb < nt; tb += (int64_t)gridDim.x * kWave) {
        const int64_t t = track_at(order, tb + lane, nt);
        int a = 0, n = 0;
        if (t < nt) {
            a = off[t];
            n = off[t + 1] - a;
        }
        const bool fit = t < nt && n >= 3 && status[t] == 0;
        if (t < nt && !fit)
            for (int i = 0; i < n; ++i) {
                gy[a + i] = 0.0f;
                gz[a + i] = 0.0f;
            }
        const int ne = fit ? n : 0;
        const int M = wave_max(ne);
        if (M == 0) continue;
        const PackedCol hp = packed_col(packed, tb + lane, n_rows);
        const float4* ckt = ck_tile(const_cast<float*>(ck), tb + lane, ck_slots(n_rows, kStride));
        const float sd = fit && side ? (float)side[t] : 1.0f;
        const float cb = fit ? gchi2[t] : 0.0f;
        // adjoint of the final state: the seed of the caller's terms in the
        // state after the last update (dL/dp), zero without one
        float pb[5] = {0, 0, 0, 0, 0}, G[15];
        if (fit && seed_p)
#pragma unroll
            for (int i = 0; i < 5; ++i) pb[i] = seed_p[t * 5 + i];
#pragma unroll
        for (int i = 0; i < 15; ++i) G[i] = 0.0f;
        auto cal = [&](const RawHit& r, auto end) {
            const float2 x = xs[r.row];
            return calibrate<end(), kIn>(th, x.x, x.y, r.yz.x, r.yz.y, sd, cm);
        };
        CalHit cur{};
        // step i needs hit i - 1, with every second checkpoint hit i - 2 too;
        // the raw hit of the next step's last need is loaded a step ahead
        CalHit prev{};
        RawHit r1{};
        // the checkpoint at or below slot i - 1, loaded a step ahead
        float4 ck4[5];
        if (fit) {
            cur = cal(raw_at(hp, n - 1), kYes);
            if (kStride == 2) prev = cal(raw_at(hp, n - 2), kNo);
            r1 = raw_at(hp, n - 1 - kStride);
            load_ck(ckt, (n - 2) / kStride, ck4);
        }
        // dL/dx of the last hit's calibrated plane from the caller's terms
        float Xcarry = fit && seed_x ? seed_x[t] : 0.0f;
        float X2 = 0.0f, Y2 = 0.0f, Z2 = 0.0f;
        // the gradients leave kGrads slots at a time
        for (int top = M - 1; top >= 1;) {
            const int lo = top / kGrads * kGrads > 1 ? top / kGrads * kGrads : 1;
            for (int i = top; i >= lo; --i) {
                if (i >= ne) continue;
                const RawHit r2 = r1;
                if (i > kStride) r1 = raw_at(hp, i - 1 - kStride);
                CalHit next{};
                if (kStride == 1) prev = cal(r2, kNo);
                else if (i >= 2) next = cal(r2, kNo);
                float p[5], C[15];
                unpack_ck(ck4, p, C);
                if (kStride == 2 && !(i & 1)) {
                    // the state after hit i - 1 from that after hit i - 2
                    const float x0 = i == 2 ? cal(r2, kYes).x : next.x;
                    Prop P;
                    Upd U;
                    prop_fwd(p, C, prev.x - x0, prm.curv, prm.s_max, P);
                    upd_fwd(p, C, prev.y, prev.z, prm.sigma_y2, prm.sigma_z2, U);
                } else if (i > kStride) {
                    load_ck(ckt, (i - 1) / kStride - 1, ck4);
                }
                const float p0[5] = {p[0], p[1], p[2], p[3], p[4]};
                Prop P;
                prop_fwd(p, C, cur.x - prev.x, prm.curv, prm.s_max, P);
                Upd U;
                upd_fwd(p, C, cur.y, cur.z, prm.sigma_y2, prm.sigma_z2, U);
                float myb, mzb;
                upd_adj(U, cb, pb, G, myb, mzb);
                const float dxb = prop_adj(P, p0, nullptr, prm.curv, pb, G);
                const float Xi = Xcarry + dxb;
                if (i == 2) {
                    X2 = Xi;
                    Y2 = myb;
                    Z2 = mzb;
                } else {
                    float gyr, gzr;
                    calibrate_adj<kIn>(th, cur, sd, cm, Xi, myb, mzb, gth, gyr, gzr);
                    grads[0][lane][i - lo] = gyr;
                    grads[1][lane][i - lo] = gzr;
                }
                Xcarry = -dxb;
                cur = prev;
                if (kStride == 2) prev = next;
            }
            // hits lo .. top, but hit 2: kGrads lanes write one track's run
            __syncthreads();
            const int i = lo + (lane & (kGrads - 1));
            for (int l = lane / kGrads; l < kWave; l += kWave / kGrads) {
                const int al = __shfl(a, l, kWave), nl = __shfl(ne, l, kWave);
                if (i <= top && i < nl && i != 2) {
                    gy[al + i] = grads[0][l][i - lo];
                    gz[al + i] = grads[1][l][i - lo];
                }
            }
            __syncthreads();              // the next slots go to the same place
            top = lo - 1;
        }
        if (!fit) continue;
        // initial state: y, z of hit 0, direction from hit 0 to hit 2
        const CalHit h0 = cur;
        const CalHit h2 = cal(raw_at(hp, 2), kYes);
        const float dX = h2.x - h0.x;
        const float T0 = (h2.y - h0.y) / dX;
        const float q0 = sqrtf(1.0f + T0 * T0);
        const float tt = (h2.z - h0.z) / (dX * q0);
        float Y0 = pb[0], Z0 = pb[1], X0 = Xcarry;
        float T0b = pb[2] / (q0 * q0 * q0);
        const float den = dX * q0;
        Z2 += pb[3] / den;
        Z0 -= pb[3] / den;
        const float denb = -pb[3] * tt / den;
        float dXb = denb * q0;
        const float q0b = denb * dX;
        T0b += q0b * T0 / q0;
        Y2 += T0b / dX;
        Y0 -= T0b / dX;
        dXb -= T0b * T0 / dX;
        X2 += dXb;
        X0 -= dXb;
        float gyr, gzr;
        calibrate_adj<kIn>(th, h0, sd, cm, X0, Y0, Z0, gth, gyr, gzr);
        gy[a] = gyr;
        gz[a] = gzr;
        calibrate_adj<kIn>(th, h2, sd, cm, X2, Y2, Z2, gth, gyr, gzr);
        gy[a + 2] = gyr;
        gz[a + 2] = gzr;
    }
    // deterministic wave reduction of the theta adjoint (one wave per block)
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        double v = gth[k];
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
        if (lane == k) partials[blockIdx.x * 16 + k] = v;
    }
}

template <int kStride>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2)))
void k_refit_adj(
    const int32_t* __restrict__ off, PackedHits packed, const int8_t* __restrict__ side,
    const int64_t* __restrict__ d_count, int64_t n_tracks, int n_rows, const float* __restrict__ row_x, tpc_params prm, CalibModel cm,
    const float* __restrict__ d_theta, const float* __restrict__ ck,
    const int32_t* __restrict__ status, const float* __restrict__ gchi2,
    const float* __restrict__ seed_p, const float* __restrict__ seed_x,
    float* __restrict__ gy, float* __restrict__ gz, double* __restrict__ partials,
    const int32_t* __restrict__ order)
{
    __shared__ float th[16];
    __shared__ float2 xs[256];
    __shared__ float grads[2][kWave][kGrads + 1];
    load_theta(d_theta, th);
    if (load_rows(row_x, n_rows, cm.TH, xs))
        refit_adj<kStride, true>(th, xs, grads, off, packed, side, d_count, n_tracks, n_rows, prm,
                                 cm, ck, status, gchi2, seed_p, seed_x, gy, gz, partials, order);
    else
        refit_adj<kStride, false>(th, xs, grads, off, packed, side, d_count, n_tracks, n_rows, prm,
                                  cm, ck, status, gchi2, seed_p, seed_x, gy, gz, partials, order);
}

// sum of the partials of the blocks that had tracks, in a fixed order: block
// k sums parameter k; thread j adds partials j, j + 256, ... of it, then a
// fixed tree.  Bound by the latency of the strided loads, so eight are in
// flight, and the blocks past the count on the device (their partials are
// zero) are left out: 35 us -> 4.8 for the 79,000 tracks of 512 sectors in
// their far larger buffers (16,384 blocks),
// 34 -> 23 for a million.
__global__ __launch_bounds__(kBlock) void k_reduce_theta(const double* __restrict__ partials,
                                                         int nb,
                                                         const int64_t* __restrict__ d_count,
                                                         int64_t n_tracks,
                                                         float* __restrict__ out)
{
    __shared__ double red[kBlock];
    const int k = blockIdx.x;
    const int64_t nt = d_count && *d_count < n_tracks ? *d_count : n_tracks;
    const int64_t tiles = (nt + kWave - 1) / kWave;
    const int nu = tiles < nb ? (int)tiles : nb;
    double v = 0.0;
    for (int b = threadIdx.x; b < nu; b += 8 * kBlock) {
        double p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            p[i] = b + i * kBlock < nu ? partials[(b + i * kBlock) * 16 + k] : 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) v += p[i];
    }
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[k] = (float)red[0];
}

// Beam-axis term of the calibration objective (section 3's online
// calibration with section 2's primaries from the origin): the refit state of
// a track's last hit (par, cov at the calibrated plane of that hit) is
// transported to the plane x = 0 of its sector frame, which holds the beam
// axis, in ceil(x / 20 cm) equal steps; r = (y0, z0) there and
// loss = r^T W r, with W = S^-1, S the transported (y, z) covariance plus
// sigma_v^2 on the diagonal (the chi2 increment of a vertex measurement) --
// or W given by the caller (w_in: held fixed while the calibration moves).
// Derivatives: with respect to the state through the product of the step
// Jacobians, and to the plane of the last hit (moving the plane with the
// state held translates the track along x: dr/dx = -(s0, t) / c0 at the axis
// plane).  Zero (ok = 0) for tracks without a fit or whose transport stops.
// One thread per track.
__global__ __launch_bounds__(kBlock) void k_vertex_residual(
    const int32_t* __restrict__ off, const int32_t* __restrict__ idx,
    const uint8_t* __restrict__ row, const float* __restrict__ y, const float* __restrict__ z,
    const int8_t* __restrict__ side, const int64_t* __restrict__ d_count, int64_t n_tracks,
    const float* __restrict__ row_x, tpc_params prm, CalibModel cm,
    const float* __restrict__ d_theta, const float* __restrict__ par,
    const float* __restrict__ cov, const int32_t* __restrict__ status, float sv2,
    const float* __restrict__ w_in, float* __restrict__ w_out, float* __restrict__ loss,
    float* __restrict__ seed_p, float* __restrict__ seed_x, int8_t* __restrict__ ok)
{
    __shared__ float th[16];
    if (threadIdx.x < 16) th[threadIdx.x] = d_theta[threadIdx.x];
    __syncthreads();
    const int64_t nt = d_count && *d_count < n_tracks ? *d_count : n_tracks;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < nt;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int a = off[t], n = off[t + 1] - a;
        float l = 0.0f, gx = 0.0f, gp[5] = {0, 0, 0, 0, 0}, w[3] = {0, 0, 0};
        bool good = status[t] == 0 && n >= 3;
        if (good) {
            const int c = idx ? idx[a + n - 1] : a + n - 1;
            const float sd = side ? (float)side[t] : 1.0f;
            const float xr = row_x[row[c]];
            const float xl = calibrate<true, false>(th, xr, 0.0f, y[c], z[c], sd, cm).x;
            float p[5], C[15];
#pragma unroll
            for (int i = 0; i < 5; ++i) p[i] = par[t * 5 + i];
#pragma unroll
            for (int i = 0; i < 15; ++i) C[i] = cov[t * 15 + i];
            // rows y, z, sin of the accumulated Jacobian d(p at x)/d(p at xl)
            float J0[5] = {1, 0, 0, 0, 0}, J1[5] = {0, 1, 0, 0, 0}, J2[5] = {0, 0, 1, 0, 0};
            int n_step = (int)ceilf(xl / 20.0f);
            if (n_step < 1) n_step = 1;
            const float dx = (0.0f - xl) / (float)n_step;
            for (int i = 0; i < n_step && good; ++i) {
                Prop P;
                if (!prop_fwd(p, C, dx, prm.curv, prm.s_max, P)) {
                    good = false;
                    break;
                }
                // rows 3, 4 of every step Jacobian are those of the identity
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    const float e3 = k == 3 ? 1.0f : 0.0f, e4 = k == 4 ? 1.0f : 0.0f;
                    const float n0 = J0[k] + P.ys * J2[k] + P.yw * e4;
                    const float n1 = J1[k] + P.zs * J2[k] + P.zt * e3 + P.zw * e4;
                    J2[k] = J2[k] + P.sw * e4;
                    J0[k] = n0;
                    J1[k] = n1;
                }
            }
            if (good) {
                if (w_in) {
                    w[0] = w_in[t * 3];
                    w[1] = w_in[t * 3 + 1];
                    w[2] = w_in[t * 3 + 2];
                } else {
                    const float s00 = C[0] + sv2, s10 = C[1], s11 = C[2] + sv2;
                    const float det = s00 * s11 - s10 * s10;
                    w[0] = s11 / det;
                    w[1] = -s10 / det;
                    w[2] = s00 / det;
                }
                const float y0 = p[0], z0 = p[1];
                const float u0 = w[0] * y0 + w[1] * z0, u1 = w[1] * y0 + w[2] * z0;
                l = y0 * u0 + z0 * u1;
#pragma unroll
                for (int k = 0; k < 5; ++k) gp[k] = 2.0f * (u0 * J0[k] + u1 * J1[k]);
                const float c0 = sqrtf((1.0f - p[2]) * (1.0f + p[2]));
                gx = -2.0f * (u0 * p[2] + u1 * p[3]) / c0;
            }
        }
        loss[t] = l;
#pragma unroll
        for (int k = 0; k < 5; ++k) seed_p[t * 5 + k] = gp[k];
        seed_x[t] = gx;
        if (w_out) {
            w_out[t * 3] = w[0];
            w_out[t * 3 + 1] = w[1];
            w_out[t * 3 + 2] = w[2];
        }
        if (ok) ok[t] = good ? 1 : 0;
    }
}

constexpr int64_t kRefitMaxBlocks = 16384;

static unsigned refit_grid(int64_t n_tracks)
{
    return grid_for_block(n_tracks, kWave, kRefitMaxBlocks);
}

// Every state is a checkpoint, or every second one: half of the 80 bytes a
// hit that bound large sets, for one more forward step per two hits in the
// adjoint.  1M tracks (us, forward + adjoint): 2150 + 2490 with every state,
// 1170 + 2160 with every second; 100,000: 256 + 352, 180 + 357; 400, where
// the adjoint's chain of instructions is what counts: 135 + 246, 122 + 290.
// The line lies where the tracks' waves fill the SIMDs.  (A device count
// below n_tracks does not move it: 16,783 tracks take 169 + 245 in buffers of
// their own, 157 + 303 in buffers for 440,000.)
constexpr int64_t kSparseTracks = int64_t(1) << 16;

// The checkpoint buffer: the tiles, then the tile order (int32 per track),
// the per-(key, run) counts of the ordering, its scan partials and the
// packed hits.  The tiles have the room that kSparseTracks - 1 tracks with
// every state need, also where every second one is kept: a buffer for n
// tracks serves every smaller set.
struct CkLayout {
    size_t order_off, cnt_off, part_off, yz_off, row_off, bad_off, total;
    int64_t nblk;
    int nkeys;
    int stride;
};

static int ck_stride(int64_t n_tracks)
{
    return n_tracks >= kSparseTracks ? 2 : 1;
}

static size_t ck_align(size_t v) { return (v + 255) & ~(size_t)255; }

static CkLayout ck_layout(int64_t n_tracks, int n_rows)
{
    CkLayout L;
    const int64_t tiles = (n_tracks + kWave - 1) / kWave;
    L.nblk = ceil_div(n_tracks > 0 ? n_tracks : 1, kOrdBlock);
    if (L.nblk > kOrdRanges) L.nblk = kOrdRanges;
    L.nkeys = n_rows + 2;
    const int64_t ncnt = L.nblk * L.nkeys;
    L.stride = ck_stride(n_tracks);
    auto states = [&](int64_t n, int stride) {
        return sizeof(float) * (size_t)ceil_div(n, kWave) * kWave *
               (size_t)ck_slots(n_rows, stride) * 20;
    };
    const size_t sparse = states(n_tracks, L.stride);
    const size_t dense = states(std::min(n_tracks, kSparseTracks - 1), 1);
    L.order_off = ck_align(std::max(sparse, dense));
    L.cnt_off = L.order_off + ck_align(sizeof(int32_t) * (size_t)(n_tracks > 0 ? n_tracks : 1));
    L.part_off = L.cnt_off + ck_align(sizeof(int32_t) * (size_t)ncnt);
    L.yz_off = L.part_off + ck_align(sizeof(int64_t) * (size_t)(ceil_div(ncnt, kScanTile) + 1));
    const size_t slots = (size_t)tiles * kWave * (size_t)n_rows;
    L.row_off = L.yz_off + ck_align(sizeof(float2) * slots);
    L.bad_off = L.row_off + ck_align(slots);
    L.total = L.bad_off + (size_t)tiles * kWave * (size_t)pack_parts(n_rows);
    return L;
}

static const int32_t* ck_order(const float* ck, int64_t n_tracks, int n_rows)
{
    return reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(ck) +
                                            ck_layout(n_tracks, n_rows).order_off);
}

static PackedHits ck_packed(const float* ck, int64_t n_tracks, int n_rows)
{
    const CkLayout L = ck_layout(n_tracks, n_rows);
    char* b = reinterpret_cast<char*>(const_cast<float*>(ck));
    return {reinterpret_cast<float2*>(b + L.yz_off), reinterpret_cast<uint8_t*>(b + L.row_off),
            reinterpret_cast<uint8_t*>(b + L.bad_off)};
}

// the tile order of the forward pass and the packed hits, into the
// checkpoint buffer
static void launch_order(const tpc_track_hits& hits, int n_rows, float* ck, hipStream_t st)
{
    const CkLayout L = ck_layout(hits.n_tracks, n_rows);
    char* b = reinterpret_cast<char*>(ck);
    int32_t* order = reinterpret_cast<int32_t*>(b + L.order_off);
    int32_t* cnt = reinterpret_cast<int32_t*>(b + L.cnt_off);
    int64_t* part = reinterpret_cast<int64_t*>(b + L.part_off);
    TPC_LAUNCH(k_order_count, dim3((unsigned)L.nblk), dim3(kOrdBlock), 0, st, hits.off,
               hits.d_count, hits.n_tracks, n_rows, cnt);
    launch_scan<int32_t>(cnt, cnt, L.nblk * L.nkeys, false, nullptr, part, st);
    TPC_LAUNCH(k_order_place, dim3((unsigned)L.nblk), dim3(kOrdBlock), 0, st, hits.off,
               hits.d_count, hits.n_tracks, n_rows, (const int32_t*)cnt, order);
    TPC_LAUNCH(k_refit_pack,
               dim3(grid_for_block(ceil_div(hits.n_tracks, kWave) * pack_parts(n_rows), 1, 65536)),
               dim3(kBlock), 0, st,
               (HitRows{hits.idx, hits.row, hits.y, hits.z, hits.off}), hits.d_count,
               hits.n_tracks, n_rows, (const int32_t*)order, ck_packed(ck, hits.n_tracks, n_rows));
}

// the adjoint and its theta reduction, partials[16 * refit_grid(n_tracks)]
static int launch_refit_adjoint(tpc_track_hits hits, int32_t n_rows, const float* d_row_x,
                                const tpc_params& prm, const tpc_calib_model& m,
                                const float* d_theta, const float* checkpoints,
                                const int32_t* status, const float* grad_chi2,
                                const float* seed_p, const float* seed_x, float* grad_y,
                                float* grad_z, float* grad_theta, double* partials,
                                hipStream_t st)
{
    const CalibModel cm = make_calib(m);
    const unsigned nb = refit_grid(hits.n_tracks);
    const PackedHits packed = ck_packed(checkpoints, hits.n_tracks, n_rows);
    const int32_t* order = ck_order(checkpoints, hits.n_tracks, n_rows);
    if (ck_stride(hits.n_tracks) == 2)
        TPC_LAUNCH(k_refit_adj<2>, dim3(nb), dim3(kWave), 0, st, hits.off, packed, hits.side,
                   hits.d_count, hits.n_tracks, n_rows, d_row_x, prm, cm, d_theta, checkpoints,
                   status, grad_chi2, seed_p, seed_x, grad_y, grad_z, partials, order);
    else
        TPC_LAUNCH(k_refit_adj<1>, dim3(nb), dim3(kWave), 0, st, hits.off, packed, hits.side,
                   hits.d_count, hits.n_tracks, n_rows, d_row_x, prm, cm, d_theta, checkpoints,
                   status, grad_chi2, seed_p, seed_x, grad_y, grad_z, partials, order);
    TPC_LAUNCH(k_reduce_theta, dim3(16), dim3(kBlock), 0, st, (const double*)partials, (int)nb,
               hits.d_count, hits.n_tracks, grad_theta);
    return hipGetLastError() == hipSuccess ? TPC_OK : TPC_ERR_HIP;
}

}  // namespace tpc

// Theta partials of the adjoint's blocks for callers that cannot allocate
// (tpc_refit_adjoint_noalloc): one copy per GPU, held until the process
// ends, shared by every call on that GPU (calls that overlap on one GPU
// race on it).  Every block of the adjoint writes its 16 partials before the
// reduction reads them, so nothing needs clearing between calls.
static __device__ __align__(256) double scratch[16 * tpc::kRefitMaxBlocks];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices];   // device address of `scratch` per GPU

}  // namespace

namespace tpc {

// Device address of this GPU's copy of `scratch`, taken once per device at
// context creation with that device current (the array's name is only a
// host-side stand-in and cannot be passed to a kernel).
int refit_scratch_setup(int device)
{
    if (device < 0 || device >= kMaxDevices) return TPC_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return TPC_OK;
    int prev = -1;
    if (hipGetDevice(&prev) != hipSuccess) return TPC_ERR_HIP;
    if (prev != device && hipSetDevice(device) != hipSuccess) return TPC_ERR_HIP;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (prev != device) (void)hipSetDevice(prev);
    if (e != hipSuccess || !ptr) return TPC_ERR_HIP;
    g_scratch_ptr[device] = static_cast<double*>(ptr);
    return TPC_OK;
}

}  // namespace tpc

extern "C" {

int tpc_refit_workspace_size(int64_t n_tracks, size_t* h_bytes)
{
    if (!h_bytes || n_tracks < 0) return TPC_ERR_INVALID_ARG;
    *h_bytes = sizeof(double) * 16 * (size_t)tpc::refit_grid(n_tracks);
    return TPC_OK;
}

int tpc_refit_checkpoint_size(int64_t n_tracks, int32_t n_rows, size_t* h_bytes)
{
    if (!h_bytes || n_tracks < 0 || n_rows < 3 || n_rows > 255) return TPC_ERR_INVALID_ARG;
    *h_bytes = tpc::ck_layout(n_tracks, n_rows).total;
    return TPC_OK;
}

int tpc_refit(tpc_context* ctx, tpc_track_hits hits, int32_t n_rows, const float* d_row_x,
              const tpc_params* h_params, const tpc_calib_model* h_model, const float* d_theta,
              float* par, float* cov, float* chi2, int32_t* status, float* checkpoints,
              size_t ck_bytes, void* stream)
{
    tpc::TimerScope timing(ctx ? ctx->timer : nullptr);
    if (!ctx || !h_params || !h_model || !d_theta || !d_row_x || !par || !cov || !chi2 ||
        !status || hits.n_tracks < 0 || hits.n_hits < 0 || n_rows < 3 || n_rows > 255 ||
        (hits.n_tracks > 0 && (!hits.off || !hits.row || !hits.y || !hits.z)) ||
        hits.n_hits >= (int64_t(1) << 31) || hits.n_tracks >= (int64_t(1) << 31))
        return TPC_ERR_INVALID_ARG;
    size_t ck_need = 0;
    if (checkpoints && (tpc_refit_checkpoint_size(hits.n_tracks, n_rows, &ck_need) ||
                        ck_bytes < ck_need))
        return TPC_ERR_INVALID_ARG;
    if (hits.n_tracks == 0) return TPC_OK;
    const tpc::CalibModel cm = tpc::make_calib(*h_model);
    hipStream_t st = (hipStream_t)stream;
    if (checkpoints) tpc::launch_order(hits, n_rows, checkpoints, st);
    const tpc::HitRows in{hits.idx, hits.row, hits.y, hits.z, hits.off};
    const dim3 g(tpc::refit_grid(hits.n_tracks));
    if (checkpoints)
        TPC_LAUNCH(tpc::k_refit_fwd<tpc::kPacked>, g, dim3(tpc::kWave), 0, st, in,
                   tpc::ck_packed(checkpoints, hits.n_tracks, n_rows), hits.side, hits.d_count,
                   hits.n_tracks, n_rows, d_row_x, *h_params, cm, d_theta, par, cov, chi2, status,
                   checkpoints, tpc::ck_stride(hits.n_tracks),
                   tpc::ck_order(checkpoints, hits.n_tracks, n_rows));
    else if (hits.idx)
        TPC_LAUNCH(tpc::k_refit_fwd<tpc::kCsrIndex>, g, dim3(tpc::kWave), 0, st, in,
                   tpc::PackedHits{}, hits.side, hits.d_count, hits.n_tracks, n_rows, d_row_x,
                   *h_params, cm, d_theta, par, cov, chi2, status, checkpoints, 1,
                   (const int32_t*)nullptr);
    else
        TPC_LAUNCH(tpc::k_refit_fwd<tpc::kCsr>, g, dim3(tpc::kWave), 0, st, in,
                   tpc::PackedHits{}, hits.side, hits.d_count, hits.n_tracks, n_rows, d_row_x,
                   *h_params, cm, d_theta, par, cov, chi2, status, checkpoints, 1,
                   (const int32_t*)nullptr);
    return hipGetLastError() == hipSuccess ? TPC_OK : TPC_ERR_HIP;
}

int tpc_refit_adjoint(tpc_context* ctx, tpc_track_hits hits, int32_t n_rows,
                      const float* d_row_x, const tpc_params* h_params,
                      const tpc_calib_model* h_model, const float* d_theta,
                      const float* checkpoints, size_t ck_bytes, const int32_t* status,
                      const float* grad_chi2,
                      float* grad_y, float* grad_z, float* grad_theta, void* d_ws,
                      size_t ws_bytes, void* stream)
{
    tpc::TimerScope timing(ctx ? ctx->timer : nullptr);
    size_t need = 0;
    if (!ctx || !h_params || !h_model || !d_theta || !d_row_x || !checkpoints || !status ||
        !grad_chi2 || !grad_y || !grad_z || !grad_theta || !d_ws || hits.n_tracks < 0 ||
        n_rows < 3 || n_rows > 255 ||
        (hits.n_tracks > 0 && (!hits.off || !hits.row || !hits.y || !hits.z)) ||
        tpc_refit_workspace_size(hits.n_tracks, &need) || need > ws_bytes ||
        tpc_refit_checkpoint_size(hits.n_tracks, n_rows, &need) || need > ck_bytes)
        return TPC_ERR_INVALID_ARG;
    return tpc::launch_refit_adjoint(hits, n_rows, d_row_x, *h_params, *h_model, d_theta,
                                     checkpoints, status, grad_chi2, nullptr, nullptr, grad_y,
                                     grad_z, grad_theta, (double*)d_ws, (hipStream_t)stream);
}

int tpc_refit_adjoint_seeded(tpc_context* ctx, tpc_track_hits hits, int32_t n_rows,
                             const float* d_row_x, const tpc_params* h_params,
                             const tpc_calib_model* h_model, const float* d_theta,
                             const float* checkpoints, size_t ck_bytes, const int32_t* status,
                             const float* grad_chi2, const float* grad_par, const float* grad_x,
                             float* grad_y, float* grad_z, float* grad_theta, void* d_ws,
                             size_t ws_bytes, void* stream)
{
    tpc::TimerScope timing(ctx ? ctx->timer : nullptr);
    size_t need = 0;
    if (!ctx || !h_params || !h_model || !d_theta || !d_row_x || !checkpoints || !status ||
        !grad_chi2 || !grad_y || !grad_z || !grad_theta || !d_ws || hits.n_tracks < 0 ||
        n_rows < 3 || n_rows > 255 ||
        (hits.n_tracks > 0 && (!hits.off || !hits.row || !hits.y || !hits.z)) ||
        tpc_refit_workspace_size(hits.n_tracks, &need) || need > ws_bytes ||
        tpc_refit_checkpoint_size(hits.n_tracks, n_rows, &need) || need > ck_bytes)
        return TPC_ERR_INVALID_ARG;
    return tpc::launch_refit_adjoint(hits, n_rows, d_row_x, *h_params, *h_model, d_theta,
                                     checkpoints, status, grad_chi2, grad_par, grad_x, grad_y,
                                     grad_z, grad_theta, (double*)d_ws, (hipStream_t)stream);
}

int tpc_vertex_residual(tpc_context* ctx, tpc_track_hits hits, int32_t n_rows,
                        const float* d_row_x, const tpc_params* h_params,
                        const tpc_calib_model* h_model, const float* d_theta, const float* par,
                        const float* cov, const int32_t* status, float sigma_v,
                        const float* w_in, float* w_out, float* loss, float* grad_par,
                        float* grad_x, int8_t* ok, void* stream)
{
    tpc::TimerScope timing(ctx ? ctx->timer : nullptr);
    if (!ctx || !h_params || !h_model || !d_theta || !d_row_x || !par || !cov || !status ||
        !loss || !grad_par || !grad_x || hits.n_tracks < 0 || n_rows < 3 || n_rows > 255 ||
        (hits.n_tracks > 0 && (!hits.off || !hits.row || !hits.y || !hits.z)) ||
        !(sigma_v >= 0.0f) || !std::isfinite(sigma_v))
        return TPC_ERR_INVALID_ARG;
    if (hits.n_tracks == 0) return TPC_OK;
    const tpc::CalibModel cm = tpc::make_calib(*h_model);
    TPC_LAUNCH(tpc::k_vertex_residual, dim3(tpc::grid_for(hits.n_tracks)), dim3(tpc::kBlock), 0,
               (hipStream_t)stream, hits.off, hits.idx, hits.row, hits.y, hits.z, hits.side,
               hits.d_count, hits.n_tracks, d_row_x, *h_params, cm, d_theta, par, cov, status,
               sigma_v * sigma_v, w_in, w_out, loss, grad_par, grad_x, ok);
    return hipGetLastError() == hipSuccess ? TPC_OK : TPC_ERR_HIP;
}

int tpc_refit_adjoint_noalloc(tpc_context* ctx, tpc_track_hits hits, int32_t n_rows,
                              const float* d_row_x, const tpc_params* h_params,
                              const tpc_calib_model* h_model, const float* d_theta,
                              const float* checkpoints, size_t ck_bytes, const int32_t* status,
                              const float* grad_chi2, float* grad_y, float* grad_z,
                              float* grad_theta, void* stream)
{
    tpc::TimerScope timing(ctx ? ctx->timer : nullptr);
    size_t need = 0;
    if (!ctx || !h_params || !h_model || !d_theta || !d_row_x || !checkpoints || !status ||
        !grad_chi2 || !grad_y || !grad_z || !grad_theta || hits.n_tracks < 0 ||
        n_rows < 3 || n_rows > 255 ||
        (hits.n_tracks > 0 && (!hits.off || !hits.row || !hits.y || !hits.z)) ||
        tpc_refit_checkpoint_size(hits.n_tracks, n_rows, &need) || need > ck_bytes)
        return TPC_ERR_INVALID_ARG;
    if (tpc::refit_grid(hits.n_tracks) > tpc::kRefitMaxBlocks) return TPC_ERR_CAPACITY;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return TPC_ERR_HIP;
    if (dev != ctx->device || dev < 0 || dev >= kMaxDevices) return TPC_ERR_INVALID_ARG;
    double* partials = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        partials = g_scratch_ptr[dev];
    }
    if (!partials) return TPC_ERR_HIP;   // set up when the context was created
    return tpc::launch_refit_adjoint(hits, n_rows, d_row_x, *h_params, *h_model, d_theta,
                                     checkpoints, status, grad_chi2, nullptr, nullptr, grad_y,
                                     grad_z, grad_theta, partials, (hipStream_t)stream);
}

}  // extern "C"
