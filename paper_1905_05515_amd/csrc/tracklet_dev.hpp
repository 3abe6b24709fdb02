// Kalman-filter tracklet construction of one chain start (device code shared
// by the staged kernel and the persistent kernel).
//
// State at the sector-local plane x: (y, z, s = sin(phi), t = tan(lambda),
// w = q/pT), covariance as the lower triangle of the symmetric 5x5 matrix
// (i*(i+1)/2 + j).  In a uniform field along z the curvature k = curv * w is
// constant: s grows linearly with x, the y step is dx (s1 + s2)/(c1 + c2)
// with c = sqrt(1 - s^2), and the arc length over the step is
// chord * asin(a)/a, a = k chord / 2, expanded to a^6.  Every expression
// below keeps the association order of its comment's formula, and sums of
// products are written as explicit fused multiply-adds (fmaf, one
// rounding); with contraction off otherwise and IEEE division and square
// root the results are the same bits on any conforming implementation.
#pragma once
#include "exact_fp32.hpp"
#include "tpc_internal.hpp"

namespace tpc {

__device__ __forceinline__ int lt(int i, int j) { return i >= j ? i * (i + 1) / 2 + j : j * (j + 1) / 2 + i; }

struct KState {
    float p[5];
    float C[15];
};

// Transport from plane x1 to x1 + dx.  Returns false (state untouched) when
// |sin(phi)| at either end of the step is not below s_max: at the far end
// the track turns back before the plane, at the near end an update has
// pushed the state out of the transport's domain (|s| >= 1 has no cosine).
__device__ __forceinline__ bool can_propagate(const KState& st, float dx, float curv, float s_max)
{
    const float s = st.p[2];
    const float s2 = fmaf(curv * st.p[4], dx, s);
    return fabsf(s) < s_max && fabsf(s2) < s_max;
}

// the transport where it is possible
__device__ __forceinline__ void transport(KState& st, float dx, float curv, float s_max)
{
    const float s = st.p[2], t = st.p[3], w = st.p[4];
    const float k = curv * w;
    const float s2 = fmaf(k, dx, s);
    const float u1 = (1.0f - s) * (1.0f + s), u2 = (1.0f - s2) * (1.0f + s2);
    // one reciprocal of cc = c1 + c2 for the three quotients by it
    float icc, T, q, e1, e2, Tq;   // e1 = s / c1, e2 = s2 / c2, Tq = T / q
    if (s_max <= 1.0f) {
        // |s| < 1 keeps every operand where the short sequences are the
        // correctly rounded operations (u >= 2^-24; a quotient e too small
        // for them vanishes beside the 1 or 2 it is added to, and T / q = T
        // there, q being 1)
        const float c1 = sqrt_exact(u1), c2 = sqrt_exact(u2);
        icc = rcp_exact(c1 + c2);
        e1 = div_exact(s, c1, rcp_exact(c1));
        e2 = div_exact(s2, c2, rcp_exact(c2));
        T = (s + s2) * icc;
        q = sqrt_exact(fmaf(T, T, 1.0f));
        Tq = copysignf(div_exact(T, q, rcp_exact(q)), T);
    } else {
        const float c1 = sqrtf(u1), c2 = sqrtf(u2);
        icc = 1.0f / (c1 + c2);
        e1 = s / c1;
        e2 = s2 / c2;
        T = (s + s2) * icc;
        q = sqrtf(fmaf(T, T, 1.0f));
        Tq = T / q;
    }
    const float L = dx * q;
    const float a = 0.5f * (k * L);
    const float a2 = a * a;
    const float g = fmaf(a2, fmaf(a2, fmaf(a2, 5.0f / 112.0f, 3.0f / 40.0f), 1.0f / 6.0f), 1.0f);
    const float S = L * g;
    const float Ts = fmaf(T, e1 + e2, 2.0f) * icc;
    const float kdx = curv * dx;
    const float Tw = (kdx * fmaf(T, e2, 1.0f)) * icc;
    const float LT = dx * Tq;
    const float G1 = fmaf(a2, fmaf(a2, fmaf(a2, 5.0f / 16.0f, 3.0f / 8.0f), 0.5f), 1.0f);
    const float Sk = (L * (L * a)) * fmaf(a2, fmaf(a2, 15.0f / 112.0f, 3.0f / 20.0f), 1.0f / 6.0f);
    const float Fys = dx * Ts;
    const float Fyw = dx * Tw;
    const float Fzs = t * ((G1 * LT) * Ts);
    const float Fzt = S;
    const float Fzw = t * fmaf(Sk, curv, (G1 * LT) * Tw);
    const float Fsw = kdx;

    // B = F C, then C' = B F^T, sums over the non-zero entries of F in
    // increasing column order, each product added by a fused multiply-add
    float B[5][5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const float cy = st.C[lt(0, j)], cz = st.C[lt(1, j)], cs = st.C[lt(2, j)];
        const float ct = st.C[lt(3, j)], cw = st.C[lt(4, j)];
        B[0][j] = fmaf(Fyw, cw, fmaf(Fys, cs, cy));
        B[1][j] = fmaf(Fzw, cw, fmaf(Fzt, ct, fmaf(Fzs, cs, cz)));
        B[2][j] = fmaf(Fsw, cw, cs);
        B[3][j] = ct;
        B[4][j] = cw;
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        st.C[lt(i, 0)] = fmaf(Fyw, B[i][4], fmaf(Fys, B[i][2], B[i][0]));
        if (i >= 1) st.C[lt(i, 1)] = fmaf(Fzw, B[i][4], fmaf(Fzt, B[i][3], fmaf(Fzs, B[i][2], B[i][1])));
        if (i >= 2) st.C[lt(i, 2)] = fmaf(Fsw, B[i][4], B[i][2]);
        if (i >= 3) st.C[lt(i, 3)] = B[i][3];
        if (i >= 4) st.C[lt(i, 4)] = B[i][4];
    }
    st.p[0] = fmaf(dx, T, st.p[0]);
    st.p[1] = fmaf(t, S, st.p[1]);
    st.p[2] = s2;
}

__device__ __forceinline__ bool propagate(KState& st, float dx, float curv, float s_max)
{
    const bool ok = can_propagate(st, dx, curv, s_max);
    if (ok) transport(st, dx, curv, s_max);
    return ok;
}

// Inverse covariance of the predicted measurement, B = S^-1 with
// S = C_yz + diag(sy2, sz2): one per row step, for every candidate's chi2
// and for the update.
struct Gain {
    float B00, B10, B11;
};

__device__ __forceinline__ Gain gain_of(const KState& st, float sy2, float sz2)
{
    const float S00 = st.C[0] + sy2, S10 = st.C[1], S11 = st.C[2] + sz2;
    const float det = fmaf(S00, S11, -(S10 * S10));
    const float idet = rcp_any(det);
    return {S11 * idet, -(S10 * idet), S00 * idet};
}

__device__ __forceinline__ float chi2_pred(const KState& st, const Gain& g, float my, float mz)
{
    const float r0 = my - st.p[0], r1 = mz - st.p[1];
    return fmaf(r1, fmaf(g.B11, r1, g.B10 * r0), r0 * fmaf(g.B10, r1, g.B00 * r0));
}

__device__ __forceinline__ float kupdate(KState& st, const Gain& g, float my, float mz)
{
    const float r0 = my - st.p[0], r1 = mz - st.p[1];
    const float B00 = g.B00, B10 = g.B10, B11 = g.B11;
    const float chi2 = fmaf(r1, fmaf(B11, r1, B10 * r0), r0 * fmaf(B10, r1, B00 * r0));
    float A0[5], A1[5], K0[5], K1[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        A0[i] = st.C[lt(i, 0)];
        A1[i] = st.C[lt(i, 1)];
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        K0[i] = fmaf(A1[i], B10, A0[i] * B00);
        K1[i] = fmaf(A1[i], B11, A0[i] * B10);
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        st.p[i] = st.p[i] + fmaf(K1[i], r1, K0[i] * r0);
#pragma unroll
        for (int j = 0; j <= i; ++j)
            st.C[lt(i, j)] = st.C[lt(i, j)] - fmaf(K1[i], A1[j], K0[i] * A0[j]);
    }
    return chi2;
}

__device__ __forceinline__ float kupdate(KState& st, float my, float mz, float sy2, float sz2)
{
    return kupdate(st, gain_of(st, sy2, sz2), my, mz);
}

__device__ __forceinline__ void reset_cov(KState& st, const tpc_params& prm)
{
#pragma unroll
    for (int i = 0; i < 15; ++i) st.C[i] = 0.0f;
    st.C[0] = prm.sigma_y2;
    st.C[2] = prm.sigma_z2;
    st.C[5] = prm.c_ss0;
    st.C[9] = prm.c_tt0;
    st.C[14] = prm.c_ww0;
}

constexpr int kCandBatch = 4;   // candidate loads issued together

// Hit of least predicted chi2 <= chi2_max on row r of sector s, ties to the
// lower cluster id; -1 if none, else its grid position with its coordinates
// in (my, mz).  The bins scanned cover +-nsigma of the prediction (every hit
// passing the gate lies inside); the gate decides.  Two z rows of bins are
// opened at a time so that their bin bounds load together.
__device__ __forceinline__ int search_row(const KState& st, const Gain& G, const tpc_sector& s, int r,
                                          const tpc_params& prm, int& n_cand,
                                          const int32_t* __restrict__ bin_start,
                                          const float* __restrict__ yg,
                                          const float* __restrict__ zg,
                                          const int32_t* __restrict__ idg, float& my, float& mz)
{
    // The window only has to contain every hit the gate can accept: the
    // hardware square root (within 1 ulp) is far inside the 1/64 widening,
    // so it needs none of the correctly rounded sequence the decisions use.
    const float S00 = st.C[0] + prm.sigma_y2, S11 = st.C[2] + prm.sigma_z2;
    const float hy = prm.search_nsigma * __builtin_amdgcn_sqrtf(S00) * TPC_WIDEN + 0.01f;
    const float hz = prm.search_nsigma * __builtin_amdgcn_sqrtf(S11) * TPC_WIDEN + 0.01f;
    const int iy0 = bin_of(st.p[0] - hy, s.y0, s.inv_by, s.nby);
    const int iy1 = bin_of(st.p[0] + hy, s.y0, s.inv_by, s.nby);
    const int iz0 = bin_of(st.p[1] - hz, s.z0, s.inv_bz, s.nbz);
    const int iz1 = bin_of(st.p[1] + hz, s.z0, s.inv_bz, s.nbz);
    float best = 0.0f;
    int bpos = -1;
    for (int iz = iz0; iz <= iz1; iz += 2) {
        const int g = s.bin_base + (r * s.nbz + iz) * s.nby;
        int lo[2], hi[2];
        lo[0] = bin_start[g + iy0];
        hi[0] = bin_start[g + iy1 + 1];
        lo[1] = hi[1] = 0;
        if (iz + 1 <= iz1) {
            lo[1] = bin_start[g + s.nby + iy0];
            hi[1] = bin_start[g + s.nby + iy1 + 1];
        }
        // the candidates of both z rows as one stream (row iz first, each in
        // grid order: the order of evaluation decides nothing but ties,
        // which go to the lower id anyway), loaded kCandBatch at a time so
        // that one memory round trip serves several candidates
        const int n0 = hi[0] - lo[0] > 0 ? hi[0] - lo[0] : 0;
        const int n1 = hi[1] - lo[1] > 0 ? hi[1] - lo[1] : 0;
        n_cand += n0 + n1;
        for (int b = 0; b < n0 + n1; b += kCandBatch) {
            float yb[kCandBatch], zb[kCandBatch];
            int pb[kCandBatch];
#pragma unroll
            for (int j = 0; j < kCandBatch; ++j) {
                const int e = b + j;
                pb[j] = e < n0 ? lo[0] + e : lo[1] + (e - n0);
                if (e < n0 + n1) {
                    yb[j] = yg[pb[j]];
                    zb[j] = zg[pb[j]];
                }
            }
#pragma unroll
            for (int j = 0; j < kCandBatch; ++j) {
                if (b + j >= n0 + n1) break;
                const float c2 = chi2_pred(st, G, yb[j], zb[j]);
                if (!(c2 <= prm.chi2_max)) continue;
                // equal chi2 (rare): the lower cluster id wins
                if (bpos < 0 || c2 < best || (c2 == best && idg[pb[j]] < idg[bpos])) {
                    best = c2;
                    bpos = pb[j];
                    my = yb[j];
                    mz = zb[j];
                }
            }
        }
    }
    return bpos;
}

__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const int w = __shfl_xor(v, o, kWave);
        v = w < v ? w : v;
    }
    return v;
}

// LDS of one wave of build_tracklets: the state after the last update of
// every lane's inward pass, five float4 per lane.  (Kept in registers it
// cost a copy of 20 registers per row, and as many again where the branches
// of a row meet.)
constexpr int kKeepVec = 5 * kWave;

__device__ __forceinline__ void keep_state(float4* keep, const KState& st)
{
    keep[0 * kWave] = make_float4(st.p[0], st.p[1], st.p[2], st.p[3]);
    keep[1 * kWave] = make_float4(st.p[4], st.C[0], st.C[1], st.C[2]);
    keep[2 * kWave] = make_float4(st.C[3], st.C[4], st.C[5], st.C[6]);
    keep[3 * kWave] = make_float4(st.C[7], st.C[8], st.C[9], st.C[10]);
    keep[4 * kWave] = make_float4(st.C[11], st.C[12], st.C[13], st.C[14]);
}

// Build the tracklets of one wave, one in each lane with `act` (every lane
// of the wave calls): tracklet ord[q], or q where there is no order.  xs
// holds the row positions; the hit list (grid position per row, -1 where
// none) is column q of t_hits[row][cap]; keep: the lane's slot of kKeepVec
// float4 in LDS.
//
// Up pass: from the start hit, one row at a time, the next hit is the next
// link of the chain while there is one (links always join adjacent rows),
// then the least-chi2 hit of a window search.  Down pass: from the outermost
// hit with the initial covariance, the hits already assigned are refitted and
// rows below the start are searched.  The loads of the next chain hit (up
// pass) are issued one row ahead; in the down pass the hit list entry of row
// r - 2 loads during row r and the coordinates of the hit of row r - 1
// during row r, so that no step waits on a load it issued itself.
//
// The wave walks the rows in step: a lane joins the up pass at the row above
// its start and the down pass at its outermost hit.  Some lane's tracklet
// nearly always spans the sector, so this adds few rows to the walk, and all
// lanes then read the bins and hits of one row (a few dozen lines of L1)
// and write one row of the hit lists as one line, where lanes each at their
// own row read their own lines and wrote single words.
__device__ __forceinline__ void build_tracklets(
    uint32_t q, const int32_t* __restrict__ ord, bool act, const tpc_sector* __restrict__ sec,
    int n_rows, const float* xs,
    const tpc_params& prm, const int32_t* __restrict__ bin_start, const float* __restrict__ yg,
    const float* __restrict__ zg, const int32_t* __restrict__ idg,
    const int32_t* __restrict__ gsr, const int32_t* __restrict__ up,
    const int32_t* __restrict__ starts, int32_t* t_hits, int64_t cap, float4* keep,
    int32_t* __restrict__ t_start, int32_t* __restrict__ t_nhits, int32_t* __restrict__ t_rin,
    float* __restrict__ t_par, float* __restrict__ t_cov, float* __restrict__ t_chi2,
    int& n_prop, int& n_upd, int& n_cand)   // of the wave; of the wave; of the lane
{
    const float sy2 = prm.sigma_y2, sz2 = prm.sigma_z2;
    // a tracklet has three clusters of its own: q < 2^31 / 3, a 32-bit byte
    // offset from the row's (uniform) base
    const uint32_t tb = q * 4u;
    auto hit_at = [&](int r) -> int32_t& {
        return *reinterpret_cast<int32_t*>(reinterpret_cast<char*>(t_hits + r * cap) + tb);
    };
    tpc_sector s{};
    KState st{};
    int r0 = n_rows;                      // a lane without a tracklet never joins
    int cc = -1, cn = -1;                 // chain hit of the coming row, of the one after
    float cy = 0.0f, cz = 0.0f;
    if (act) {
        const uint32_t t = ord ? (uint32_t)ord[q] : q;
        const int h0 = starts[t];
        const int v0 = gsr[h0];
        s = sec[v0 >> 8];
        r0 = v0 & 255;
        cc = up[h0];
        cn = up[cc];
        // state from the first and third chain hits
        const float dX = xs[gsr[cn] & 255] - xs[r0];
        const float T0 = (yg[cn] - yg[h0]) / dX;
        const float q0 = sqrtf(1.0f + T0 * T0);
        st.p[0] = yg[h0];
        st.p[1] = zg[h0];
        st.p[2] = T0 / q0;
        st.p[3] = (zg[cn] - zg[h0]) / (dX * q0);
        st.p[4] = 0.0f;
        reset_cov(st, prm);
        cy = yg[cc];
        cz = zg[cc];
        t_start[t] = h0;
        hit_at(r0) = h0;
    }
    // the up pass keeps the direction and q/pT at the outermost hit
    *keep = make_float4(st.p[2], st.p[3], st.p[4], 0.0f);

    // ---- up pass
    const int r_lo = wave_min(r0);
    int r = 0;
    for (; r <= r_lo && r < n_rows; ++r)
        if (act && r != r0) hit_at(r) = -1;
    int last = r0, miss = 0, nh = 1;
    bool go = act;
    for (; r < n_rows && __any(go); ++r) {
        const float dx = xs[r] - xs[r - 1];
        int hv = -1;
        bool upd = false;
        const bool step = go && r > r0;
        n_prop += __popcll(__ballot(step));
        if (step) {
            const bool chain = cc >= 0;
            float ny = 0.0f, nz = 0.0f;
            int cnn = -1;
            if (cn >= 0) {
                ny = yg[cn];
                nz = zg[cn];
                cnn = up[cn];
            }
            go = can_propagate(st, dx, prm.curv, prm.s_max);
            if (go) {
                transport(st, dx, prm.curv, prm.s_max);
                const Gain G = gain_of(st, sy2, sz2);
                int c = cc;
                float my = cy, mz = cz;
                if (!chain)
                    c = search_row(st, G, s, r, prm, n_cand, bin_start, yg, zg, idg, my, mz);
                if (c >= 0) {
                    kupdate(st, G, my, mz);
                    *keep = make_float4(st.p[2], st.p[3], st.p[4], 0.0f);
                    upd = true;
                    last = r;
                    ++nh;
                    miss = 0;
                } else {
                    go = ++miss < prm.max_miss;
                }
                hv = c;
                if (chain) {
                    cc = cn;
                    cy = ny;
                    cz = nz;
                    cn = cnn;
                }
            }
        }
        n_upd += __popcll(__ballot(upd));
        if (act && r != r0) hit_at(r) = hv;
    }
    for (; r < n_rows; ++r)
        if (act) hit_at(r) = -1;

    // ---- down pass
    r = -wave_min(act ? -last : 1);
    float csum = 0.0f;
    int rin = last;
    bool fit = false;                     // joined, and neither failed nor ended
    // assigned hits of this row and the next one down
    int e1 = r >= r0 ? hit_at(r) : -1, e2 = r - 1 >= r0 ? hit_at(r - 1) : -1;
    float ay = 0.0f, az = 0.0f;
    if (e1 >= 0) {
        ay = yg[e1];
        az = zg[e1];
    }
    miss = 0;
    go = act;
    for (; r >= 0 && __any(go); --r) {
        const int e0 = e1;
        float my = ay, mz = az;
        e1 = e2;
        if (e1 >= 0) {
            ay = yg[e1];
            az = zg[e1];
        }
        e2 = r - 2 >= r0 ? hit_at(r - 2) : -1;
        bool upd = false;
        n_prop += __popcll(__ballot(fit));
        if (fit) {
            const float dx = xs[r] - xs[r + 1];
            fit = can_propagate(st, dx, prm.curv, prm.s_max);
            if (fit) {
                transport(st, dx, prm.curv, prm.s_max);
                const Gain G = gain_of(st, sy2, sz2);
                int c = e0;
                if (r < r0)
                    c = search_row(st, G, s, r, prm, n_cand, bin_start, yg, zg, idg, my, mz);
                if (c >= 0) {
                    csum = csum + kupdate(st, G, my, mz);
                    keep_state(keep, st);
                    upd = true;
                    if (r < r0) {
                        hit_at(r) = c;
                        ++nh;
                    }
                    rin = r;
                    miss = 0;
                } else if (r < r0) {
                    fit = go = ++miss < prm.max_miss;
                }
            }
        }
        if (r == last) {                  // never of a lane without a tracklet: last = n_rows
            st.p[0] = my;
            st.p[1] = mz;
            const float4 d = *keep;
            st.p[2] = d.x;
            st.p[3] = d.y;
            st.p[4] = d.z;
            reset_cov(st, prm);
            keep_state(keep, st);
            fit = true;
        }
        // a propagation stop drops the assigned hits from here down
        if (go && !fit && r < last) {
            if (e0 >= 0) {
                hit_at(r) = -1;
                --nh;
            }
            go = r > r0;
        }
        n_upd += __popcll(__ballot(upd));
    }
    if (!act) return;
    const uint32_t t = ord ? (uint32_t)ord[q] : q;
    t_nhits[t] = nh;
    t_rin[t] = rin;
    float v[20];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const float4 k = keep[i * kWave];
        v[4 * i] = k.x;
        v[4 * i + 1] = k.y;
        v[4 * i + 2] = k.z;
        v[4 * i + 3] = k.w;
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) t_par[(int64_t)t * 5 + i] = v[i];
#pragma unroll
    for (int i = 0; i < 15; ++i) t_cov[(int64_t)t * 15 + i] = v[5 + i];
    t_chi2[t] = csum;
}

// work counters of a wave into the status block: n_prop and n_upd of the
// wave, n_cand of every lane
__device__ __forceinline__ void add_work(tpc_status* status, int n_prop, int n_upd, int n_cand)
{
    unsigned long long c = n_cand;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0 && (n_prop | n_upd)) {
        atomicAdd((unsigned long long*)&status->n_propagations, (unsigned long long)n_prop);
        atomicAdd((unsigned long long*)&status->n_updates, (unsigned long long)n_upd);
        atomicAdd((unsigned long long*)&status->n_candidates, c);
    }
}

}  // namespace tpc
