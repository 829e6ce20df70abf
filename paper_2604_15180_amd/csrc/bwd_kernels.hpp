// Backward kernels (Sec. 3.3 "Backward pass", Alg. 2-3 of the AdaSplash-2 paper):
//   dq_kernel   : per 32*QB*NW query rows, over the set bits of their mask rows, in one sweep:
//                 delta_r = sum_j U_rj dP_rj / sum_j U_rj,  U = P^(2-alpha), dP = dO V^T
//                 dQ = [ (U o dP) K - delta (U K) ] / sqrt(d)  ( = dS K / sqrt(d), Alg. 3)
//   dkdv_kernel : per 32*QB*NW keys, over the set bits of their mask columns:
//                 dV += P^T dO,  dK += dS^T Q / sqrt(d)                               (Alg. 2)
// With y = (alpha-1) s - tau on the support:  P = y^r,  U = y^(r-1),  r = 1/(alpha-1).
#pragma once
#include "common.hpp"
#include "gather.hpp"

namespace ea {

// Two floats -> one register of two fp16 values (round to nearest even).
EA_DEV uint32_t pack_f16x2(float a, float b) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    h2 v;
    v[0] = (_Float16)a; v[1] = (_Float16)b;
    return __builtin_bit_cast(uint32_t, v);
}
// Second-stage operands in two fp16 halves.  A product whose B operand is rounded to fp16 carries a
// relative error of 2^-12 per element; summed over the hundreds or thousands of query rows that
// attend to one key (or over keys that share a large common component) those errors are what is left
// when the exact terms cancel, and they pass 1e-2 (1 + |gradient|).  So the operand is cut in two:
// hi = x with all but its 11 leading significant bits cleared (an fp16 value exactly), lo = x - hi
// (exact in fp32) rounded to fp16; hi + lo carries 21 bits of x, and the product is two MFMAs on the
// same A fragment.  SPLIT_NONE: one fp16 operand; SPLIT_SIGNED: the operands whose terms cancel
// (dS, U (dP - e)) are cut; SPLIT_ALL: P and U as well.
constexpr int SPLIT_NONE = 0, SPLIT_SIGNED = 1, SPLIT_ALL = 2;
#ifndef EA_BWD_SPLIT
#define EA_BWD_SPLIT SPLIT_ALL
#endif
EA_DEV float f16_head(float x) { return __uint_as_float(__float_as_uint(x) & 0xffffe000u); }
// packs of (hi, hi) and (lo, lo) of two floats
EA_DEV void pack_split(float a, float b, uint32_t& hi, uint32_t& lo) {
    const float ha = f16_head(a), hb = f16_head(b);
    hi = pack_f16x2(ha, hb);
    lo = pack_f16x2(a - ha, b - hb);
}
// x -> what fp16 rounding of x leaves behind (the plain tile bodies: stage2 rounds to nearest)
template <int QB> EA_DEV void f16_tail(f32x16 (&Y)[2][QB]) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int v = 0; v < 16; ++v) Y[kb][qb][v] -= (float)(_Float16)Y[kb][qb][v];
}
EA_DEV f16x8 frag_of(const uint32_t (&w)[8], int s2) {
    u32x4 v;
    v[0] = w[4 * s2]; v[1] = w[4 * s2 + 1]; v[2] = w[4 * s2 + 2]; v[3] = w[4 * s2 + 3];
    return __builtin_bit_cast(f16x8, v);
}

// One 64-key tile of the dQ sweep for a wave's 32 rows, 16-bit operands, every statement placed by
// hand.  A wave with 128 accumulator registers runs alone on its SIMD, so nothing but its own
// instruction order lets the vector ALUs work while the matrix pipe is busy.  The tile is cut into
// its two 32-key halves and the work on them is staggered:
//     stage 1, half 0                                    (matrix pipe only)
//     stage 1, half 1    with the score math of half 0   (one or two scores after every MFMA)
//     stage 2, half 0    with the score math of half 1
//     stage 2, half 1                                    (matrix pipe only)
// LDS reads run PF steps ahead of the MFMAs that use them.  An MFMA lasts 32 cycles and a vector
// instruction 4, so up to 7 vector instructions fit behind each MFMA at no cost.
template <class E, class E2, int D, int AM, int SPLIT>
EA_DEV void dq_tile_staggered(const char* kbuf, const char* vbuf, const Owned<E, D, 1>& qf, const Owned<E, D, 1>& gf,
                              f32x16 (&XA)[D / 32][1], f32x16 (&XB)[D / 32][1], float thr, float ctr, float c, float r,
                              float& num, float& den, const Frag1<E, D>& f1, const Frag2<E2, D>& f2) {
    constexpr int NS = D / 16, ND = D / 32;
    constexpr int N1 = 2 * NS;            // stage-1 steps (kb, s): two MFMAs each (scores, dP)
    constexpr int N2 = 4 * ND;            // stage-2 steps (kb, s2, db): two MFMAs each (XA, XB)
    constexpr int PF = 4;                 // steps the LDS reads run ahead
    constexpr int EPM = 8 / NS;           // scores handled after each MFMA of an overlapped phase
    static_assert(8 % NS == 0 && 4 % ND == 0 && EPM == 4 / ND, "halves must divide evenly over the MFMAs");
    using frag = typename E::frag;
    using frag2 = typename E2::frag;
    f32x16 S[2], P[2];
    uint32_t tp[2][8], up[2][8];          // t = u (dP - e) and u as fp16 pairs: the stage-2 B operands
    uint32_t tl[2][8], ul[2][8];          // their low halves (SPLIT)
    frag ak[N1], av[N1];
    frag2 at[N2];
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    auto score_math = [&](int kb, int e) {
        const float y = fmaf(c, S[kb][e], -thr);
        float u;
        if constexpr (AM == ALPHA_15) u = fmaxf(y, 0.f);
        else u = (y > 0.f) ? pow_r1<AM>(y, r) : 0.f;
        const float t = u * (P[kb][e] - ctr);
        num += t;
        den += u;
        S[kb][e] = t;
        P[kb][e] = u;
        if (e & 1) {
            if constexpr (SPLIT >= SPLIT_SIGNED) pack_split(S[kb][e - 1], S[kb][e], tp[kb][e >> 1], tl[kb][e >> 1]);
            else tp[kb][e >> 1] = pack_f16x2(S[kb][e - 1], S[kb][e]);
            if constexpr (SPLIT >= SPLIT_ALL) pack_split(P[kb][e - 1], P[kb][e], up[kb][e >> 1], ul[kb][e >> 1]);
            else up[kb][e >> 1] = pack_f16x2(P[kb][e - 1], P[kb][e]);
        }
    };
    auto read2 = [&](int i2) { at[i2] = f2(kbuf, i2 / (2 * ND), (i2 / ND) & 1, i2 % ND); };

#pragma unroll
    for (int i = 0; i < PF; ++i) { ak[i] = f1(kbuf, i / NS, i % NS); av[i] = f1(vbuf, i / NS, i % NS); }
    sched_fence();
#pragma unroll
    for (int i = 0; i < N1; ++i) {
        const int kb = i / NS, s = i % NS;
        if (i + PF < N1) { ak[i + PF] = f1(kbuf, (i + PF) / NS, (i + PF) % NS); av[i + PF] = f1(vbuf, (i + PF) / NS, (i + PF) % NS); }
        else read2(i + PF - N1);
        S[kb] = E::mma(ak[i], qf.f[0][s], s == 0 ? zero : S[kb]);
        sched_fence();
        if (kb == 1) {
#pragma unroll
            for (int k = 0; k < EPM; ++k) score_math(0, 2 * EPM * s + k);
        }
        sched_fence();
        P[kb] = E::mma(av[i], gf.f[0][s], s == 0 ? zero : P[kb]);
        sched_fence();
        if (kb == 1) {
#pragma unroll
            for (int k = 0; k < EPM; ++k) score_math(0, 2 * EPM * s + EPM + k);
        }
        sched_fence();
    }
#pragma unroll
    for (int i = 0; i < N2; ++i) {
        const int kb = i / (2 * ND), s2 = (i / ND) & 1, db = i % ND, j = i % (2 * ND);
        if (i + PF < N2) read2(i + PF);
        E2::template mma_acc<false>(at[i], frag_of(tp[kb], s2), XA[db][0]);
        sched_fence();
        if (kb == 0) {
#pragma unroll
            for (int k = 0; k < EPM; ++k) score_math(1, 2 * EPM * j + k);
        }
        sched_fence();
        E2::template mma_acc<false>(at[i], frag_of(up[kb], s2), XB[db][0]);
        sched_fence();
        if (kb == 0) {
#pragma unroll
            for (int k = 0; k < EPM; ++k) score_math(1, 2 * EPM * j + EPM + k);
        }
        sched_fence();
        if constexpr (SPLIT >= SPLIT_SIGNED) { E2::template mma_acc<false>(at[i], frag_of(tl[kb], s2), XA[db][0]); sched_fence(); }
        if constexpr (SPLIT >= SPLIT_ALL) { E2::template mma_acc<false>(at[i], frag_of(ul[kb], s2), XB[db][0]); sched_fence(); }
    }
}

template <class E, class E2, int D, int QB, int NW, int NBUF>
struct DqSmem {
    static constexpr int BR = 32 * QB * NW;
    static constexpr int MR = (BR + 63) / 64;
    static constexpr int RBYTES = RowTile<E, D>::BYTES;
    static constexpr int SET = 2 * RBYTES;                   // K, V tiles
};

template <class E, class E2, int D, int QB, int AM, int NW, int NBUF>
__global__ __launch_bounds__(NW * 64) void dq_kernel(Params p) {
    using SM = DqSmem<E, E2, D, QB, NW, NBUF>;
    using elem = typename E::elem;
    constexpr int BR = SM::BR, MR = SM::MR;
    constexpr int THREADS = NW * 64;
    // buffer sets (K tile, V tile) as separate variables (see stream_tiles); all LDS is static
    __shared__ __align__(1024) char set0[SM::SET];
    __shared__ __align__(1024) char set1[NBUF == 2 ? SM::SET : 1024];
    __shared__ uint32_t fm[MR * MAX_W];
    __shared__ int tl[MAX_T];
    __shared__ int tl_count[4];
    __shared__ unsigned long long blk_stats[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int N = p.N, T = p.T, W = p.W;
    int bh, I;
    map_block(blockIdx.x, p.BH, (N + BR - 1) / BR, bh, I);
    const long q0 = (long)I * BR, qw0 = q0 + wave * 32 * QB;
    const bool active = qw0 < N;
    // row groups whose supports were listed get dQ and delta from bwd_rows_kernel
    if (p.gflag && p.gflag[(long)bh * ((N + p.grows - 1) / p.grows) + q0 / p.grows]) return;
    const long hoff = (long)bh * N * D;
    const elem* Kh = (const elem*)p.K + hoff;
    const elem* Vh = (const elem*)p.V + hoff;
    const int myrow = (wave * 32 * QB) / 64;
    const HeadConsts hc = head_consts(p, bh);
    const float c = hc.c, r = hc.r;

    for (int i = tid; i < MR * W; i += THREADS)
        fm[i] = (I * MR + i / W < T) ? (uint32_t)p.mask[((long)bh * T + (long)I * MR + i / W) * W + (i % W)] : 0u;
    build_tile_list(fm, MR, W, tl, tl_count, tid);

    Owned<E, D, QB> qf, gf;
    load_owned<E, D, QB>(qf, (const elem*)p.Q + hoff, active ? qw0 : 0, lane);
    load_owned<E, D, QB>(gf, (const elem*)p.dO + hoff, active ? qw0 : 0, lane);
    float thr[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) thr[qb] = active ? p.tau[(long)bh * N + qw0 + 32 * qb + n] : 0.f;

    // One sweep over the set bits of the mask rows.  With dS = U (dP - delta) and any centre e:
    //     dQ sqrt(d) = sum_j dS_j K_j = sum_j (U (dP - e))_j K_j - (delta - e) sum_j U_j K_j
    //                = XA - (delta - e) XB,     delta - e = sum(U (dP - e)) / sum(U),
    // so delta comes out of the row sums of the same sweep and the scores are computed once.
    // The centre e = <dO_r, O_r> = sum_j P_rj dP_rj is the P-weighted mean of dP over the support
    // (delta is the U-weighted one): it keeps XA - (delta - e) XB free of the cancellation that
    // e = 0 would bring when dP is nearly constant over the support.  Without O, e = 0.
    // With a narrow-range stage-2 type the whole backward runs on dO / max|dO| (amax undoes it at
    // the end): then |dP_rj| = |<dO_r, V_j>| <= sqrt(d) |V_j| and |U (dP - e)| <= 2 sqrt(d) max|V_j|,
    // far inside fp16's range for any V that itself fits fp16 comfortably, and fp16 keeps 11
    // significant bits at any magnitude in its normal range, so no further scaling is needed.
    float amax = 1.f;
    if constexpr (E2::SCALED) {
        amax = __uint_as_float(p.scal[0]);
        if (!(amax > 0.f)) amax = 1.f;
    }
    float ctr[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        float acc = 0.f;
        if (p.O && active) {
            // lane half h takes half of the row; 16-byte loads, all in flight together
            const f32x4* orow = (const f32x4*)(p.O + hoff + (qw0 + 32 * qb + n) * (long)D + h * (D / 2));
            const elem* grow = (const elem*)p.dO + hoff + (qw0 + 32 * qb + n) * (long)D + h * (D / 2);
            f32x4 ov[D / 8];
#pragma unroll
            for (int e = 0; e < D / 8; ++e) ov[e] = orow[e];
            if constexpr (sizeof(elem) == 2) {
                typedef elem ex8 __attribute__((ext_vector_type(8)));
                ex8 gv[D / 16];
#pragma unroll
                for (int e = 0; e < D / 16; ++e) gv[e] = ((const ex8*)grow)[e];
#pragma unroll
                for (int e = 0; e < D / 2; ++e) acc = fmaf(ov[e / 4][e % 4], (float)gv[e / 8][e % 8], acc);
            } else {
#pragma unroll
                for (int e = 0; e < D / 2; ++e) acc = fmaf(ov[e / 4][e % 4], (float)grow[e], acc);
            }
        }
        ctr[qb] = xhalf_sum(acc);
    }

    f32x16 XA[D / 32][QB], XB[D / 32][QB];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int v = 0; v < 16; ++v) { XA[db][qb][v] = 0.f; XB[db][qb][v] = 0.f; }

    f32x16 S[2][QB], dP[2][QB];
    unsigned long long ntile = 0;
    const Frag1<E, D> frag1(lane);
    const Frag2<E2, D> frag2(lane);
    float num[QB], den[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) num[qb] = den[qb] = 0.f;
    auto issue_kv = [&](int it, char* b) {
        const long j = tl[it];
        issue_rows<E, D, NW>(b, Kh, j * 64, wave, lane);
        issue_rows<E, D, NW>(b + SM::RBYTES, Vh, j * 64, wave, lane);
    };
    // any tile, statements left to the compiler's order
    auto tile_plain_order = [&](int it, const char* kbuf) {
        const int j = tl[it];
        if (!mask_bit(fm, W, myrow, j)) return;
        const char* vbuf = kbuf + SM::RBYTES;
        ++ntile;
        stage1<E, D, QB>(S, kbuf, qf, lane);
        if (p.causal && (long)j * 64 + 63 > qw0) causal_hide<QB, true>(S, j * 64, (int)qw0, lane);
        stage1<E, D, QB>(dP, vbuf, gf, lane);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float y = fmaf(c, S[kb][qb][v], -thr[qb]);
                    float u;
                    if constexpr (AM == ALPHA_15) u = fmaxf(y, 0.f);
                    else u = (y > 0.f) ? pow_r1<AM>(y, r) : 0.f;
                    const float t = u * (dP[kb][qb][v] - ctr[qb]);
                    num[qb] += t;
                    den[qb] += u;
                    S[kb][qb][v] = t;
                    dP[kb][qb][v] = u;
                }
        stage2<E2, D, QB, true>(XA, kbuf, S, lane);
        stage2<E2, D, QB, true>(XB, kbuf, dP, lane);
        if constexpr (E2::EPL == 8 && EA_BWD_SPLIT >= SPLIT_SIGNED) { f16_tail<QB>(S); stage2<E2, D, QB, true>(XA, kbuf, S, lane); }
        if constexpr (E2::EPL == 8 && EA_BWD_SPLIT >= SPLIT_ALL) { f16_tail<QB>(dP); stage2<E2, D, QB, true>(XB, kbuf, dP, lane); }
    };
    if constexpr (E::EPL == 8 && QB == 1 && NBUF == 2) {
        // tiles wholly below the diagonal (the head of the ascending list) take the staggered body;
        // the one or two on it, and one more when that makes the head's length even, the plain one
        const int nt = *tl_count;
        int ndiag = 0;
        if (p.causal)
            while (ndiag < nt && (long)tl[nt - 1 - ndiag] * 64 + 63 > q0) ++ndiag;
        stream_tiles_split((nt - ndiag) & ~1, nt, set0, set1, issue_kv,
            [&](int it, const char* kbuf) {
                if (!mask_bit(fm, W, myrow, tl[it])) return;
                ++ntile;
                dq_tile_staggered<E, E2, D, AM, EA_BWD_SPLIT>(kbuf, kbuf + SM::RBYTES, qf, gf, XA, XB, thr[0], ctr[0], c, r, num[0], den[0], frag1, frag2);
            },
            tile_plain_order);
    } else {
        stream_tiles<NBUF>(*tl_count, set0, NBUF == 2 ? set1 : set0, issue_kv, tile_plain_order);
    }
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) { settle_acc(XA[db][qb]); settle_acc(XB[db][qb]); }

    // delta (in units of max|dO|) for the dK/dV kernel, and the combination of the two sums
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float dn = xhalf_sum(den[qb]);
        const float drel = dn > 0.f ? xhalf_sum(num[qb]) / dn : 0.f;      // delta - e
        if (h == 0 && active) {
            // for the dK/dV kernel, as the biases its two stage-1 products start from
            p.delta[(long)bh * N + qw0 + 32 * qb + n] = -(drel + ctr[qb]);
            p.ntau[(long)bh * N + qw0 + 32 * qb + n] = -thr[qb] / hc.rho;
        }
        const float sa = p.inv_sqrt_d * amax, sb = drel * p.inv_sqrt_d * amax;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) XA[db][qb][v] = sa * XA[db][qb][v] - sb * XB[db][qb][v];
    }
    if (active) store_owned_T<D, QB>(p.dQ + hoff, qw0, XA, 1.f, lane);
    {
        const int slot[1] = {3};
        const unsigned long long val[1] = {ntile * QB};
        flush_counters<1>(blk_stats, p.stats, slot, val, tid, lane);
    }
}

// One 64-query tile of the dK/dV walk for a wave's 32 keys, staggered like dq_tile_staggered:
// stage 1 = (Q tile . K_owned^T, dO tile . V_owned^T), score math, stage 2 = (dV^T += dO^T P,
// dK^T += Q^T dS).  The thresholds and deltas of the tile's 64 query rows vary along the
// accumulator registers, so they cost no arithmetic at all: the accumulators of the two stage-1
// products start from -tau / rho and -delta (read from LDS, four rows per 16-byte read) instead of
// zero.  With the owned keys scaled by kappa the first product is then y / rho, y = (alpha-1) s -
// tau, and the second dP - delta.  alpha 1.5 and 2: P = y^r and dS = y^(r-1) (dP - delta) come out in units of
// rho^r and rho^(r-1), which the kernel's epilogue multiplies back in.  General alpha: rho^(r-1) goes into the exponent
// of U = y^(r-1), and P is left in units of rho (at alpha = 1.03 rho^r can be 1e10: P over it is zero in fp16).
template <class E, class E2, int D, int AM, int SPLIT>
EA_DEV void dkdv_tile_staggered(const char* qbuf, const char* gbuf, const float* ntau_s, const float* ndel_s,
                                const Owned<E, D, 1>& kf, const Owned<E, D, 1>& vf, f32x16 (&XV)[D / 32][1],
                                f32x16 (&XK)[D / 32][1], float r, float lrho_u, int h, const Frag1<E, D>& f1,
                                const Frag2<E2, D>& f2) {
    constexpr int NS = D / 16, ND = D / 32;
    constexpr int N1 = 2 * NS, N2 = 4 * ND, PF = 4, EPM = 8 / NS;
    static_assert(8 % NS == 0 && 4 % ND == 0 && EPM == 4 / ND, "halves must divide evenly over the MFMAs");
    using frag = typename E::frag;
    using frag2 = typename E2::frag;
    f32x16 S[2], P[2];
    uint32_t pp[2][8], sp[2][8];          // P and dS as fp16 pairs: the stage-2 B operands
    uint32_t pl[2][8], sl[2][8];          // their low halves (SPLIT)
    frag aq[N1], ag[N1];
    frag2 tg[N2], tq[N2];

    // registers 4 g .. 4 g + 3 of half kb are four consecutive tile rows
    auto bias = [&](const float* vec, int kb) {
        f32x16 b;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 t = *(const f32x4*)(vec + trow(kb, 4 * g, h));
#pragma unroll
            for (int e = 0; e < 4; ++e) b[4 * g + e] = t[e];
        }
        return b;
    };
    auto score_math = [&](int kb, int e) {
        const float yp = fmaxf(S[kb][e], 0.f);
        float u;
        if constexpr (AM == ALPHA_15) u = yp;
        else if constexpr (AM == ALPHA_20) u = (yp > 0.f) ? 1.f : 0.f;
        else u = (yp > 0.f) ? pow_r1_rho(yp, r, lrho_u) : 0.f;
        S[kb][e] = u * yp;
        P[kb][e] = u * P[kb][e];
        if (e & 1) {
            if constexpr (SPLIT >= SPLIT_ALL) pack_split(S[kb][e - 1], S[kb][e], pp[kb][e >> 1], pl[kb][e >> 1]);
            else pp[kb][e >> 1] = pack_f16x2(S[kb][e - 1], S[kb][e]);
            if constexpr (SPLIT >= SPLIT_SIGNED) pack_split(P[kb][e - 1], P[kb][e], sp[kb][e >> 1], sl[kb][e >> 1]);
            else sp[kb][e >> 1] = pack_f16x2(P[kb][e - 1], P[kb][e]);
        }
    };
    auto read2 = [&](int i2) {
        tg[i2] = f2(gbuf, i2 / (2 * ND), (i2 / ND) & 1, i2 % ND);
        tq[i2] = f2(qbuf, i2 / (2 * ND), (i2 / ND) & 1, i2 % ND);
    };

#pragma unroll
    for (int i = 0; i < PF; ++i) { aq[i] = f1(qbuf, i / NS, i % NS); ag[i] = f1(gbuf, i / NS, i % NS); }
    S[0] = bias(ntau_s, 0); P[0] = bias(ndel_s, 0);
    sched_fence();
#pragma unroll
    for (int i = 0; i < N1; ++i) {
        const int kb = i / NS, s = i % NS;
        if (i + PF < N1) { aq[i + PF] = f1(qbuf, (i + PF) / NS, (i + PF) % NS); ag[i + PF] = f1(gbuf, (i + PF) / NS, (i + PF) % NS); }
        else read2(i + PF - N1);
        if (i == NS - 2) { S[1] = bias(ntau_s, 1); P[1] = bias(ndel_s, 1); }
        S[kb] = E::mma(aq[i], kf.f[0][s], S[kb]);
        sched_fence();
        if (kb == 1) {
#pragma unroll
            for (int k = 0; k < EPM; ++k) score_math(0, 2 * EPM * s + k);
        }
        sched_fence();
        P[kb] = E::mma(ag[i], vf.f[0][s], P[kb]);
        sched_fence();
        if (kb == 1) {
#pragma unroll
            for (int k = 0; k < EPM; ++k) score_math(0, 2 * EPM * s + EPM + k);
        }
        sched_fence();
    }
#pragma unroll
    for (int i = 0; i < N2; ++i) {
        const int kb = i / (2 * ND), s2 = (i / ND) & 1, db = i % ND, j = i % (2 * ND);
        if (i + PF < N2) read2(i + PF);
        E2::template mma_acc<false>(tg[i], frag_of(pp[kb], s2), XV[db][0]);
        sched_fence();
        if (kb == 0) {
#pragma unroll
            for (int k = 0; k < EPM; ++k) score_math(1, 2 * EPM * j + k);
        }
        sched_fence();
        E2::template mma_acc<false>(tq[i], frag_of(sp[kb], s2), XK[db][0]);
        sched_fence();
        if (kb == 0) {
#pragma unroll
            for (int k = 0; k < EPM; ++k) score_math(1, 2 * EPM * j + EPM + k);
        }
        sched_fence();
        if constexpr (SPLIT >= SPLIT_SIGNED) { E2::template mma_acc<false>(tq[i], frag_of(sl[kb], s2), XK[db][0]); sched_fence(); }
        if constexpr (SPLIT >= SPLIT_ALL) { E2::template mma_acc<false>(tg[i], frag_of(pl[kb], s2), XV[db][0]); sched_fence(); }
    }
}

// Which of the MC mask columns jc0.. hold query tile i of head bh (bit c: column jc0 + c); none for
// query tiles of row groups whose supports were listed (those are left to bwd_cols_kernel).
template <int MC>
EA_DEV int column_flags(const Params& p, int bh, int i, int jc0) {
    if (p.gflag && p.gflag[(long)bh * ((p.N + p.grows - 1) / p.grows) + (i * 64) / p.grows]) return 0;
    int flags = 0;
#pragma unroll
    for (int cidx = 0; cidx < MC; ++cidx) {
        const int j = jc0 + cidx;
        if (j >= p.T) continue;
        const uint32_t w = (uint32_t)p.mask[((long)bh * p.T + i) * p.W + (j >> 5)];
        flags |= (int)((w >> (j & 31)) & 1u) << cidx;
    }
    return flags;
}

// Length of every key block's mask column, for dkdv_kernel's launch in parts; a column of more than
// one part has its rows of dK, dV cleared here, since all its parts add to them.
template <int D, int BC>
__global__ __launch_bounds__(128) void col_count_kernel(Params p) {
    constexpr int MC = (BC + 63) / 64;
    __shared__ int total;
    const int tid = threadIdx.x;
    const int GC = (p.N + BC - 1) / BC;
    int bh, J;
    map_block(blockIdx.x, p.BH, GC, bh, J);
    if (p.gflag && *p.nplain == 0) return;
    if (tid == 0) total = 0;
    __syncthreads();
    const int jc0 = J * MC;
    int mine = 0;
    for (int i = (p.causal ? jc0 : 0) + tid; i < p.T; i += 128) mine += column_flags<MC>(p, bh, i, jc0) != 0;
    if (mine) atomicAdd(&total, mine);
    __syncthreads();
    const int cnt = total;
    if (tid == 0) p.colcnt[(long)bh * GC + J] = cnt;
    if (cnt > p.col_part_len) {
        const long k0 = (long)J * BC, nk = min((long)BC, p.N - k0);
        f32x4* const dk = (f32x4*)(p.dK + ((long)bh * p.N + k0) * D);
        f32x4* const dv = (f32x4*)(p.dV + ((long)bh * p.N + k0) * D);
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        for (long e = tid; e < nk * (D / 4); e += 128) { dk[e] = zero; dv[e] = zero; }
    }
}

template <class E, class E2, int D, int QB, int NW, int NBUF>
struct DkdvSmem {
    static constexpr int BC = 32 * QB * NW;
    static constexpr int MC = (BC + 63) / 64;
    static constexpr int RBYTES = RowTile<E, D>::BYTES;
    static constexpr int SET = 2 * RBYTES + 4 * 2 * TILE;    // Q, dO tiles, tau, delta
};

template <class E, class E2, int D, int QB, int AM, int NW, int NBUF>
__global__ __launch_bounds__(NW * 64) void dkdv_kernel(Params p) {
    using SM = DkdvSmem<E, E2, D, QB, NW, NBUF>;
    using elem = typename E::elem;
    constexpr int BC = SM::BC, MC = SM::MC;
    constexpr int THREADS = NW * 64;
    static_assert(NW >= 2, "tau and delta rows are fetched by waves 0 and 1");
    // buffer sets (Q tile, dO tile, tau[64], delta[64]) as separate variables (see stream_tiles)
    __shared__ __align__(1024) char set0[SM::SET];
    __shared__ __align__(1024) char set1[NBUF == 2 ? SM::SET : 1024];
    __shared__ int tl[MAX_T];                // entries: query tile | column flags << 16
    __shared__ int wcnt[16];                 // per-wave counts, [8] = running total
    __shared__ unsigned long long blk_stats[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int N = p.N, T = p.T, W = p.W;
    int bh, J;
    const int GC = (N + BC - 1) / BC, part = (int)blockIdx.x / (p.BH * GC);
    map_block((int)blockIdx.x % (p.BH * GC), p.BH, GC, bh, J);
    J = GC - 1 - J;                           // causal: the first key tiles have the longest columns
    // every row group went by gather: bwd_cols_kernel writes dK, dV itself
    if (p.gflag && *p.nplain == 0) return;
    // launched in parts (col_part_len > 0): a part past the column's end has nothing to do; all
    // parts of a column that has several add to rows that col_count_kernel cleared
    const bool shared_out = p.col_part_len > 0 && p.colcnt[(long)bh * GC + J] > p.col_part_len;
    if (part > 0 && p.colcnt[(long)bh * GC + J] <= part * p.col_part_len) return;
    const long k0 = (long)J * BC, kw0 = k0 + wave * 32 * QB;
    const bool active = kw0 < N;
    const long hoff = (long)bh * N * D;
    const elem* Qh = (const elem*)p.Q + hoff;
    const elem* Gh = (const elem*)p.dO + hoff;
    // dO is used divided by max|dO| throughout (see dq_kernel)
    float go_amax = 1.f;
    if constexpr (E2::SCALED) {
        go_amax = __uint_as_float(p.scal[0]);
        if (!(go_amax > 0.f)) go_amax = 1.f;
    }
    const int mycol = (wave * 32 * QB) / 64;  // my mask column within the group
    const int jc0 = J * MC;                   // first mask column of the group
    const HeadConsts hc = head_consts(p, bh);
    const float r = hc.r, lrho_u = hc.lrho_u;

    // ---- column walk of the row-packed mask: list of query tiles with a set bit -------------
    const int i_min = p.causal ? jc0 : 0;
    if (tid == 0) wcnt[8] = 0;
    __syncthreads();
    for (int base = i_min; base < T; base += THREADS) {
        const int i = base + tid;
        const int flags = i < T ? column_flags<MC>(p, bh, i, jc0) : 0;
        const unsigned long long bal = __ballot(flags != 0);
        if (lane == 0) wcnt[wave] = __popcll(bal);
        __syncthreads();
        int off = wcnt[8];
        for (int w2 = 0; w2 < wave; ++w2) off += wcnt[w2];
        off += __popcll(bal & ((1ull << lane) - 1ull));
        if (flags != 0) tl[off] = i | (flags << 16);
        __syncthreads();
        if (tid == 0) {
            int tot = wcnt[8];
            for (int w2 = 0; w2 < NW; ++w2) tot += wcnt[w2];
            wcnt[8] = tot;
        }
        __syncthreads();
    }
    int ntl = wcnt[8];
    if (p.col_part_len > 0) {
        // Long columns (a key that every later query tile attends to walks up to T tiles while most
        // columns hold a few) are cut into parts of col_part_len tiles, each worked off by a group
        // of its own: this one keeps its part of the list, moved to the front.
        const int lo = part * p.col_part_len, len = max(0, min(ntl - lo, p.col_part_len));
        if (part > 0) {
            int keep[(MAX_T + THREADS - 1) / THREADS];
#pragma unroll
            for (int q = 0; q < (MAX_T + THREADS - 1) / THREADS; ++q) keep[q] = q * THREADS + tid < len ? tl[lo + q * THREADS + tid] : 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < (MAX_T + THREADS - 1) / THREADS; ++q)
                if (q * THREADS + tid < len) tl[q * THREADS + tid] = keep[q];
            __syncthreads();
        }
        ntl = len;
    }
    if (ntl == 0) {
        // no query tile for these keys (none attends to them, or all that do went by gather): their
        // dK, dV are zero, and a part of a shared column has nothing to add
        if (active && !shared_out) {
            f32x4* const dk = (f32x4*)(p.dK + hoff + kw0 * D);
            f32x4* const dv = (f32x4*)(p.dV + hoff + kw0 * D);
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            for (int e = lane; e < 32 * QB * D / 4; e += 64) { dk[e] = zero; dv[e] = zero; }
        }
        return;
    }

    Owned<E, D, QB> kf, vf;
    load_owned<E, D, QB>(kf, (const elem*)p.K + hoff, active ? kw0 : 0, lane);
    // keys scaled by kappa, a power of two: exact, and the scores come out as kappa <q, k>
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int s = 0; s < D / E::KSTEP; ++s) kf.f[qb][s] = kf.f[qb][s] * (elem)hc.kappa;
    load_owned<E, D, QB>(vf, (const elem*)p.V + hoff, active ? kw0 : 0, lane);

    f32x16 XV[D / 32][QB], XK[D / 32][QB];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int v = 0; v < 16; ++v) { XV[db][qb][v] = 0.f; XK[db][qb][v] = 0.f; }

    f32x16 S[2][QB], dP[2][QB];
    unsigned long long ntile_done = 0;
    constexpr int VEC_OFF = 2 * SM::RBYTES;
    auto issue_qg = [&](int it, char* b) {
        const long i = __builtin_amdgcn_readfirstlane(tl[it] & 0xffff);
        issue_rows<E, D, NW>(b, Qh, i * 64, wave, lane);
        issue_rows<E, D, NW>(b + SM::RBYTES, Gh, i * 64, wave, lane);
        // the tile's 64 values of -tau / rho (wave 0) and of -delta (wave 1), one float per lane
        if (wave == 0) load4_to_lds(uniform_address(p.ntau + ((long)bh * N + i * 64)), 4u * lane, lds_address(b + VEC_OFF));
        if (wave == 1) load4_to_lds(uniform_address(p.delta + ((long)bh * N + i * 64)), 4u * lane, lds_address(b + VEC_OFF + 4 * TILE));
    };
    // any tile, statements left to the compiler's order
    auto tile_plain_order = [&](int it, const char* qbuf) {
        const int ent = tl[it];
        const long i = ent & 0xffff;
        if (!((ent >> (16 + mycol)) & 1)) return;
        const char* gbuf = qbuf + SM::RBYTES;
        const float* tau_s = (const float*)(qbuf + VEC_OFF);
        const float* del_s = tau_s + TILE;
        stage1<E, D, QB>(S, qbuf, kf, lane);
        // streamed rows are queries here: hide key > query
        if (p.causal && i * 64 < kw0 + 32 * QB - 1) causal_hide<QB, false>(S, (int)i * 64, (int)kw0, lane);
        stage1<E, D, QB>(dP, gbuf, vf, lane);
        ++ntile_done;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v4 = 0; v4 < 16; v4 += 4) {
                // registers v4..v4+3 are four consecutive tile rows: one 16-byte read each
                const int row = trow(kb, v4, h);
                const f32x4 tq4 = *(const f32x4*)(tau_s + row), dq4 = *(const f32x4*)(del_s + row);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int v = v4 + e;
                    const float tq = tq4[e], dq = dq4[e];
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) {
                        // (same units as the staggered body)
                        const float yp = fmaxf(S[kb][qb][v] + tq, 0.f);
                        float u;
                        if constexpr (AM == ALPHA_15) u = yp;
                        else if constexpr (AM == ALPHA_20) u = (yp > 0.f) ? 1.f : 0.f;
                        else u = (yp > 0.f) ? pow_r1_rho(yp, r, lrho_u) : 0.f;
                        S[kb][qb][v] = u * yp;
                        dP[kb][qb][v] = u * (dP[kb][qb][v] + dq);
                    }
                }
            }
        stage2<E2, D, QB, true>(XV, gbuf, S, lane);
        stage2<E2, D, QB, true>(XK, qbuf, dP, lane);
        if constexpr (E2::EPL == 8 && EA_BWD_SPLIT >= SPLIT_SIGNED) { f16_tail<QB>(dP); stage2<E2, D, QB, true>(XK, qbuf, dP, lane); }
        if constexpr (E2::EPL == 8 && EA_BWD_SPLIT >= SPLIT_ALL) { f16_tail<QB>(S); stage2<E2, D, QB, true>(XV, gbuf, S, lane); }
    };
    if constexpr (E::EPL == 8 && QB == 1 && NBUF == 2) {
        // query tiles on the diagonal (the head of the ascending list), and one more when that makes
        // their number even, take the plain body; all tiles wholly below it the staggered one
        int ndiag = 0;
        if (p.causal)
            while (ndiag < ntl && (long)(tl[ndiag] & 0xffff) * 64 < k0 + BC - 1) ++ndiag;
        const Frag1<E, D> frag1(lane);
        const Frag2<E2, D> frag2(lane);
        stream_tiles_split(min(ntl, (ndiag + 1) & ~1), ntl, set0, set1, issue_qg, tile_plain_order,
            [&](int it, const char* qbuf) {
                if (!((tl[it] >> (16 + mycol)) & 1)) return;
                ++ntile_done;
                const float* tau_s = (const float*)(qbuf + VEC_OFF);
                dkdv_tile_staggered<E, E2, D, AM, EA_BWD_SPLIT>(qbuf, qbuf + SM::RBYTES, tau_s, tau_s + TILE, kf, vf, XV, XK, r, lrho_u, h, frag1, frag2);
            });
    } else {
        stream_tiles<NBUF>(ntl, set0, NBUF == 2 ? set1 : set0, issue_qg, tile_plain_order);
    }
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) { settle_acc(XV[db][qb]); settle_acc(XK[db][qb]); }
    if (active) {
        // units of P and U, see dkdv_tile_staggered
        const float unit_p = AM == ALPHA_15 ? hc.rho * hc.rho : hc.rho, unit_u = AM == ALPHA_15 ? hc.rho : 1.f;
        if (!shared_out) {
            store_owned_T<D, QB>(p.dV + hoff, kw0, XV, go_amax * unit_p, lane);
            store_owned_T<D, QB>(p.dK + hoff, kw0, XK, p.inv_sqrt_d * go_amax * unit_u, lane);
        } else {
            add_owned_T<D, QB>(p.dV + hoff, kw0, XV, go_amax * unit_p, lane);
            add_owned_T<D, QB>(p.dK + hoff, kw0, XK, p.inv_sqrt_d * go_amax * unit_u, lane);
        }
    }
    {
        const int slot[1] = {4};
        const unsigned long long val[1] = {ntile_done * QB};
        flush_counters<1>(blk_stats, p.stats, slot, val, tid, lane);
    }
}

// ---- backward of sparse row groups by gather --------------------------------------------------
// Where a row's support is a handful of keys, most tiles the mask marks hold one or two non-zeros,
// and the four matrix products per tile of dq_kernel / dkdv_kernel are spent on zeros.  For such
// row groups the backward of Sec. 3.3 is evaluated entry by entry instead:
//   bwd_list_kernel : one matrix product per marked tile (the scores); every score above the
//                     row's tau goes, with its key index, to a list private to the lane that
//                     computed it (two lists per row, as in tau_list_kernel).  A group whose
//                     lists stay short is flagged; dq_kernel and dkdv_kernel skip flagged groups.
//   bwd_rows_kernel : per row, over its listed support: dP_j = <dO_r, V_j>, delta, and
//                     dQ_r = sum_j dS_j K_j / sqrt(d) (Alg. 3, row by row); every entry is also
//                     filed under its key: (row, dS, P).
//   bwd_cols_kernel : per key, over the entries filed under it:
//                     dK_j += sum dS Q_r / sqrt(d), dV_j += sum P dO_r (Alg. 2, column by
//                     column), added to what dkdv_kernel
//                     stored for the other row groups (or, when none was left to it, written as
//                     dK_j, dV_j themselves).
//   bwd_file_kernel : hub keys, which have more entries than a key's list holds: bwd_rows_kernel
//                     logs the rest, this kernel orders the log by key, and work-groups of
//                     bwd_cols_kernel sum each hub key's entries, again in the order of their rows.
// They read the caller's Q, K, V, dO (not the 16-bit copies) and work in fp32.
// The gather path pays while a marked 64 x 64 tile holds only a few non-zeros: the group is flagged
// when its lists hold at most bwd_entries_per_tile entries per marked tile (and no list is full;
// which of the two limits: see there); or BWD_ENTRIES_PER_ROW per row (and no list is full); the sweep is left early once the entries
// so far run a quarter above that rate.

// Entries a row group may list to take the gather path, by its marked tiles and rows.  A group with few
// marked tiles (the first rows of a causal head) still has one entry or more per row, and is cheap either way: it
// goes with the rest, so that the matrix kernels' input copies are not made for its sake alone.
// Never more than LOG_PER_ROW a row, as in the forward: the log of hub keys has room for that.
template <class E, int D, int AM> EA_DEV int gather_budget(int marked, int rows, bool higher) {
    constexpr int PER_ROW_X128 = BWD_ENTRIES_PER_ROW * D * D / 128 / (AM == ALPHA_GEN ? 2 : 1);
    return min(max(bwd_entries_per_tile(D, sizeof(typename E::elem), higher) * marked, marked <= BWD_FEW_TILES ? PER_ROW_X128 * rows / 128 : 0),
               LOG_PER_ROW * rows);
}

// Whether the higher limit holds for a group by what the mask alone says: `marked` of `all` marked tiles, `groups` row groups
EA_DEV bool higher_limit(int marked, long all, int groups) { return groups <= BWD_FEW_GROUPS || 4l * marked * groups <= all; }

// Set bits of the whole mask, from bwd_begin_kernel's partial sums (called by whole waves)
EA_DEV long marked_tiles(const Params& p, int lane) {
    static_assert(MASK_PARTS == 64, "one partial sum per lane");
    int c = p.mask_parts[lane];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
    return c;
}
template <class E, int D, int QB, int AM, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_list_kernel(Params p) {
    using elem = typename E::elem;
    using KT = RowTile<E, D>;
    constexpr int BR = 32 * QB * NW, MR = (BR + 63) / 64, THREADS = NW * 64;
    __shared__ __align__(1024) char set0[KT::BYTES];
    __shared__ __align__(1024) char set1[KT::BYTES];
    __shared__ uint32_t fm[MR * MAX_W];
    __shared__ unsigned short tl[MAX_T];
    __shared__ int tl_count[4];
    __shared__ int gsum[4];                  // [0] support entries so far, [1] marked tiles, [2] a list is full, [3] the group's decision to leave
    __shared__ unsigned long long blk_stats[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int N = p.N, T = p.T, W = p.W;
    int bh, I;
    map_block(blockIdx.x, p.BH, (N + BR - 1) / BR, bh, I);
    const long q0 = (long)I * BR, qw0 = q0 + wave * 32 * QB;
    const bool active = qw0 < N;
    const elem* Qh = (const elem*)p.Q + (long)bh * N * D;
    const elem* Kh = (const elem*)p.K + (long)bh * N * D;
    const int myrow = (wave * 32 * QB) / 64;
    const HeadConsts hc = head_consts(p, bh);
    const float c = hc.c;

    // a mask with few marked tiles altogether: the matrix kernels are done before the gather
    // kernels' passes over dK, dV would be
    const int G = (N + BR - 1) / BR;
    const long all_marked = marked_tiles(p, lane);
    if (all_marked < (long)BWD_MIN_TILES_PER_BLOCK * p.BH * T) {
        if (tid == 0) {
            p.gflag[(long)bh * ((N + BR - 1) / BR) + I] = 0;
            atomicAdd(p.nplain, 1);
        }
        return;
    }
    if (tid < 4) gsum[tid] = 0;
    __syncthreads();
    {
        int marked = 0;
        for (int i = tid; i < MR * W; i += THREADS) {
            fm[i] = (I * MR + i / W < T) ? (uint32_t)p.mask[((long)bh * T + (long)I * MR + i / W) * W + (i % W)] : 0u;
            marked += __popc(fm[i]);
        }
        if (marked) atomicAdd(&gsum[1], marked);
    }
    build_tile_list(fm, MR, W, tl, tl_count, tid);
    const int nt = *tl_count;
    const int budget = gather_budget<E, D, AM>(gsum[1], min(BR, N - (int)q0), higher_limit(gsum[1], all_marked, p.BH * G));

    Owned<E, D, QB> qf;
    load_owned<E, D, QB>(qf, Qh, active ? qw0 : 0, lane);
    float thr[QB], floor_raw[QB];
    char* lptr[QB];
    int cnt[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        thr[qb] = active ? p.tau[(long)bh * N + qw0 + 32 * qb + n] : INFINITY;
        const float thr_raw = thr[qb] / c;   // a score passes only if it is above about this
        floor_raw[qb] = thr_raw - (1e-5f * fabsf(thr_raw) + 1e-30f);
        lptr[qb] = (char*)p.lists + ((size_t)((long)bh * N + (active ? qw0 : 0) + 32 * qb + n) * 2 + h) * (size_t)(BWD_LIST_CAP * 8);
        cnt[qb] = 0;
    }
    unsigned long long ntile = 0;
    f32x16 C[2][QB];
    auto issue = [&](int it, char* buf) { issue_rows<E, D, NW>(buf, Kh, (long)tl[it] * 64, wave, lane); };
    auto compute = [&](int it, const char* buf) {
        const int j = tl[it];
        if (!active || !mask_bit(fm, W, myrow, j)) return;
        stage1<E, D, QB, EA_FENCE, 0>(C, buf, qf, lane);    // rolling fragments (registers of two k-steps): four waves per SIMD fit
        if (p.causal && (long)j * 64 + 63 > qw0) causal_hide<QB, true>(C, j * 64, (int)qw0, lane);
        ++ntile;
        const int key0 = j * 64 + 8 * h;
        bool full = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float gm[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                gm[g] = C[g >> 1][qb][8 * (g & 1)];
#pragma unroll
                for (int v = 1; v < 8; ++v) gm[g] = fmaxf(gm[g], C[g >> 1][qb][8 * (g & 1) + v]);
            }
            const float lm = fmaxf(fmaxf(gm[0], gm[1]), fmaxf(gm[2], gm[3]));
            if (!__any(lm > floor_raw[qb])) continue;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (!__any(gm[g] > floor_raw[qb])) continue;
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const float sc = C[g >> 1][qb][8 * (g & 1) + v];
                    if (fmaf(c, sc, -thr[qb]) > 0.f) {
                        uint2 ent;          // tile row of register v of group g: see causal_hide
                        ent.x = __float_as_uint(sc); ent.y = (uint32_t)(key0 + 32 * (g >> 1) + 16 * (g & 1) + v);
                        *(uint2*)(lptr[qb] + 8 * min(cnt[qb], BWD_LIST_CAP - 1)) = ent;
                        ++cnt[qb];
                        lds_add_u32(&gsum[0], 1u);
                    }
                }
            }
            full |= cnt[qb] > BWD_LIST_CAP;
        }
        if (__any(full) && lane == 0) atomicOr(&gsum[2], 1);
    };
    // the walk of stream_tiles, left as soon as the gather path cannot pay any more.  The counters
    // keep moving while the waves of a group work on a tile, so the group's decision is taken by
    // one thread, from the values it finds right after a barrier, and published in gsum[3]; every
    // wave reads it after the NEXT barrier, before which nobody writes it again: all waves leave
    // at the same tile, or none does.
    auto hopeless = [&](int it) {
        if (*(volatile int*)&gsum[2]) return true;
        const int e = *(volatile int*)&gsum[0];
        return e > budget || (it >= 8 && 4l * e * nt > 5l * budget * it);
    };
    bool gave_up = false;
    if (nt > 0) issue(0, set0);
    for (int it = 0; it < nt; it += 2) {
        wait_loads();
        __syncthreads();
        if ((it & 7) == 0 && tid == 0) gsum[3] = hopeless(it);
        if (it + 1 < nt) issue(it + 1, set1);
        compute(it, set0);
        if (it + 1 >= nt) break;
        wait_loads();
        __syncthreads();
        if ((it & 7) == 0 && *(volatile int*)&gsum[3]) { gave_up = true; break; }
        if (it + 2 < nt) issue(it + 2, set0);
        compute(it + 1, set1);
    }
    lds_settle();            // this wave's counter updates have reached LDS
    wait_loads();
    __syncthreads();
    if (tid == 0) gsum[3] = gave_up || hopeless(nt);
    __syncthreads();
    const int nrows = min(BR, N - (int)q0);
    const bool gather = !*(volatile int*)&gsum[3];
    if (active) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) p.scnt[((long)bh * N + qw0 + 32 * qb + n) * 2 + h] = gather ? cnt[qb] : 0;
    }
    if (tid == 0) {
        p.gflag[(long)bh * ((N + BR - 1) / BR) + I] = gather;
        if (!gather) atomicAdd(p.nplain, 1);
    }
    {
        const int slot[2] = {10, 11};
        const unsigned long long val[2] = {ntile * QB, (tid == 0 && gather) ? (unsigned long long)nrows : 0ull};
        flush_counters<2>(blk_stats, p.stats, slot, val, tid, lane);
    }
}

// When the caller hands the forward's workspace to the backward, the supports need not be found
// again: for the row groups whose output the forward gathered, the front of its candidate lists is
// the support (raw score, key index), with the counts beside it.  This kernel takes the place of
// bwd_list_kernel's sweep: per row group of the backward it applies the same rule - at most so many
// support entries per marked tile, or per row where few tiles are marked - to the forward's counts; at head dim 128 the higher limit
// also where the entries per key let it.
template <class E, int D, int AM>
__global__ __launch_bounds__(128) void bwd_decide_kernel(Params p) {
    __shared__ int gsum[2];
    const int tid = threadIdx.x;
    const int N = p.N, T = p.T, W = p.W, BR = p.grows, G = (N + BR - 1) / BR;
    int bh, I;
    map_block(blockIdx.x, p.BH, G, bh, I);
    const int fwd_grows = (int)p.fwd_scal[2];
    const long all_marked = marked_tiles(p, tid & 63);
    bool gather = all_marked >= (long)BWD_MIN_TILES_PER_BLOCK * p.BH * T && fwd_grows > 0
                  && p.fwd_gflag[(long)bh * ((N + fwd_grows - 1) / fwd_grows) + (I * BR) / fwd_grows] != 0;
    if (tid < 2) gsum[tid] = 0;
    __syncthreads();
    if (gather) {
        const int row = I * BR + tid;
        int ent = 0, marked = 0;
        if (tid < BR && row < N) ent = p.scnt[((long)bh * N + row) * 2] + p.scnt[((long)bh * N + row) * 2 + 1];
        const int MR = (BR + 63) / 64;
        for (int i = tid; i < MR * W; i += 128)
            if (I * MR + i / W < T) marked += __popc((uint32_t)p.mask[((long)bh * T + (long)I * MR + i / W) * W + (i % W)]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) { ent += __shfl_xor(ent, off); marked += __shfl_xor(marked, off); }
        if ((tid & 63) == 0) { atomicAdd(&gsum[0], ent); atomicAdd(&gsum[1], marked); }
    }
    __syncthreads();
    if (tid == 0) {
        if (gather) {
            const int ent = gsum[0], marked = gsum[1], rows = min(BR, N - I * BR);
            bool higher = higher_limit(marked, all_marked, p.BH * G);
            if (D == 128 && !higher) {
                // entries of a key of the group's rows if the rows after it (without a causal mask: all rows) attend to as many keys
                const float later = p.causal ? 0.69314718f * __builtin_amdgcn_logf((float)N / ((float)(I * BR) + 0.5f * (float)rows)) : 1.f;
                higher = (float)ent * later <= BWD_KEY_ENTRIES * (float)rows;
            }
            gather = ent <= gather_budget<E, D, AM>(marked, rows, higher);
        }
        p.gflag[(long)bh * G + I] = gather;
        if (!gather) atomicAdd(p.nplain, 1);
        else atomicAdd(&p.stats[(blockIdx.x & (STATS_COPIES - 1)) * STATS_WORDS + 11], (unsigned long long)min(BR, N - I * BR));
    }
}

// Sixteen lanes per row (GatherLanes).  Per row, over its entries: dP_j = <dO_r, V_j>, delta = sum u dP / sum u,
// dQ_r = sum_j dS_j K_j / sqrt(d) with dS = u (dP - delta); every entry is filed under its key as
// (row, dS, P).  dP of the first KEEP entries stays in registers between the two passes; a longer
// row computes it a second time.  An entry whose key's list is full goes to the log of its row's segment;
// the first of a key reports the key as a hub key.  SCALED: dkdv_kernel works on dO / max|dO|, so the delta handed to it is in those units.
// (16-bit inputs: held to the registers of seven waves per SIMD; left to itself the compiler takes 82, five waves.)
template <class E, int D, int AM, bool SCALED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(typename E::elem) == 2 ? 7 : 5))) void bwd_rows_kernel(Params p) {
    using elem = typename E::elem;
    using L = GatherLanes<E, D>;
    using vec = typename L::vec;
    constexpr int EPT = L::EPT, KEEPC = 3, BT = 4;     // chunks kept in registers; rows of V or K in flight per lane
    static_assert(L::STEPS % BT == 0, "a chunk is a whole number of batches");
    const int tid = threadIdx.x, sub = tid & 15, rsel = tid >> 4, lane = tid & 63;
    // a work-group takes GATHER_ROWS rows of a row group (one per 16 lanes): the rows are
    // chains of dependent loads, so many short work-groups hide their latency better than few long ones
    static_assert(GATHER_ROWS == 16, "one row per sixteen lanes");
    const int N = p.N, G = (N + p.grows - 1) / p.grows, parts = p.grows / GATHER_ROWS;
    int bh, I;
    map_block(blockIdx.x, p.BH, G * parts, bh, I);
    const int part = I % parts;
    I /= parts;
    if (!p.gflag[(long)bh * G + I]) return;
    const int row = I * p.grows + part * GATHER_ROWS + rsel;
    if (row >= N) return;                              // (N is a multiple of 64: whole work-groups)
    const HeadConsts hc = head_consts(p, bh);
    const float c = hc.c, r = hc.r;
    float amax = 1.f;
    if constexpr (SCALED) {
        amax = __uint_as_float(p.scal[0]);
        if (!(amax > 0.f)) amax = 1.f;
    }
    const long hoff = (long)bh * N * D, gi = (long)bh * N + row;
    const HeadRows<E, D> Kh(p.K, (long)bh * N, N, sub), Vh(p.V, (long)bh * N, N, sub);
    const int cap8 = p.list_cap * 8;                   // bytes of one lane list
    const char* l0 = (const char*)p.lists + (size_t)gi * (size_t)(2 * cap8);        // the second list follows the first
    const float tau = p.tau[gi];
    const int s0 = p.scnt[gi * 2], tot = s0 + p.scnt[gi * 2 + 1];
    const vec gv = *(const vec*)((const elem*)p.dO + hoff + (long)row * D + L::column(sub));
    const int nmax = longest_list(tot);

    auto entry_ptr = [&](int i) { return l0 + (i < s0 ? i * 8 : cap8 + (i - s0) * 8); };
    struct Entry { uint32_t key; float u, pr; };
    auto load_entry = [&](int i) {
        uint2 e = make_uint2(0u, NO_ENTRY);
        if (i < tot) e = *(const uint2*)entry_ptr(i);
        const float y = fmaf(c, __uint_as_float(e.x), -tau);
        const bool in = i < tot && y > 0.f;
        Entry x;
        x.key = e.y;
        x.u = in ? pow_r1<AM>(y, r) : 0.f;
        x.pr = in ? pow_r<AM>(y, r) : 0.f;
        return x;
    };
    // dP of a chunk's entries, each left in the lane that holds the entry (0 in one that holds none)
    auto chunk_dP = [&](uint32_t key, int left) {
        float dP = 0.f;
        unroll_steps<L::STEPS / BT>([&](auto b) {
            constexpr int S0 = decltype(b)::value * BT;
            if (S0 * L::PAR >= left) return;
            vec v[BT];
            unroll_steps<BT>([&](auto u) { v[decltype(u)::value] = Vh.load(L::template of_step<S0 + decltype(u)::value>(key)); });
            unroll_steps<BT>([&](auto u) {
                constexpr int S = S0 + decltype(u)::value;
                const float t = L::entry_sum(dot_share<E, EPT>(gv, v[decltype(u)::value], 0.f));
                if (L::template holds<S>(sub)) dP = t;
            });
        });
        return key == NO_ENTRY ? 0.f : dP;
    };
    // An entry's slot in its key's list.  In the first chunk, rows of the wave that hold the same key at the same place
    // of their lists (a sink, the first keys of a head that every row attends to) ask for their slots in one addition: on
    // such a key the additions queue up
    // (4 sinks, 32 heads of 4096 tokens, d = 64: backward 363 -> 262 us; one sink, 32 heads of 16384, d = 128: 1464 -> 789).
    int* const count = p.kcnt + (long)bh * N;
    auto take_slots_together = [&](uint32_t key, bool mine) __attribute__((always_inline)) {
        const uint32_t k = mine ? key : NO_ENTRY | (uint32_t)lane;
        const auto x1 = __builtin_amdgcn_permlane16_swap(k, k, false, false);
        const uint32_t k1 = (lane & 16) ? x1[0] : x1[1];                           // what lane ^ 16 holds; k2, k3: lane ^ 32, lane ^ 48
        const auto x2 = __builtin_amdgcn_permlane32_swap(k, k, false, false), x3 = __builtin_amdgcn_permlane32_swap(k1, k1, false, false);
        const uint32_t k2 = (lane & 32) ? x2[0] : x2[1], k3 = (lane & 32) ? x3[0] : x3[1];
        const bool e1 = k1 == k, e2 = k2 == k, e3 = k3 == k;
        int slot = 0;
        if (!__any(e1 || e2 || e3)) {
            if (mine) slot = atomicAdd(count + key, 1);
            return slot;
        }
        const int g = lane >> 4;
        const int rank = (e1 && (g & 1)) + (e2 && (g & 2)) + (e3 && (g & 2));      // (g ^ 3 < g: g is 2 or 3)
        int lead = g;
        if (e1) lead = min(lead, g ^ 1);
        if (e2) lead = min(lead, g ^ 2);
        if (e3) lead = min(lead, g ^ 3);
        if (mine && rank == 0) slot = atomicAdd(count + key, 1 + e1 + e2 + e3);
        return __shfl(slot, (lead << 4) | sub) + rank;
    };
    Entry ent[KEEPC];
    float dP[KEEPC];
    int slot[KEEPC];
    float num = 0.f, den = 0.f;
    unroll_steps<KEEPC>([&](auto cc) {
        constexpr int C = decltype(cc)::value;
        if (16 * C >= nmax) return;
        const int i = 16 * C + L::entry_of(sub);
        ent[C] = load_entry(i);
        slot[C] = 0;
        if constexpr (C == 0) slot[C] = take_slots_together(ent[C].key, i < tot);
        else if (i < tot) slot[C] = atomicAdd(count + ent[C].key, 1);
        dP[C] = chunk_dP(ent[C].key, nmax - 16 * C);
        num = fmaf(ent[C].u, dP[C], num);
        den += ent[C].u;
    });
    for (int i0 = 16 * KEEPC; i0 < nmax; i0 += 16) {
        const Entry e = load_entry(i0 + L::entry_of(sub));
        num = fmaf(e.u, chunk_dP(e.key, nmax - i0), num);
        den += e.u;
    }
    num = group_sum<16>(num);
    den = group_sum<16>(den);
    const float delta = den > 0.f ? num / den : 0.f;

    // this row's segment of the log (the work-group's rows lie in one)
    const int seg = row / LOG_ROWS, seg_room = LOG_PER_ROW * min(LOG_ROWS, N - seg * LOG_ROWS);
    LogEntry* const log = p.klog + ((size_t)bh * N + (size_t)seg * LOG_ROWS) * LOG_PER_ROW;
    auto log_entries = [&](unsigned long long which, uint32_t key, int sl, float dS, float pr) {
        const int lead = __ffsll((long long)which) - 1;
        int at = 0;
        if (lane == lead) at = atomicAdd(&p.log_cnt[bh * MAX_LOG_SEGMENTS + seg], __popcll(which));
        at = __builtin_amdgcn_readlane(at, lead) + __popcll(which & ((1ull << lane) - 1ull));
        if (!((which >> lane) & 1)) return;
        const uint32_t past = (uint32_t)(sl - KEY_LIST_CAP);
        if (at < seg_room)                             // (always: see gather_budget)
            log[at] = LogEntry{key | past << ROW_BITS, (uint32_t)row | past >> SLOT_LOW_BITS << ROW_BITS, dS, pr};
        if (past == 0u) p.hub_key[(long)bh * N + atomicAdd(&p.hub_cnt[bh], 1)] = (int32_t)key;
    };
    float x[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) x[k] = 0.f;
    // file a chunk's entries under their keys and add their share of dQ
    auto finish_chunk = [&](const Entry& e, float dPe, int sl, int i0) __attribute__((always_inline)) {
        const float dS = e.key == NO_ENTRY ? 0.f : e.u * (dPe - delta);
        const int i = i0 + L::entry_of(sub);
        if (i < tot && sl < KEY_LIST_CAP) ((KeyEntry*)p.klist)[((long)bh * N + e.key) * KEY_LIST_CAP + sl] = KeyEntry{(uint32_t)row, dS, e.pr};
        const unsigned long long past = __ballot(i < tot && sl >= KEY_LIST_CAP);
        if (past) log_entries(past, e.key, sl, dS, e.pr);
        unroll_steps<L::STEPS / BT>([&](auto b) {
            constexpr int S0 = decltype(b)::value * BT;
            if (S0 * L::PAR >= nmax - i0) return;
            vec v[BT];
            unroll_steps<BT>([&](auto u) { v[decltype(u)::value] = Kh.load(L::template of_step<S0 + decltype(u)::value>(e.key)); });
            unroll_steps<BT>([&](auto u) { add_scaled<EPT>(x, L::template of_step<S0 + decltype(u)::value>(dS), v[decltype(u)::value]); });
        });
    };
    unroll_steps<KEEPC>([&](auto cc) {
        constexpr int C = decltype(cc)::value;
        if (16 * C < nmax) finish_chunk(ent[C], dP[C], slot[C], 16 * C);
    });
    for (int i0 = 16 * KEEPC; i0 < nmax; i0 += 16) {
        const Entry e = load_entry(i0 + L::entry_of(sub));
        int sl = 0;
        if (i0 + L::entry_of(sub) < tot) sl = atomicAdd(count + e.key, 1);
        finish_chunk(e, chunk_dP(e.key, nmax - i0), sl, i0);
    }
#pragma unroll
    for (int k = 0; k < EPT; ++k) x[k] = L::halves_sum(x[k]) * p.inv_sqrt_d;
    L::store(p.dQ + gi * D, x, sub);
    if (sub == 0) {
        p.delta[gi] = -delta / amax;
        p.ntau[gi] = -tau / hc.rho;
    }
}

// The log by key: where each hub key's part of hub_index starts (by the keys' counts in the order they were
// reported; every work-group of a head forms the same offsets for itself), and the log entries' places there.
// Keys with more entries than HUB_BATCH are summed from the log segments themselves.  Nothing to do, and gone
// after one load, in heads without hub keys.
constexpr int FILE_GROUPS = 16;          // work-groups per head, each with every FILE_GROUPS-th segment of the log
constexpr int HUB_BATCH = 1024;          // entries of a hub key that are put in order in LDS at a time
static __global__ __launch_bounds__(256) void bwd_file_kernel(Params p) {
    __shared__ int wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int N = p.N, bh = blockIdx.x / FILE_GROUPS, part = blockIdx.x % FILE_GROUPS;
    const int n = p.hub_cnt[bh];
    if (n == 0) return;
    const long hk = (long)bh * N;
    int before = 0;
    for (int i0 = 0; i0 < n; i0 += 256) {
        const int i = i0 + tid;
        int key = 0, len = 0;
        if (i < n) {
            key = p.hub_key[hk + i];
            const int cnt = p.kcnt[hk + key];
            if (cnt <= HUB_BATCH) len = cnt - KEY_LIST_CAP;
        }
        int incl = len;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(incl, off);
            if (lane >= off) incl += t;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        int at = before + incl - len;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            at += w < wave ? wsum[w] : 0;
            before += wsum[w];
        }
        if (i < n) p.hub_off[hk + key] = at;
        __syncthreads();
    }
    // the offsets are read back by other threads of this work-group: its stores have reached the L2, and
    // the loads go there
    wait_loads();
    __syncthreads();
    uint32_t* const index = p.hub_index + (size_t)bh * N * LOG_PER_ROW;
    for (int seg = part; seg * LOG_ROWS < N; seg += FILE_GROUPS) {
        const int m = min(p.log_cnt[bh * MAX_LOG_SEGMENTS + seg], LOG_PER_ROW * min(LOG_ROWS, N - seg * LOG_ROWS));
        const uint32_t first = (uint32_t)(seg * LOG_ROWS) * LOG_PER_ROW;
        for (int e = tid; e < m; e += 256) {
            const LogEntry* le = p.klog + (size_t)bh * N * LOG_PER_ROW + first + e;
            const uint32_t key = le->key_slot & ((1u << ROW_BITS) - 1), past = le->key_slot >> ROW_BITS | le->row_slot >> ROW_BITS << SLOT_LOW_BITS;
            if (p.kcnt[hk + key] > HUB_BATCH) continue;
            index[__hip_atomic_load(&p.hub_off[hk + key], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + (int)past] = first + e;
        }
    }
}

// dK or dV of one hub key by a whole work-group: its entries in the order of their query rows in LDS, up to
// HUB_BATCH of them at once, a run of them for every sixteen lanes, and the sixteen partial sums added in order.
// Up to HUB_BATCH entries are ranked against each other; a key with more is worked off by segments of LOG_ROWS
// rows, whose entries have a place each by their row.
// Bound: one work-group reads the rows of a key's entries (2 D bytes each), so that a sink takes as long as its
// rows take at one CU's rate.  Backward of 32 heads of 16384 tokens (d = 128) with one sink 8640 -> 800 us, 8 heads of
// 65536 7460 -> 1550 us, against fp32 atomics on the key's rows, whose sums changed from run to run besides; steps with
// a few hundred small hub keys: 16384 tokens, sigma = 1, 4664 -> 4529, 65536 planted 4250 -> 4146 us.
template <class E, int D> struct HubLds {
    uint32_t row[HUB_BATCH];             // in order
    float w[HUB_BATCH];
    union {
        struct { uint32_t filed_row[HUB_BATCH]; float filed_w[HUB_BATCH]; };    // as they were filed
        struct {
            float by_row[LOG_ROWS];      // a segment's entries at their row's place,
            uint32_t bits[LOG_ROWS / 32];               // which rows are there, and how many before each word
            int before[LOG_ROWS / 32 + 1];
        };
        float part[16][D];
    };
};
// Work-groups per head: about two per CU over all heads (those of heads without hub keys cost a work-group's launch each:
// 64 heads of 4096 tokens, 32 per head against 8: 1.5 us)
__host__ __device__ constexpr int hub_groups(int BH) { return BH >= 128 ? 4 : BH <= 8 ? 64 : 512 / BH; }
template <class E, int D>
EA_DEV void hub_key_sums(const Params& p, HubLds<E, D>& s, int bh, int first_item, int groups, bool fresh) {
    using elem = typename E::elem;
    using L = GatherLanes<E, D>;
    using vec = typename L::vec;
    constexpr int EPT = L::EPT, BT = sizeof(elem) == 2 ? 8 : 4;    // rows in flight (one work-group per key: more than elsewhere)
    static_assert(HUB_BATCH <= 4 * 256 && LOG_ROWS <= HUB_BATCH && LOG_ROWS / 32 < 64, "a segment is a batch, its bits are at most a word per lane");
    const int tid = threadIdx.x, sub = tid & 15, group = tid >> 4, lane = tid & 63;
    const int N = p.N, n = p.hub_cnt[bh];
    const long hk = (long)bh * N;
    const LogEntry* const log = p.klog + (size_t)hk * LOG_PER_ROW;
    const uint32_t* const index = p.hub_index + (size_t)hk * LOG_PER_ROW;
    constexpr uint32_t ROW_MASK = (1u << ROW_BITS) - 1;
    for (int item = first_item; item < 2 * n; item += groups) {
        const uint32_t key = (uint32_t)p.hub_key[hk + (item >> 1)];
        const bool is_dk = !(item & 1);
        const int cnt = p.kcnt[hk + key];
        const KeyEntry* const el = (const KeyEntry*)p.klist + (hk + key) * KEY_LIST_CAP;
        const HeadRows<E, D> rows(is_dk ? p.Q : p.dO, hk, N, sub);
        float acc[EPT];
#pragma unroll
        for (int k = 0; k < EPT; ++k) acc[k] = 0.f;
        // sum of the m entries now in s.row, s.w, added to acc
        auto add_batch = [&](int m) {
            const int share = (m + 15) / 16, mine = min(max(m - group * share, 0), share);
            const int nmax = longest_list(mine);
            for (int i0 = 0; i0 < nmax; i0 += 16) {
                const int i = i0 + L::entry_of(sub);
                uint32_t row = NO_ENTRY;
                float w = 0.f;
                if (i < mine) { row = s.row[group * share + i]; w = s.w[group * share + i]; }
                unroll_steps<L::STEPS / BT>([&](auto b) {
                    constexpr int S0 = decltype(b)::value * BT;
                    if (S0 * L::PAR >= nmax - i0) return;
                    vec v[BT];
                    unroll_steps<BT>([&](auto u) { v[decltype(u)::value] = rows.load(L::template of_step<S0 + decltype(u)::value>(row)); });
                    unroll_steps<BT>([&](auto u) { add_scaled<EPT>(acc, L::template of_step<S0 + decltype(u)::value>(w), v[decltype(u)::value]); });
                });
            }
        };
        if (cnt <= HUB_BATCH) {
            const int off = p.hub_off[hk + key];
            for (int i = tid; i < cnt; i += 256) {
                uint32_t row;
                float w;
                if (i < KEY_LIST_CAP) { row = el[i].row; w = is_dk ? el[i].dS : el[i].pr; }
                else {
                    const LogEntry le = log[min(index[off + i - KEY_LIST_CAP], (uint32_t)N * LOG_PER_ROW - 1u)];
                    row = le.row_slot & ROW_MASK; w = is_dk ? le.dS : le.pr;
                }
                s.filed_row[i] = row; s.filed_w[i] = w;
            }
            __syncthreads();
            if (tid < cnt) {
                uint32_t row[4];
                int rank[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) { row[q] = s.filed_row[min(tid + 256 * q, cnt - 1)]; rank[q] = 0; }
                for (int j = 0; j < cnt; ++j) {
                    const uint32_t rj = s.filed_row[j];
#pragma unroll
                    for (int q = 0; q < 4; ++q) rank[q] += rj < row[q];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (tid + 256 * q < cnt) { s.row[rank[q]] = row[q]; s.w[rank[q]] = s.filed_w[tid + 256 * q]; }
            }
            __syncthreads();
            add_batch(cnt);
        } else {
            for (int seg = 0; seg * LOG_ROWS < N; ++seg) {
                const int r0 = seg * LOG_ROWS;
                if (tid < LOG_ROWS / 32) s.bits[tid] = 0u;
                __syncthreads();
                auto put = [&](uint32_t row, float w) {
                    const uint32_t at = row - (uint32_t)r0;
                    s.by_row[at] = w;
                    atomicOr(&s.bits[at >> 5], 1u << (at & 31));
                };
                if (tid < KEY_LIST_CAP && (int)(el[tid].row / LOG_ROWS) == seg) put(el[tid].row, is_dk ? el[tid].dS : el[tid].pr);
                const int m = min(p.log_cnt[bh * MAX_LOG_SEGMENTS + seg], LOG_PER_ROW * min(LOG_ROWS, N - r0));
                for (int i = tid; i < m; i += 256) {
                    const LogEntry* le = log + (size_t)r0 * LOG_PER_ROW + i;
                    if ((le->key_slot & ROW_MASK) == key) put(le->row_slot & ROW_MASK, is_dk ? le->dS : le->pr);
                }
                __syncthreads();
                if (tid < 64) {
                    const int c = lane < LOG_ROWS / 32 ? __popc(s.bits[lane]) : 0;
                    int incl = c;
#pragma unroll
                    for (int off = 1; off < 64; off <<= 1) {
                        const int t = __shfl_up(incl, off);
                        if (lane >= off) incl += t;
                    }
                    if (lane <= LOG_ROWS / 32) s.before[lane] = incl - c;
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < LOG_ROWS / 256; ++q) {
                    const int at = tid + 256 * q;
                    const uint32_t word = s.bits[at >> 5], bit = 1u << (at & 31);
                    if (word & bit) {
                        const int pos = s.before[at >> 5] + __popc(word & (bit - 1u));
                        s.row[pos] = (uint32_t)(r0 + at);
                        s.w[pos] = s.by_row[at];
                    }
                }
                __syncthreads();
                add_batch(s.before[LOG_ROWS / 32]);
                __syncthreads();
            }
        }
#pragma unroll
        for (int k = 0; k < EPT; ++k) acc[k] = L::halves_sum(acc[k]);
        L::store(s.part[group], acc, sub);
        __syncthreads();
        if (tid < D) {
            float sum = 0.f;
#pragma unroll
            for (int g = 0; g < 16; ++g) sum += s.part[g][tid];
            if (is_dk) sum *= p.inv_sqrt_d;
            float* out = (is_dk ? p.dK : p.dV) + (hk + key) * D + tid;
            *out = fresh ? sum : *out + sum;
        }
        __syncthreads();
    }
}

// Sixteen lanes per key (GatherLanes).  Where dkdv_kernel has stored dK, dV for the other row groups, the key's
// rows are read, added to, and written back; when no row group was left to dkdv_kernel (it then
// stores nothing) the sums are the rows, and keys without entries get zeros.
// The entries of a key were filed in the order an integer atomic handed out their slots, which
// changes from run to run.  They are summed in the order of their query rows instead (a row files
// at most one entry per key, so the rows are distinct): every lane holds one entry in sixteen, finds
// its rank among the key's rows through LDS and leaves it there in its place, and dK, dV of a key come
// out bit-identical in every run.  The first work-groups (hub_groups per head) take the hub keys, which the others
// pass over.
template <class E, int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(typename E::elem) == 2 || D == 64 ? 6 : 5))) void bwd_cols_kernel(Params p) {
    using elem = typename E::elem;
    using L = GatherLanes<E, D>;
    using vec = typename L::vec;
    constexpr int EPT = L::EPT, BT = 4;                // rows of Q and of dO in flight per lane
    typedef float f4 __attribute__((ext_vector_type(4)));
    static_assert(BWD_COLS_KEYS == 16, "one key per sixteen lanes");
    constexpr int PER_LANE = KEY_LIST_CAP / 16;        // entries of a key's list per lane of its 16
    struct KeyLds { uint32_t row[16][KEY_LIST_CAP]; float2 val[16][KEY_LIST_CAP]; };
    __shared__ union { KeyLds keys; HubLds<E, D> hub; } lds;
    auto& row_s = lds.keys.row;
    auto& val_s = lds.keys.val;
    const int tid = threadIdx.x, sub = tid & 15, rsel = tid >> 4;
    const int N = p.N, G = (N + BWD_COLS_KEYS - 1) / BWD_COLS_KEYS, HG = hub_groups(p.BH), hub_blocks = p.BH * HG;
    const bool fresh = *p.nplain == 0;
    if ((int)blockIdx.x < hub_blocks) {
        hub_key_sums<E, D>(p, lds.hub, blockIdx.x / HG, blockIdx.x % HG, HG, fresh);
        return;
    }
    int bh, I;
    map_block((int)blockIdx.x - hub_blocks, p.BH, G, bh, I);
    const int key = I * BWD_COLS_KEYS + rsel;
    if (key >= N) return;                              // (N is a multiple of 64: whole work-groups)
    const long kj = (long)bh * N + key, hoff = (long)bh * N * D;
    const HeadRows<E, D> Qh(p.Q, (long)bh * N, N, sub), Gh(p.dO, (long)bh * N, N, sub);
    const int filed = p.kcnt[kj], cnt = filed > KEY_LIST_CAP ? 0 : filed;
    const int nmax = longest_list(cnt);
    if (nmax == 0 && !fresh) return;
    const KeyEntry* el = (const KeyEntry*)p.klist + kj * KEY_LIST_CAP;
    auto wave_fence = [] {                             // (the 16 lanes of a key sit in one wave, whose LDS operations execute in issue order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    KeyEntry e[PER_LANE];
    int rank[PER_LANE];
    unroll_steps<PER_LANE>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        e[q] = KeyEntry{0xffffffffu, 0.f, 0.f};
        rank[q] = 0;
        if (16 * q < nmax && sub + 16 * q < cnt) { e[q] = el[sub + 16 * q]; row_s[rsel][sub + 16 * q] = e[q].row; }
    });
    wave_fence();
    if (nmax <= 16) {
        for (int j = 0; j < nmax; ++j) rank[0] += j < cnt && row_s[rsel][j] < e[0].row;
    } else if (nmax <= 48) {
        for (int j = 0; j < nmax; ++j) {
            const uint32_t rj = j < cnt ? row_s[rsel][j] : 0xffffffffu;
#pragma unroll
            for (int q = 0; q < 3; ++q) rank[q] += rj < e[q].row;
        }
    } else {
        for (int j = 0; j < nmax; ++j) {
            const uint32_t rj = j < cnt ? row_s[rsel][j] : 0xffffffffu;
#pragma unroll
            for (int q = 0; q < PER_LANE; ++q) rank[q] += rj < e[q].row;
        }
    }
    wave_fence();
    unroll_steps<PER_LANE>([&](auto qq) {
        constexpr int q = decltype(qq)::value;
        if (16 * q < nmax && sub + 16 * q < cnt) {
            row_s[rsel][rank[q]] = e[q].row;
            val_s[rsel][rank[q]] = make_float2(e[q].dS, e[q].pr);
        }
    });
    wave_fence();
    float ak[EPT], av[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) { ak[k] = 0.f; av[k] = 0.f; }
    for (int i0 = 0; i0 < nmax; i0 += 16) {
        const int i = i0 + L::entry_of(sub);
        uint32_t row = NO_ENTRY;
        float2 w = make_float2(0.f, 0.f);              // dS, P
        if (i < cnt) { row = row_s[rsel][i]; w = val_s[rsel][i]; }
        unroll_steps<L::STEPS / BT>([&](auto b) {
            constexpr int S0 = decltype(b)::value * BT;
            if (S0 * L::PAR >= nmax - i0) return;
            vec qv[BT], gv[BT];
            unroll_steps<BT>([&](auto u) {
                constexpr int U = decltype(u)::value;
                const uint32_t of_entry = L::template of_step<S0 + U>(row);
                qv[U] = Qh.load(of_entry);
                gv[U] = Gh.load(of_entry);
            });
            unroll_steps<BT>([&](auto u) {
                constexpr int U = decltype(u)::value;
                add_scaled<EPT>(ak, L::template of_step<S0 + U>(w.x), qv[U]);
                add_scaled<EPT>(av, L::template of_step<S0 + U>(w.y), gv[U]);
            });
        });
    }
    if (filed > KEY_LIST_CAP || (cnt == 0 && !fresh)) return;
#pragma unroll
    for (int k = 0; k < EPT; ++k) { ak[k] = L::halves_sum(ak[k]) * p.inv_sqrt_d; av[k] = L::halves_sum(av[k]); }
    float* dk = p.dK + kj * D;
    float* dv = p.dV + kj * D;
    if (!fresh) {
        // (a lane adds what it will store: with two entries side by side each half stores half of its share)
#pragma unroll
        for (int k = 0; k < EPT; k += 4) {
            const f4 a = *(const f4*)(dk + L::column(sub) + k), b = *(const f4*)(dv + L::column(sub) + k);
#pragma unroll
            for (int q = 0; q < 4; ++q) { ak[k + q] += a[q]; av[k + q] += b[q]; }
        }
    }
    L::store(dk, ak, sub);
    L::store(dv, av, sub);
}

// What the backward starts from, in one launch (three of them cost 4 - 5 us each): cleared key counters (and behind them
// the counters of plain row groups, hub keys and log entries), cleared statistics (stats null: they are cleared already), and the
// set bits of the mask, a partial sum for each of the first MASK_PARTS blocks.
static __global__ __launch_bounds__(256) void bwd_begin_kernel(int32_t* counters, long n, unsigned long long* stats, int nstats, unsigned int* scal,
                                                               const int32_t* mask, long nwords, int32_t* mask_parts) {
    __shared__ int part[4];
    const long first = blockIdx.x * 256L + threadIdx.x, stride = (long)gridDim.x * 256;
    for (long i = first; i < n; i += stride) counters[i] = 0;
    if (stats) {
        for (long i = first; i < nstats; i += stride) stats[i] = 0ull;
        if (first < 4) scal[first] = 0u;
    }
    if (blockIdx.x >= MASK_PARTS) return;
    int c = 0;
    for (long i = first; i < nwords; i += MASK_PARTS * 256L) c += __popc((uint32_t)mask[i]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) mask_parts[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

}  // namespace ea
