// Forward kernels (Alg. 1 of the AdaSplash-2 paper), re-cut for CDNA4:
//   tau_kernel : Phases 1 and 2 in one dense sweep (row maximum, LDS histogram of the scores within
//                one unit of the running maximum, per-row tile maxima), histogram solve -> tau_0,
//                candidate tiles (those holding a score above tau_0), first Phase-3 sweep over them
//                (f, f', f'' at tau_0, one safeguarded Halley/Newton step, working mask at tau_0)
//   out_kernel : Phase 4 (O = P V over the working mask), which is also the next evaluation of f;
//                further refinement only for rows that fail it; exported mask at the final tau
// One work-group = 32*QB*NW query rows of one head; wave w owns rows 32*QB*w .. of them as MFMA
// B operands in registers; 64-key tiles of K (and V) stream through LDS.
#pragma once
#include <type_traits>

#include "common.hpp"
#include "gather.hpp"
#include "histogram.hpp"

namespace ea {

// ---- pieces of the refinement (Sec. 3.2, Phase 3 of Alg. 1) shared by both forward kernels ----
// Accumulate sum y^r, sum y^(r-1), sum y^(r-2) over the scores of one sub-tile that lie above tau
// (alpha = 1.5: the last one is a count; alpha = 2: the middle one is).  Returns whether any did.
template <int AM, int QB>
EA_DEV bool eval_scores(const f32x16 (&C)[2][QB], const float (&thr)[QB], float c, float r, float (&F)[QB],
                        float (&G)[QB], float (&Hs)[QB], int (&cnt)[QB]) {
    bool hit = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        float lmax = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) lmax = fmaxf(lmax, C[kb][qb][v]);
        if (__any(fmaf(c, lmax, -thr[qb]) > 0.f)) {
            hit = true;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float y = fmaf(c, C[kb][qb][v], -thr[qb]);
                    if constexpr (AM == ALPHA_15) {
                        const float yp = fmaxf(y, 0.f);
                        F[qb] = fmaf(yp, yp, F[qb]);
                        G[qb] += yp;
                        cnt[qb] += (y > 0.f);
                    } else if constexpr (AM == ALPHA_20) {
                        F[qb] += fmaxf(y, 0.f);
                        cnt[qb] += (y > 0.f);
                    } else {
                        if (y > 0.f) {
                            const float p2 = pow_r2<AM>(y, r);
                            Hs[qb] += p2;
                            G[qb] = fmaf(p2, y, G[qb]);
                            F[qb] = fmaf(p2 * y, y, F[qb]);
                        }
                    }
                }
        }
    }
    return hit;
}

// Stopping length of the refinement at threshold tau: the caller's tolerance, but no less than four
// units in the last place of tau - fp32 thresholds of large scores (|tau| > 2 at tol = 1e-6) cannot
// move by less, and a row would otherwise iterate until its bracket has collapsed.
EA_DEV float step_tol(float tol, float tau) { return fmaxf(tol, 4.8e-7f * fabsf(tau)); }

// The iterate before the current one and its f, for the secant steps of alpha > 2; t is NaN while
// there is none (at the start of a kernel: the state is not carried from one kernel to the next).
struct SecantPrev { float t = __builtin_nanf(""), f = 0.f; };

// One safeguarded hybrid step from (tau, f = F - 1) with G = sum y^(r-1), Hs = sum y^(r-2):
// Halley for alpha <= 1.5, Newton for 1.5 < alpha <= 2, and for alpha > 2, where f' is unbounded
// next to every score (Prop. 2), a secant step through the last two iterates; the bracket's
// midpoint whenever the proposed point leaves (lo, hi) or does not exist (no earlier iterate, or
// f unchanged).  Updates the bracket; returns the proposed threshold.  tol: the callers' stopping
// length, used by the secant branch only.
template <int AM>
EA_DEV float hybrid_step(float tau, float f, float G, float Hs, float r, float alpha, float& lo, float& hi,
                         SecantPrev& prev, float tol) {
    if (f > 0.f) lo = tau; else hi = tau;
    const float f1 = -r * G;
    float delta;
    if (alpha <= 1.5f) {
        const float f2 = r * (r - 1.f) * Hs;
        delta = -2.f * f * f1 / (2.f * f1 * f1 - f * f2);
    } else {
        delta = -f / f1;
    }
    if constexpr (AM == ALPHA_GEN) {
        if (alpha > 2.f) {
            delta = -f * (tau - prev.t) / (f - prev.f);      // NaN or inf when there is no usable secant
            prev.t = tau; prev.f = f;
            // Callers stop when the step is shorter than tol.  Here a short step is no sign of
            // convergence (f rises vertically at every score, so a secant taken on its flat side
            // can be short far from the root): while the bracket is wider than tol such a step is
            // lengthened to 2 tol - either f changes sign, and the bracket is then no wider than
            // that, or the iterate has moved on by as much.  A step shorter than tol is then left
            // only inside a bracket narrower than tol, or as the half of one narrower than 2 tol.
            if (fabsf(delta) < tol && hi - lo >= tol) delta = f > 0.f ? 2.f * tol : -2.f * tol;
        }
    }
    float cand = tau + delta;
    if (!(cand > lo && cand < hi)) cand = 0.5f * (lo + hi);
    return cand;
}

template <class E, int D, int QB, int NB, int NW, int NBUF>
struct TauSmem {
    static constexpr int BR = 32 * QB * NW;
    static constexpr int MR = (BR + 63) / 64;
    // A row's histogram: NB bins per unit of (alpha-1) s on an absolute grid, of which the NB+1
    // bins that reach from one unit below the running maximum up to it are live, in a circular
    // buffer of SLOTS = NB+1 words (a power of two, so NB = 63).
    static constexpr int SLOTS = NB + 1;
    static_assert((SLOTS & (SLOTS - 1)) == 0 && SLOTS * 4 <= 256, "circular index is taken with a byte mask");
    // QB == 2: the two rows of a lane (n and n + 32 of its wave) share the words of one buffer,
    // 16 bits each, so the histograms of 256 rows take the LDS of 128; a bin then holds up to
    // 65535 keys, which the host guarantees by using this variant only while N < 65536.
    static_assert(QB == 1 || QB == 2, "one or two rows per lane");
    static constexpr int CBITS = 32 / QB;
    static constexpr int HIST_WORDS = 32 * NW * SLOTS;
};

template <class E, int D, int QB, int AM, int NB, int NW, int NBUF>
__global__ __launch_bounds__(NW * 64) void tau_kernel(Params p) {
    using SM = TauSmem<E, D, QB, NB, NW, NBUF>;
    using KT = RowTile<E, D>;
    constexpr int THREADS = NW * 64;
    using elem = typename E::elem;
    constexpr int BR = SM::BR, MR = SM::MR, SLOTS = SM::SLOTS;
    // All LDS is static, and the two K buffers are separate variables (see stream_tiles).
    __shared__ __align__(1024) char kbuf[KT::BYTES];
    __shared__ __align__(1024) char kbuf_b[NBUF == 2 ? KT::BYTES : 1024];
    __shared__ __align__(256) uint32_t hist[SM::HIST_WORDS];
    __shared__ uint32_t wm[MR * MAX_W];
    __shared__ uint32_t cand[MR * MAX_W];
    __shared__ int tl[MAX_T];
    __shared__ int tl_count[4];
    __shared__ unsigned long long blk_stats[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int N = p.N, T = p.T, W = p.W;
    int bh, I;
    map_block(blockIdx.x, p.BH, (N + BR - 1) / BR, bh, I);
    const long q0 = (long)I * BR, qw0 = q0 + wave * 32 * QB;
    const bool active = qw0 < N;          // N is a multiple of 64: the last group may be half empty
    if (p.oflag) {
        // run as the fallback of tau_list_kernel: only groups that hold a flagged 64-row block
        int flagged = 0;
        for (int i = 0; i < MR; ++i)
            if (I * MR + i < T) flagged |= p.oflag[(long)bh * T + (long)I * MR + i];
        if (!flagged) return;
    }
    _Float16* tmax_g = p.tmax + (long)bh * T * N;      // [T][N] per-row tile maxima, rounded up
    const elem* Qh = (const elem*)p.Q + (long)bh * N * D;
    const elem* Kh = (const elem*)p.K + (long)bh * N * D;
    const int njt = p.causal ? min((int)((q0 + BR) / 64), T) : T;          // tiles the group streams
    const int wjt = !active ? 0 : p.causal ? (int)((qw0 + 32 * QB - 1) / 64) + 1 : T;   // tiles this wave needs
    const int myrow = (wave * 32 * QB) / 64;                               // my mask row in the group
    const HeadConsts hc = head_consts(p, bh);
    const float c = hc.c, r = hc.r;

    Owned<E, D, QB> qf;
    load_owned<E, D, QB>(qf, Qh, active ? qw0 : 0, lane);
    for (int i = tid; i < MR * W; i += THREADS) { wm[i] = 0u; cand[i] = 0u; }
    for (int i = tid; i < SM::HIST_WORDS; i += THREADS) hist[i] = 0u;

    f32x16 C[2][QB];
    unsigned long long ntile_done = 0;
    char* const kbuf1 = NBUF == 2 ? kbuf_b : kbuf;
    auto issue_seq = [&](int it, char* buf) { issue_rows<E, D, NW>(buf, Kh, (long)it * 64, wave, lane); };
    auto scores = [&](int j, const char* buf) {
        stage1<E, D, QB>(C, buf, qf, lane);
        if (p.causal && (long)j * 64 + 63 > qw0) causal_hide<QB, true>(C, j * 64, (int)qw0, lane);
        ++ntile_done;
    };

    // ---- Phases 1 and 2 in one dense sweep: row maximum and histogram -------------------------
    // The histogram of Eq. 7-8 is centred on the row maximum, which a single sweep only knows at
    // its end.  Here the bins lie on an absolute grid instead (bin a holds NB x in [a, a+1), x =
    // (alpha-1) s), and a row keeps the window of bins from one unit below its running maximum
    // up to it: every score that can exceed tau* >= max - 1 (Eq. 5) is inside the window when it
    // is met, and stays inside as the maximum grows.  Prop. 1 only uses that a bin's left edge is
    // at most h below its scores, so its bounds hold on this grid as well.  When the maximum
    // moves up by k bins, the k slots that pass from the bottom of the window to its top are
    // cleared (by the row's first lane; LDS operations of one wave execute in program order).
    //
    // A score's slot, times 4, is the integer part of rel = 4 NB c s + k4 taken modulo 256, with
    // k4 = 4 (rot - a_lo): a_lo is the window's lowest bin and rot = a_lo mod SLOTS its slot.
    // The score is inside the window iff rel >= 4 rot.
    const float cb = c * NB, c4 = 4.f * cb;
    float run[QB], k4[QB], thr4[QB];
    int a_top[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) { run[qb] = -INFINITY; k4[qb] = 0.f; thr4[qb] = INFINITY; a_top[qb] = INT_MIN; }
    // Besides the running maximum, every (row, key tile) maximum goes to HBM (fp16, rounded up):
    // once tau_0 is known, only tiles holding a score above it can matter to f or to P.
    stream_tiles<NBUF>(njt, kbuf, kbuf1, issue_seq, [&](int j, const char* buf) {
        if (j >= wjt) return;
        scores(j, buf);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float gm[4];                            // maxima of the four groups of 8 registers
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                gm[g] = C[g >> 1][qb][8 * (g & 1)];
#pragma unroll
                for (int v = 1; v < 8; ++v) gm[g] = fmaxf(gm[g], C[g >> 1][qb][8 * (g & 1) + v]);
            }
            const float lm = fmaxf(fmaxf(gm[0], gm[1]), fmaxf(gm[2], gm[3]));
            const float tm = xhalf_max(lm);
            if (h == 0) tmax_g[(long)j * N + qw0 + 32 * qb + n] = (_Float16)(tm + fabsf(tm) * (1.f / 1024.f) + 1e-7f);
            const int row0 = wave * 32 * QB + 32 * qb;
            char* hrow = (char*)(hist + (wave * 32 + n) * SLOTS);
            const bool rise = tm > run[qb];
            if (__any(rise)) {                      // some row's maximum moves up
                int first = 0, last = -1;           // bins to clear: first..last (none)
                if (rise) {
                    run[qb] = tm;
                    int nt = (int)floorf(fminf(fmaxf(cb * tm, -1e9f), 1e9f));
                    int a_lo = nt - (SLOTS - 1), rot = a_lo & (SLOTS - 1);
                    float kk = 4.f * (float)(rot - a_lo);
                    // the maximum itself must land in the window's top slot, not wrap past it
                    if ((int)fmaf(c4, tm, kk) >= 4 * rot + 4 * SLOTS) {
                        nt += 1; a_lo += 1; rot = a_lo & (SLOTS - 1); kk = 4.f * (float)(rot - a_lo);
                    }
                    if (a_top[qb] != INT_MIN) { first = max(a_top[qb], nt - SLOTS) + 1; last = nt; }
                    a_top[qb] = nt; k4[qb] = kk; thr4[qb] = 4.f * (float)rot;
                }
                // the whole wave clears the slots of one rising row at a time: lane i takes slot i
                unsigned long long todo = __ballot(h == 0 && last >= first);
                while (todo) {
                    const int src = __ffsll((long long)todo) - 1;
                    todo &= todo - 1;
                    const int f0 = __builtin_amdgcn_readlane(first, src);
                    const int cnt = __builtin_amdgcn_readlane(last - first, src);
                    if (((lane - f0) & (SLOTS - 1)) <= cnt) {
                        uint32_t* word = hist + (wave * 32 + src) * SLOTS + lane;
                        if constexpr (QB == 1) *word = 0u;
                        else lds_and_b32(word, qb == 0 ? 0xffff0000u : 0x0000ffffu);
                    }
                }
            }
            if (__any(fmaf(c4, lm, k4[qb]) >= thr4[qb])) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if (!__any(fmaf(c4, gm[g], k4[qb]) >= thr4[qb])) continue;
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        const float rel = fmaf(c4, C[g >> 1][qb][8 * (g & 1) + v], k4[qb]);
                        if (rel >= thr4[qb]) lds_add_u32(hrow + ((int)rel & (4 * SLOTS - 4)), 1u << (SM::CBITS * qb & 31));
                    }
                }
            }
        }
    });
    lds_settle();
    // tau_0 = max(tau_h, max - 1) and the bracket [tau_0, tau_h + 1/NB] (Prop. 1, Eq. 5), raw units.
    // A wave reads only the histograms it filled itself: no barrier.  Lane (n, h) solves row block
    // qb = h of row n (with one row per lane, lane half 0 does), then the two lanes of a row swap.
    float thr[QB], blo[QB], bhi[QB];
    {
        constexpr float hb = 1.f / NB;
        const int sq = (QB == 2) ? h : 0;
        int top = a_top[0];
        float mx = run[0];
        if constexpr (QB == 2) { if (h) { top = a_top[1]; mx = run[1]; } }
        const int a_lo = top == INT_MIN ? 0 : top - (SLOTS - 1);
        const float origin = (float)a_lo * hb;                        // left edge of the window
        float gap;
        const float tau_h = solve_histogram<AM, SLOTS, SM::CBITS, QB == 1>(hist + (wave * 32 + n) * SLOTS, a_lo & (SLOTS - 1),
                                                                  SM::CBITS * sq & 31, hb, r, fmaf(c, mx, -1.f) - origin, gap) + origin;
        const float slack = 1e-6f + 2.5e-7f * fabsf(origin);          // fp32 rounding of bins and closed form
        const float my_t0 = fmaxf(tau_h - slack, fmaf(c, mx, -1.f));
        const float my_hi = tau_h + (hb + gap) + slack;
        const float o_t0 = xhalf_other(my_t0, h), o_hi = xhalf_other(my_hi, h);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const bool mine = (h == (QB == 2 ? qb : 0));
            thr[qb] = mine ? my_t0 : o_t0;
            blo[qb] = thr[qb];
            bhi[qb] = mine ? my_hi : o_hi;
            // right-edge binning moves every bin, and with it the root, up by one bin width: that
            // root, tau_h + h >= tau*, is the bracket's upper end, and it stands as the threshold
            if (active && h == 0) {
                p.rs_t0[(long)bh * N + qw0 + 32 * qb + n] = thr[qb];
                p.rs_up0[(long)bh * N + qw0 + 32 * qb + n] = bhi[qb];
            }
            if (p.right_edge) thr[qb] = bhi[qb];
        }
    }
    // candidate tiles of this wave's rows: those holding a score above tau_0.  64 tiles per
    // round: lane (n, h) looks at tiles j0 + 2u + h, u = 0..31, of row n, with all 32 loads in
    // flight together (one load at a time would string up to T/2 memory round trips).
    {
        float t0[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) t0[qb] = thr[qb];
        // (the tile maxima read below were stored by lanes of this same wave and are read here for
        // the first time: waiting for the wave's stores is enough, see tau_list_kernel)
        wait_loads();
        for (int j0 = 0; j0 < wjt; j0 += 64) {
            _Float16 tm[32][QB];
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                const int j = min(j0 + 2 * u + h, wjt - 1);        // clamped: tested against wjt below
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) tm[u][qb] = tmax_g[(long)j * N + qw0 + 32 * qb + n];
            }
            unsigned long long bits = 0;
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                bool cnd = false;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) cnd |= fmaf(c, (float)tm[u][qb], -t0[qb]) >= 0.f;
                cnd = cnd && (j0 + 2 * u + h < wjt);
                const unsigned long long bal = __ballot(cnd);
                if (bal & 0xffffffffull) bits |= 1ull << (2 * u);
                if (bal >> 32) bits |= 1ull << (2 * u + 1);
            }
            if (lane == 0) {
                const int w0 = j0 >> 5;
                if ((uint32_t)bits) atomicOr(&cand[myrow * W + w0], (uint32_t)bits);
                if (bits >> 32) atomicOr(&cand[myrow * W + w0 + 1], (uint32_t)(bits >> 32));
            }
        }
    }
    __syncthreads();
    build_tile_list(cand, MR, W, tl, tl_count, tid);
    auto issue_list = [&](int it, char* buf) { issue_rows<E, D, NW>(buf, Kh, (long)tl[it] * 64, wave, lane); };

    // ---- Phase 3: refinement sweeps; the first also records the working mask --------------
    // One evaluation of f, f', f'' at tau_0 over the candidate tiles and one safeguarded step;
    // the tiles that hold a score above tau_0 form the working mask.  Later evaluations ride on
    // Phase 4 (out_kernel).
    {
        float F[QB], G[QB], Hs[QB];
        int cnt[QB];      // number of scores above tau (alpha = 1.5: f'' sum; alpha = 2: f' sum)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) { F[qb] = G[qb] = Hs[qb] = 0.f; cnt[qb] = 0; }
        stream_tiles<NBUF>(*tl_count, kbuf, kbuf1, issue_list, [&](int it, const char* buf) {
            const int j = tl[it];
            if (!mask_bit(cand, W, myrow, j)) return;
            scores(j, buf);
            const bool hit = eval_scores<AM, QB>(C, thr, c, r, F, G, Hs, cnt);
            if (hit && lane == 0) atomicOr(&wm[myrow * W + (j >> 5)], 1u << (j & 31));
        });
        // threshold after this step, its bracket, f' at the point evaluated, and
        // (iterations | done << 16), for the output kernel; both lanes of a row compute the same
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            if constexpr (AM == ALPHA_15) Hs[qb] = (float)cnt[qb];
            if constexpr (AM == ALPHA_20) G[qb] = (float)cnt[qb];
            const float f = xhalf_sum(F[qb]) - 1.f, g = xhalf_sum(G[qb]), hs = xhalf_sum(Hs[qb]);
            bool done = fabsf(f) <= p.tol || p.right_edge;
            float tau = thr[qb];
            if (!done) {
                SecantPrev none;
                const float stol = step_tol(p.tol, tau);
                const float cand_tau = hybrid_step<AM>(tau, f, g, hs, r, hc.alpha, blo[qb], bhi[qb], none, stol);
                done = fabsf(cand_tau - tau) < stol;
                tau = cand_tau;
            }
            if (active && h == 0) {
                const long gi = (long)bh * N + qw0 + 32 * qb + n;
                p.tau[gi] = tau;
                p.rs_lo[gi] = blo[qb];
                p.rs_hi[gi] = bhi[qb];
                p.rs_state[gi] = 1 | ((int)done << 16);
                p.rs_f1[gi] = -r * g;
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < MR * W; i += THREADS)
        if (I * MR + i / W < T) p.wmask[((long)bh * T + (long)I * MR + i / W) * W + (i % W)] = (int32_t)wm[i];
    {
        const int slot[2] = {0, 5};
        const unsigned long long val[2] = {ntile_done * QB, wave == 0 ? 1ull : 0ull};
        flush_counters<2>(blk_stats, p.stats, slot, val, tid, lane);
    }
}

// ---- threshold kernel with candidate lists -----------------------------------------------------
// Phases 1-3 of Alg. 1 from ONE dense sweep.  By Eq. 5, tau* >= max - 1 (in units of (alpha-1) s),
// and both the maximum and tau* over a prefix of the keys are at most their values over all keys,
// so a score that lies below a lower bound of the prefix's threshold when it is met can never lie
// above the final one.  Every other score - a handful per row when attention is sparse - is listed, with
// its key, by the lane that computed it (each lane sees 16 of every 32 keys of its row, so
// a row has two lists; no atomics, no ordering between lanes).  The lower bound starts as (running maximum - 1);
// when it is refreshed (see below), the row's LDS histogram of the listed scores (Eq. 6-8;
// absolute bin grid with a sliding window, as in tau_kernel) is solved (Eq. 9), and its root tau_h, a lower
// bound of the prefix's tau* by Prop. 1, becomes the new bound.  Scores that were skipped lie below the bound and
// contribute nothing to f at or above it, so f there, and with it Prop. 1, is that of all scores.
// After the sweep the lists hold a superset of the row's support as exact fp32 scores, and the
// rest happens on them: the refinement iterations of Sec. 3.2 from tau_0 = tau_h, each an
// evaluation of f, f', f'' over the listed true scores instead of another sweep of Q K^T.  The key
// tiles of the entries above tau_0 are the working mask.
// The histogram is made from the lists, by a wave's lanes side by side, when the bound is refreshed: after 4, 8, 16, ...
// tiles, if a list has grown enough since - all waves of a work-group at the same tile, as each of them holds up the
// others at the next barrier.  Rows whose first tile shows that their lists will be long are counted entry by entry instead.
// Bound: instructions issued, about 4 clocks of a SIMD for one of whatever kind (sigma = 1: 515 a tile and wave, 9000 clocks
// for the four waves of a SIMD; sigma = 3: 190 and 3700), most of them for candidates where there are many: some lane has one in 15 of a
// tile's 32 score registers at sigma = 1, though only two of the 64 lanes in each.  Such a register takes 8 instructions
// (14 if counted; 13 and 17 as the compiler puts it), one without 2, and a tile without candidates about 90, of which 32 are the products and
// their reads.  Forward, steps: 1088 tokens, d = 64, 87 -> 71 us; 4096 tokens 464 -> 428; 8192 tokens, alpha = 1.25, 787 -> 725; 3136 tokens,
// d = 128, 153 -> 142; 65536 tokens 3600 -> 3490; 16384 tokens, sigma = 1, level (2515: its list stores are what memory takes).
// A list that fills up (attention close to uniform: hundreds of non-zeros per row) flags its 64-row
// block; flagged blocks are redone by the sweep-based tau_kernel, which runs right after and exits
// at once everywhere else.
template <class E, int D, int AM, int NB, int NW, int NBUF>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW == 8 ? 4 : 1))) void tau_list_kernel(Params p) {
    using SM = TauSmem<E, D, 1, NB, NW, NBUF>;
    using KT = RowTile<E, D>;
    using elem = typename E::elem;
    constexpr int THREADS = NW * 64, BR = SM::BR, MR = SM::MR, SLOTS = SM::SLOTS;
    constexpr int LIST_STEP = 8;
    // List growth (entries of any lane) since the last refresh of the bound from which the next scheduled one is done, and
    // from which one is done at once (GROW_COUNTING: of lists counted as they grow).  Steps with GROW 12 / 24 / 48 / 64:
    // forward of 1088 tokens, d = 64, 75 / 77 / 71 / 70 us, 3136 tokens, sigma = 2, 164 / 155 / 142 / 142, 4096 tokens 414 / 423 / 425 / 442.
    // GROW_COUNTING 12 / 20 / 32: alpha = 2, 8192 tokens, d = 64, sigma = 0.6, 706 / 723 / 745 us, 64 heads of 2048, sigma = 0.8, 368 / 369 / 378, fp32, 1024
    // tokens, 134 / 131 / 130, 16384 tokens, sigma = 1, 2350 / 2345 / 2383.  GROW_HARD 48 / 64 / 96: 4096 tokens 446 / 407 / 401, alpha = 1.25, 8192 tokens,
    // 756 / 717 / 689, 1088 tokens 75 / 69 / 69.  The first scheduled refresh after 4 or 8 tiles: level.
    constexpr int GROW = 48, GROW_COUNTING = 20, GROW_HARD = 64, FIRST_REFRESH = 4;
    // list length from which on a refresh drops entries below the bound (it takes two passes over memory: later where
    // the histogram needs no pass of its own; 16384 tokens, sigma = 1, 144 / 208: 2600 / 2546 us;
    // PRUNE_FROM 144 or 192: level at alpha = 1.25, 1.5 and 2, few lists of sparse rows come that far)
    constexpr int PRUNE_FROM = 144, PRUNE_FROM_COUNTING = 208;
    // ... and only while the row with most keys of support so far, and the count that it will grow to if it keeps rising with the
    // logarithm of the keys seen, leave room in the lists: a prune of every wave costs as much as the fallback kernel, and one that drops
    // little only puts the overflow off; where the lists hold out in the end a few rows in the fallback kernel cost all its time.  Forward, d = 64, pruned
    // always / by this rule / never: 32 heads of 4096 tokens, alpha = 1.5, sigma = 0.4, 3310 / 2090 / 1350 us, 64 of 2048 without a mask 3410 / 1280 / 1100,
    // alpha = 1.25, sigma = 1.2, 2600 / 1760 / 1460, 1.5, 695 / 686 / 1175, 64 of 4096, alpha = 1.25, sigma = 1.5, 1245 / 1253 / 1808, 8 of 16384,
    // sigma = 0.7, 1260 / 1258 / 2390.  With (352, 576) instead: 1800, 1180, 1520, 680, 1790 and 1260, and d = 128, alpha = 1.25,
    // sigma = 1.4, 1500 against 930; with (416, 640): 2265, 2747, 1888, 698, 1250 and 1260.
    constexpr int PRUNE_SUPPORT = 416;
    constexpr float PRUNE_SUPPORT_END = 576.f;
    // prunes of a wave at most: what they drop stays counted.  (A list that is full after them flags its block, as any other.)
    constexpr int MAX_PRUNES = 120;
    // Groups of eight scores of a wave's first tile (of 256) with a candidate from which its entries are counted as they are
    // listed: long lists then need no pass to be counted.  112 / 180 / 230 / never: 4096 tokens, sigma = 1.5, 531 / 428 / 425 / 425,
    // 16384 tokens, sigma = 1, 2530 / 2530 / 2600 / 3300 us.
    constexpr int FIRST_TILE_BUSY = 180;
    constexpr int TILE_ENTRIES = 32;     // entries a lane can list from one tile
    // entries per lane held in registers after the sweep (8 / 16: 4096 tokens 413 / 407 us, alpha = 2, sigma = 0.6, 8192 tokens 729 / 723, 1088 tokens 70.4 / 69.5)
    constexpr int REG_ENTRIES = 16;
    // counters: waves 2w and 2w + 1 share the words of one histogram buffer, 16 bits each.  A row counts what its two lists
    // hold in the end and what prunes dropped from them.
    constexpr int CB = 16;
    static_assert(NW % 2 == 0 && 2 * LIST_CAP * (MAX_PRUNES + 1) < 65536, "a counter holds what a row can count");
    constexpr int RING_BYTES = NBUF * KT::BYTES, HIST_BYTES = NW / 2 * 32 * SLOTS * 4;
    __shared__ __align__(1024) char lds[RING_BYTES + HIST_BYTES];
    char* const kring = lds;
    uint32_t* const hist = (uint32_t*)(lds + RING_BYTES);
    // used only once the sweep is over: in place of the ring
    constexpr int POST_BYTES = 2 * MR * MAX_W * 4 + ((MR * 4 + 7) & ~7) + 48;
    static_assert(POST_BYTES <= RING_BYTES, "post-sweep arrays must fit in the ring");
    uint32_t* const wm = (uint32_t*)lds;                          // working mask (tiles above tau_0)
    uint32_t* const fmk = wm + MR * MAX_W;                        // final mask (tiles of the support)
    int* const over_s = (int*)(fmk + MR * MAX_W);
    int* const gsum = (int*)((char*)over_s + ((MR * 4 + 7) & ~7));   // [1] support size, [2] obstacles
    unsigned long long* const blk_stats = (unsigned long long*)(gsum + 4);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int N = p.N, T = p.T, W = p.W;
    int bh, I;
    map_block(blockIdx.x, p.BH, (N + BR - 1) / BR, bh, I);
    const long q0 = (long)I * BR, qw0 = q0 + wave * 32;
    const bool active = qw0 < N;
    const elem* Qh = (const elem*)p.Q + (long)bh * N * D;
    const elem* Kh = (const elem*)p.K + (long)bh * N * D;
    const int njt = p.causal ? min((int)((q0 + BR) / 64), T) : T;
    int wjt = !active ? 0 : p.causal ? (int)((qw0 + 31) / 64) + 1 : T;      // tiles this wave works on
    const int jdiag = p.causal ? (int)(qw0 / 64) : T;     // the first tile that holds keys past a row of this wave
    const int myrow = (wave * 32) / 64;
    const HeadConsts hc = head_consts(p, bh);
    const float c = uniform(hc.c), r = uniform(hc.r), alpha = uniform(hc.alpha);     // (in scalar registers)
    constexpr float hb = 1.f / NB;

    Owned<E, D, 1> qf;
    load_owned<E, D, 1>(qf, Qh, active ? qw0 : 0, lane);
    for (int i = tid; i < HIST_BYTES / 4; i += THREADS) hist[i] = 0u;      // (the walk begins with a barrier)

    // this lane's list: 8-byte entries at lists_w + list0()
    char* const lists_w = (char*)p.lists + ((size_t)bh * N + (active ? qw0 : 0)) * (size_t)(2 * LIST_CAP * 8);
    const uint64_t lists_u = uniform_address(lists_w);
    auto list0 = [] {                                    // (formed anew where it is wanted: no register of the sweep's)
        const int l = lane_id_opaque();
        return (uint32_t)((l & 31) * 2 + (l >> 5)) * (uint32_t)(LIST_CAP * LIST_STEP);
    };
    uint32_t at = list0();                               // where the next entry goes
    uint32_t trig = GROW * LIST_STEP, trig_hard = GROW_HARD * LIST_STEP;    // list lengths from which on the bound is refreshed
    auto entries = [&] { return (int)((at - list0()) / (uint32_t)LIST_STEP); };      // (more than LIST_CAP: entries were lost)
    auto load_entries = [&](auto& e, int i0, int cnt) __attribute__((always_inline)) {      // entries from i0 on, i0 even (-inf past the list's end)
        constexpr int K = sizeof(e) / sizeof(e[0]);
        const char* const l = lists_w + (list0() + (uint32_t)i0 * (uint32_t)LIST_STEP);
#pragma unroll
        for (int u = 0; u < K; u += 2) {
            uint4 x = make_uint4(0xff800000u, 0u, 0xff800000u, 0u);
            if (i0 + u < cnt) x = *(const uint4*)(l + u * LIST_STEP);
            e[u] = make_uint2(x.x, x.y);
            e[u + 1] = make_uint2(i0 + u + 1 < cnt ? x.z : 0xff800000u, x.w);
        }
    };
    auto store_entry = [&](uint32_t to, uint2 e) { *(uint2*)(lists_w + to) = e; };
    int a_top = INT_MIN;
    float run = -INFINITY, low = -3.0e38f, lowraw = -3.0e38f;     // running maximum, lower bound, root of the histogram so far (raw scores)
    const int hshift = 16 * (wave & 1);
    uint32_t* const hrow = hist + ((wave >> 1) * 32 + n) * SLOTS;
    const uint32_t hrow_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const uint32_t*)hrow;
    const float inv_c = uniform(1.f / c), cb = uniform(c * NB), c4 = uniform(4.f * cb);
    float k4 = 0.f, bottom4 = 0.f, top_raw = -INFINITY;

    // Root of the row's histogram (Eq. 9) as it stands (both lanes of a row hold the same): tau_0 =
    // max(tau_h, max - 1) less the fp32 slack, and the bracket's upper end.
    // (`support`, the counts above it: while the sweep runs only a lower bound is wanted; for general alpha, whose exact
    // solve takes power functions per bin, the closed-form bound then stands in for the root)
    auto histogram_bound = [&](float& lo, float& up, int* support) {
        lds_settle();
        const int a_lo = a_top == INT_MIN ? 0 : a_top - (SLOTS - 1);
        const float origin = (float)a_lo * hb;                        // left edge of the window
        float tau_h, gap = 0.f;
        if (AM == ALPHA_GEN && support)
            tau_h = histogram_lower_bound<SLOTS, CB, true>(hrow, a_lo & (SLOTS - 1), hshift, hb, r, support) + origin;
        else
            tau_h = solve_histogram<AM, SLOTS, CB, true>(hrow, a_lo & (SLOTS - 1), hshift, hb, r, fmaf(c, run, -1.f) - origin, gap, support) + origin;
        const float slack = 1e-6f + 2.5e-7f * fabsf(origin);          // fp32 rounding of bins and closed form
        lo = fmaxf(tau_h - slack, fmaf(c, run, -1.f));
        up = tau_h + (hb + gap) + slack;
    };

    // The window of live bins follows the running maximum (see tau_kernel).  Bins below the bound are of no
    // use, so the window is moved up by as many bins more as the bound leaves free at its bottom: most
    // of the maxima that follow then fall inside it, and slots are cleared a few times per row only.
    auto move_window = [&] {
        int first = 0, last = -1;                       // bins to clear: first..last (none)
        if (run > top_raw) {
            int nt = (int)floorf(fminf(fmaxf(cb * run, -1e9f), 1e9f));
            const int spare = (int)floorf(fminf(fmaxf(cb * lowraw, -1e9f), 1e9f)) - 1 - (nt - (SLOTS - 1));
            nt += min(max(spare, 0), SLOTS / 2);
            int a_lo = nt - (SLOTS - 1), rot = a_lo & (SLOTS - 1);
            float kk = 4.f * (float)(rot - a_lo);
            // the maximum itself must land in the window's top slot, not wrap past it
            if ((int)fmaf(c4, run, kk) >= 4 * rot + 4 * SLOTS) {
                nt += 1; a_lo += 1; rot = a_lo & (SLOTS - 1); kk = 4.f * (float)(rot - a_lo);
            }
            if (a_top != INT_MIN) { first = max(a_top, nt - SLOTS) + 1; last = nt; }
            a_top = nt; k4 = kk; bottom4 = (float)(4 * rot);
            // scores up to here lie in the window for certain (less than half a bin from its top edge)
            top_raw = fmaxf(run, ((float)nt + 0.5f) * (hb * inv_c));
        }
        // the whole wave clears the slots of one rising row at a time: lane i takes slot i
        unsigned long long todo = __ballot(h == 0 && last >= first);
        while (todo) {
            const int src = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            const int f0 = __builtin_amdgcn_readlane(first, src);
            const int ncl = __builtin_amdgcn_readlane(last - first, src);
            if (((lane - f0) & (SLOTS - 1)) <= ncl) lds_and_b32(hist + ((wave >> 1) * 32 + src) * SLOTS + lane, ~(0xffffu << hshift));
        }
    };
    bool counting = false;                               // the same for all lanes: entries are counted as they are listed
    // What the lists hold beyond the first `counted` entries, counted in the histogram
    int counted = 0;
    auto count_lists = [&] {
        if (counting) return;
        if (__any(run > top_raw)) move_window();
        const uint32_t one = 1u << hshift;
        const int cnt = min(entries(), LIST_CAP), from = counted & ~1, most = wave_max(cnt - from);
        wait_loads();                                   // this wave's stores have completed
#pragma unroll 1
        for (int i0 = 0; i0 < most; i0 += 16) {
            uint2 e[16];
            load_entries(e, from + i0, cnt);
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const float rel = fmaf(c4, __uint_as_float(e[u].x), k4);
                // (an entry further than one unit below the maximum is below the window, and of no use)
                if (rel >= bottom4 && (u > 0 || i0 > 0 || from == counted)) lds_add_at(hrow_lds + ((uint32_t)(int)rel & (4 * SLOTS - 4)), one);
            }
        }
        counted = max(counted, cnt);
    };

    f32x16 C[2][1];
    float gm[4], lm;
    // scores of tile j and the maxima of the four groups of 8 registers and of the lane
    auto tile_scores = [&](int j, const char* buf) {
        stage1<E, D, 1, EA_FENCE, NW == 8 ? 0 : 8>(C, buf, qf, lane);
        if (j >= jdiag) causal_hide<1, true>(C, j * 64, (int)qw0, lane);
        settle_vec<E>(C[0][0], C[1][0]);
#pragma unroll
        for (int g = 0; g < 4; ++g) gm[g] = max8_raw(C[g >> 1][0], 8 * (g & 1));
        lm = max2_raw(max3_raw(gm[0], gm[1], gm[2]), gm[3]);
    };
    bool listed = false, tight = false;                  // the same for all lanes: lists have grown; two tiles may fill one
    // candidates: raw scores at or above the row's current lower bound; most tiles of a sparse row block hold none
    auto list_tile = [&](int j) {
        if (!__any(lm >= low)) return;                   // (nor does the maximum move: low <= run)
        __builtin_amdgcn_s_setprio(3);                   // (the others of the group wait for the wave with most candidates)
        run = max2_raw(run, xhalf_max(lm));
        low = max2_raw(run - inv_c, lowraw);
        const uint32_t key0 = (uint32_t)(j * 64 + 8 * h);
        if (j == 0) {
            // many candidates in the first tile: lists will be long
            int busy = 0;
#pragma unroll
            for (int g = 0; g < 4; ++g) busy += __popcll(__ballot(gm[g] >= low));
            counting = busy >= FIRST_TILE_BUSY;
            if (counting) trig_hard = GROW_COUNTING * LIST_STEP;
        }
        auto scan = [&](auto count) __attribute__((always_inline)) {
            unroll_steps<4>([&](auto g) __attribute__((always_inline)) {
                constexpr int G = decltype(g)::value;
                if (!__any(gm[G] >= low)) return;
                // tile row of register v of group g: see causal_hide
                unroll_steps<8>([&](auto v) __attribute__((always_inline)) {
                    constexpr int V = decltype(v)::value, OFF = 32 * (G >> 1) + 16 * (G & 1) + V;
                    const float sc = C[G >> 1][0][8 * (G & 1) + V];
                    if constexpr (decltype(count)::value) list_and_count_candidate<OFF>(sc, low, key0, at, lists_u, c4, k4, bottom4, hrow_lds, 4 * SLOTS - 4, 1u << hshift);
                    else list_candidate<OFF>(sc, low, key0, at, lists_u);
                });
            });
        };
        if (tight) {
            // (a full list keeps overwriting its last entry: its block is redone anyway)
            if (counting && __any(run > top_raw)) move_window();
            const uint32_t last = list0() + (uint32_t)((LIST_CAP - 1) * LIST_STEP);
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const float sc = C[g >> 1][0][8 * (g & 1) + v];
                    if (sc >= low) {
                        store_entry(min(at, last), make_uint2(__float_as_uint(sc), key0 + 32 * (g >> 1) + 16 * (g & 1) + v));
                        const float rel = fmaf(c4, sc, k4);
                        if (counting && at <= last && rel >= bottom4) lds_add_at(hrow_lds + ((uint32_t)(int)rel & (4 * SLOTS - 4)), 1u << hshift);
                        at += LIST_STEP;
                    }
                }
        } else if (counting) {
            if (__any(run > top_raw)) move_window();
            scan(std::true_type{});
        } else scan(std::false_type{});
        listed = true;
        __builtin_amdgcn_s_setprio(0);
    };
    int prunes = 0;
    // a better lower bound from the histogram so far, after `tiles` tiles
    auto refresh = [&](int tiles) {
        count_lists();
        float lo, up;
        int support;
        histogram_bound(lo, up, &support);
        const float braw = lo * inv_c;
        lowraw = braw - fabsf(braw) * 1e-6f;
        low = max2_raw(low, lowraw);
        int cnt = entries(), most = wave_max(cnt);
        if (most > LIST_CAP) { wjt = tiles; return; }    // the block is redone: nothing more is listed
        auto room = [&] {
            const int s = wave_max(support);
            return s <= PRUNE_SUPPORT && (float)s * (1.f + 0.69f * __builtin_amdgcn_logf((float)wjt / (float)tiles)) <= PRUNE_SUPPORT_END;
        };
        if (most > (counting ? PRUNE_FROM_COUNTING : PRUNE_FROM) && prunes < MAX_PRUNES && room()) {
            ++prunes;
            // long lists: entries below the bound are dropped, the others move to the front in their order (counted they stay:
            // bins below the histogram's root have no part in it, nor in the root of any later one)
            uint32_t front = list0();
#pragma unroll 1
            for (int i0 = 0; i0 < most; i0 += 8) {
                uint2 e[8];
                load_entries(e, i0, cnt);
                // (all eight are in registers before the first is overwritten)
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (__uint_as_float(e[u].x) >= low) { store_entry(front, e[u]); front += LIST_STEP; }
            }
            at = front;
            cnt = counted = entries();
            most = wave_max(cnt);
        }
        trig = (uint32_t)(most + GROW) * LIST_STEP;
        // (the two tiles before the next look at the lists add up to TILE_ENTRIES each)
        tight = most > LIST_CAP - 3 * TILE_ENTRIES;
        trig_hard = (uint32_t)min(most + (counting ? GROW_COUNTING : GROW_HARD), LIST_CAP + 1) * LIST_STEP;
        if (!tight) trig_hard = min(trig_hard, (uint32_t)(LIST_CAP - 2 * TILE_ENTRIES + 1) * LIST_STEP);
    };
    // Tile it + 1 is loaded under the scores of tile it and waited for before the tile's candidates are listed: the
    // wait covers list stores of tile it - 1, which have had the tile's matrix products to complete, and none of its own.
    {
        auto issue = [&](int it) { issue_rows<E, D, NW>(kring + (it % NBUF) * KT::BYTES, Kh, (long)it * 64, wave, lane); };
        static_assert(NBUF == 2, "double buffer");
        if (njt > 0) issue(0);
        wait_vm_at_most<0>();
        __syncthreads();
        auto step = [&](int it, const char* buf) __attribute__((always_inline)) {
            if (it + 1 < njt) issue(it + 1);             // (everyone is done with tile it - 1)
            if (it < wjt) tile_scores(it, buf);
            sched_fence();
            wait_vm_at_most<0>();
            if (it < wjt) list_tile(it);
            __syncthreads();                             // tile it + 1 has landed for every wave
        };
        auto look = [&](int tiles) __attribute__((always_inline)) {      // after every second tile
            if (!listed || tiles >= wjt) return;
            listed = false;
            const bool scheduled = tiles >= FIRST_REFRESH && (tiles & (tiles - 1)) == 0;
            if (__any(at - list0() >= (scheduled ? min(trig, trig_hard) : trig_hard))) refresh(tiles);
        };
        if constexpr (D == 128 && E::EPL == 8) {
            // (two tiles a turn: the buffers' addresses are then constants, 8 instructions a tile; at d = 64 it is 4, and
            // the code of one tile body less to fetch counts for more in short sequences)
            for (int it = 0; it < njt; it += 2) {
                step(it, kring);
                if (it + 1 >= njt) break;
                step(it + 1, kring + KT::BYTES);
                look(it + 2);
            }
        } else {
            for (int it = 0; it < njt; ++it) {
                step(it, kring + (it & 1) * KT::BYTES);
                if (it & 1) look(it + 1);
            }
        }
    }
    for (int i = tid; i < MR * W; i += THREADS) { wm[i] = 0u; fmk[i] = 0u; }
    if (tid < MR) over_s[tid] = 0;
    if (tid < 4) gsum[tid] = 0;
    __syncthreads();
    // The lists are read back by the lanes that wrote them and by no others: a wave's vector memory operations
    // on one address take effect in program order, so no fence is needed.  A device-scope fence here writes the
    // whole L2 back once per work-group, which cost 0.1 - 0.4 ms per launch.
    wait_loads();

    // ---- solve and refinement on the lists -----------------------------------------------------
    float thr = 0.f, thr0 = 0.f;
    int over = 0, iters = 0, done = 1, mycnt = 0, nmax = 0;
    uint2 ent[REG_ENTRIES];
    bool in_regs = false;
    // body(score, key) for every listed entry, and for some past the list's end with a score of -inf
    auto from_regs = [&](auto&& body) __attribute__((always_inline)) {
        unroll_steps<REG_ENTRIES / 8>([&](auto b) __attribute__((always_inline)) {
            constexpr int I0 = 8 * decltype(b)::value;
            if (I0 >= nmax) return;
#pragma unroll
            for (int u = 0; u < 8; ++u) body(__uint_as_float(ent[I0 + u].x), ent[I0 + u].y);
        });
    };
    auto from_memory = [&](auto&& body) __attribute__((always_inline)) {
#pragma unroll 1
        for (int i0 = 0; i0 < nmax; i0 += 16) {
            uint2 e[16];
            load_entries(e, i0, mycnt);
            // (all sixteen are in registers before a body stores the first)
#pragma unroll
            for (int u = 0; u < 16; ++u) body(__uint_as_float(e[u].x), e[u].y);
        }
    };
    if (active) {
        float blo, bhi;
        over = entries() > LIST_CAP;
        mycnt = min(entries(), LIST_CAP);
        nmax = wave_max(mycnt);
        in_regs = nmax <= REG_ENTRIES;
        if (in_regs) load_entries(ent, 0, mycnt);
        if (in_regs && !counting && !__any(counted)) {
            if (__any(run > top_raw)) move_window();
            const uint32_t one = 1u << hshift;
            from_regs([&](float sc, uint32_t) {
                const float rel = fmaf(c4, sc, k4);
                if (rel >= bottom4) lds_add_at(hrow_lds + ((uint32_t)(int)rel & (4 * SLOTS - 4)), one);
            });
        } else count_lists();
        histogram_bound(thr0, bhi, nullptr);
        if (h == 0) {
            p.rs_t0[(long)bh * N + qw0 + n] = thr0;
            p.rs_up0[(long)bh * N + qw0 + n] = bhi;
        }
        float f1_last = -1.f;
        blo = thr0;
        thr = p.right_edge ? bhi : thr0;      // tau_h + h >= tau*: the right-edge root, taken as it is
        done = 0;
        // refinement (Sec. 3.2): evaluations of f, f', f'' over the listed scores.  Lists in memory: the first
        // evaluation, at tau_0 <= tau* (every later threshold lies above it), moves the entries it
        // finds above the threshold to the front of their list, and those that follow read a fraction of it.
        SecantPrev prev;
        // (alpha > 2: a row with a score within the tolerance of its root ends up bisecting, since f
        // rises vertically there; the sweeps over the lists are cheap, those of the output kernel
        // are not, so the limit is doubled here)
        const int nsweeps = r < 1.f ? 2 * p.max_sweeps : p.max_sweeps;
        for (int sweep = 0; sweep < nsweeps; ++sweep) {
            float F = 0.f, G = 0.f, Hs = 0.f;
            auto eval = [&](float sc) {
                const float y = fmaf(c, sc, -thr);
                if constexpr (AM == ALPHA_15) { const float yp = fmaxf(y, 0.f); F = fmaf(yp, yp, F); G += yp; Hs += y > 0.f ? 1.f : 0.f; }
                else if constexpr (AM == ALPHA_20) { F += fmaxf(y, 0.f); G += y > 0.f ? 1.f : 0.f; }
                else if (y > 0.f) {
                    const float p2 = pow_r2<AM>(y, r);
                    Hs += p2; G = fmaf(p2, y, G); F = fmaf(p2 * y, y, F);
                }
                return y > 0.f;
            };
            if (in_regs) from_regs([&](float sc, uint32_t) { eval(sc); });
            else {
                uint32_t front = list0(), lastj = 0xffffffffu;
                from_memory([&](float sc, uint32_t key) {
                    if (eval(sc) && sweep == 0) {
                        store_entry(front, make_uint2(__float_as_uint(sc), key));
                        front += LIST_STEP;
                        const uint32_t j = key >> 6;                  // its tiles are the working mask
                        if (j != lastj) { atomicOr(&wm[myrow * W + (j >> 5)], 1u << (j & 31)); lastj = j; }
                    }
                });
                if (sweep == 0) {
                    mycnt = (int)((front - list0()) / (uint32_t)LIST_STEP); nmax = wave_max(mycnt);
                    in_regs = nmax <= REG_ENTRIES;
                    if (in_regs) load_entries(ent, 0, mycnt);
                }
            }
            const float f = xhalf_sum(F) - 1.f, g = xhalf_sum(G), hs = xhalf_sum(Hs);
            if (!done) {
                iters += 1;
                f1_last = -r * g;
                if (fabsf(f) <= p.tol || p.right_edge) done = 1;
                else {
                    const float stol = step_tol(p.tol, thr);
                    const float cand_tau = hybrid_step<AM>(thr, f, g, hs, r, alpha, blo, bhi, prev, stol);
                    if (fabsf(cand_tau - thr) < stol) done = 1;
                    thr = cand_tau;
                }
            }
            if (!__any(!done)) break;
        }
        if (h == 0) {
            const long gi = (long)bh * N + qw0 + n;
            p.tau[gi] = thr;
            p.rs_lo[gi] = blo;
            p.rs_hi[gi] = bhi;
            p.rs_state[gi] = iters | (done << 16);
            p.rs_f1[gi] = f1_last;
        }
    }
    if (__any(over) && lane == 0) atomicOr(&over_s[myrow], 1);

    // ---- sparse row groups: the support itself, for the gather kernel ---------------------------
    // The entries above the final tau - the row's support, a handful of keys - are moved to the front of their
    // list, with their key indices; gather_out_kernel then forms O from those rows of V alone, and the
    // block-sparse output kernel skips the row group.
    if (__any(over || !done) && lane == 0) atomicOr(&gsum[2], 1);
    __syncthreads();
    const int nrows = min(BR, N - (int)q0);
    const bool sparse = p.gflag && gsum[2] == 0;
    if (sparse) {
        int w = 0;
        if (active) {
            uint32_t front = list0();
            uint32_t lastj = 0xffffffffu;
            auto keep = [&](float sc, uint32_t key) {
                if (fmaf(c, sc, -thr) > 0.f) {
                    store_entry(front, make_uint2(__float_as_uint(sc), key));
                    front += LIST_STEP;
                    const uint32_t j = key >> 6;
                    if (j != lastj) { atomicOr(&fmk[myrow * W + (j >> 5)], 1u << (j & 31)); lastj = j; }
                }
            };
            if (in_regs) from_regs(keep); else from_memory(keep);
            w = (int)((front - list0()) / (uint32_t)LIST_STEP);
            p.scnt[((long)bh * N + qw0 + n) * 2 + h] = w;
        }
        int nsup = w;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) nsup += __shfl_xor(nsup, off);
        if (lane == 0) atomicAdd(&gsum[1], nsup);
    }
    __syncthreads();
    const bool gather = sparse && gsum[1] <= GATHER_SUP_MAX * nrows;
    if (!gather && active && in_regs) {
        uint32_t lastj = 0xffffffffu;
        from_regs([&](float sc, uint32_t key) {
            const uint32_t j = key >> 6;
            if (fmaf(c, sc, -thr0) > 0.f && j != lastj) { atomicOr(&wm[myrow * W + (j >> 5)], 1u << (j & 31)); lastj = j; }
        });
    }
    if (blockIdx.x == 0 && tid == 0) p.scal[2] = p.gflag ? (unsigned int)BR : 0u;     // (0: no flags were written)
    if (p.gflag && tid == 0) {
        p.gflag[(long)bh * ((N + BR - 1) / BR) + I] = gather;
        if (!gather) atomicAdd(&p.scal[1], 1u);       // a row group out_kernel will have to serve
    }
    if (gather) {
        if (active && h == 0 && p.iters) p.iters[(long)bh * N + qw0 + n] = iters;
        for (int i = tid; i < MR * W; i += THREADS)
            if (I * MR + i / W < T) p.mask[((long)bh * T + (long)I * MR + i / W) * W + (i % W)] = (int32_t)fmk[i];
    } else {
        __syncthreads();
        for (int i = tid; i < MR * W; i += THREADS)
            if (I * MR + i / W < T) p.wmask[((long)bh * T + (long)I * MR + i / W) * W + (i % W)] = (int32_t)wm[i];
    }
    if (tid < MR && I * MR + tid < T) p.oflag[(long)bh * T + (long)I * MR + tid] = over_s[tid];
    {
        int nover = 0;
        if (tid == 0)
            for (int i = 0; i < MR; ++i) nover += over_s[i];
        const int slot[3] = {0, 8, 9};
        const unsigned long long val[3] = {(unsigned long long)min(wjt, njt), (unsigned long long)nover, (tid == 0 && gather) ? (unsigned long long)nrows : 0ull};
        flush_counters<3>(blk_stats, p.stats, slot, val, tid, lane);
    }
}

template <class E, class E2, int D, int QB, bool MASK_ONLY, int NW, int NBUF>
struct OutSmem {
    static constexpr int BR = 32 * QB * NW;
    static constexpr int MR = (BR + 63) / 64;
    static constexpr int KBYTES = RowTile<E, D>::BYTES;
    static constexpr int VBYTES = MASK_ONLY ? 0 : RowTile<E2, D>::BYTES;
    static constexpr int SET = KBYTES + VBYTES;              // one buffer set (static LDS)
};

// Phase 4.  MASK_ONLY: no V, no O - only the mask at the given tau (used by the backward when
// the caller passes no mask).
template <class E, class E2, int D, int QB, int AM, bool MASK_ONLY, int NW, int NBUF>
__global__ __launch_bounds__(NW * 64) void out_kernel(Params p) {
    using SM = OutSmem<E, E2, D, QB, MASK_ONLY, NW, NBUF>;
    using elem = typename E::elem;
    constexpr int BR = SM::BR, MR = SM::MR;
    constexpr int THREADS = NW * 64;
    // buffer sets: K tile, V tile right after it; two separate variables (see stream_tiles)
    __shared__ __align__(1024) char set0[SM::SET];
    __shared__ __align__(1024) char set1[NBUF == 2 ? SM::SET : 1024];
    __shared__ uint32_t wm[MR * MAX_W];
    __shared__ uint32_t fm[MR * MAX_W];
    __shared__ int tl[MAX_T];
    __shared__ int tl_count[4];
    __shared__ unsigned long long blk_stats[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31;
    const int N = p.N, T = p.T, W = p.W;
    int bh, I;
    map_block(blockIdx.x, p.BH, (N + BR - 1) / BR, bh, I);
    const long q0 = (long)I * BR, qw0 = q0 + wave * 32 * QB;
    const bool active = qw0 < N;
    if constexpr (!MASK_ONLY) {
        // row groups whose supports were listed get their output from gather_out_kernel
        if (p.gflag && p.gflag[(long)bh * ((N + p.grows - 1) / p.grows) + q0 / p.grows]) return;
    }
    const elem* Qh = (const elem*)p.Q + (long)bh * N * D;
    const elem* Kh = (const elem*)p.K + (long)bh * N * D;
    // V in the stage-2 element type (for bf16 inputs: the fp16 copy made by convert_kernel)
    const typename E2::elem* Vh = MASK_ONLY ? nullptr : (const typename E2::elem*)p.V2 + (long)bh * N * D;
    const int myrow = (wave * 32 * QB) / 64;
    const HeadConsts hc = head_consts(p, bh);
    const float c = hc.c, r = hc.r;

    for (int i = tid; i < MR * W; i += THREADS) {
        wm[i] = (I * MR + i / W < T) ? (uint32_t)p.wmask[((long)bh * T + (long)I * MR + i / W) * W + (i % W)] : 0u;
        fm[i] = 0u;
    }
    build_tile_list(wm, MR, W, tl, tl_count, tid);

    Owned<E, D, QB> qf;
    load_owned<E, D, QB>(qf, Qh, active ? qw0 : 0, lane);
    // per-row solver state, held by both lanes of a row
    constexpr bool REFINE = !MASK_ONLY;
    float thr[QB], lo[QB], hi[QB], f1_prev[QB];
    int done[QB], iters[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const long g = (long)bh * N + qw0 + 32 * qb + n;
        thr[qb] = active ? p.tau[g] : 0.f;
        lo[qb] = hi[qb] = 0.f; done[qb] = 1; iters[qb] = 0; f1_prev[qb] = -1.f;
        if (REFINE && active) {
            lo[qb] = p.rs_lo[g]; hi[qb] = p.rs_hi[g]; f1_prev[qb] = p.rs_f1[g];
            const int st = p.rs_state[g];
            iters[qb] = st & 0xffff; done[qb] = st >> 16;
        }
    }

    f32x16 X[D / 32][QB];
    f32x16 C[2][QB];
    unsigned long long ntile_done = 0, npv_done = 0, nstat_done = 0;
    auto issue_kv = [&](int it, char* buf) {
        const long j = tl[it];
        issue_rows<E, D, NW>(buf, Kh, j * 64, wave, lane);
        if constexpr (!MASK_ONLY) issue_rows<E2, D, NW>(buf + SM::KBYTES, Vh, j * 64, wave, lane);
    };
    auto issue_k = [&](int it, char* buf) { issue_rows<E, D, NW>(buf, Kh, (long)tl[it] * 64, wave, lane); };

    // Phase 4 doubles as the next evaluation of f: the row sums of P are f(tau) + 1.  A row is
    // finished when |f| <= tol, or (alpha <= 2, where f' is bounded) when the step -f / f' (with f'
    // from its previous evaluation: a chord step) is shorter than tol; it then takes that step, and
    // O, computed less than tol away in tau, stands.  Only when some row fails both, a scores-only sweep gathers f', f'' at the
    // same tau, the hybrid step moves those rows, and Phase 4 runs again.
    auto pv_pass = [&](float (&rowsum)[QB]) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int v = 0; v < 16; ++v) X[db][qb][v] = 0.f;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) rowsum[qb] = 0.f;
        stream_tiles<NBUF>(*tl_count, set0, NBUF == 2 ? set1 : set0, issue_kv, [&](int it, const char* buf) {
            const int j = tl[it];
            if (!mask_bit(wm, W, myrow, j)) return;
            stage1<E, D, QB>(C, buf, qf, lane);
            if (p.causal && (long)j * 64 + 63 > qw0) causal_hide<QB, true>(C, j * 64, (int)qw0, lane);
            ++ntile_done;
            float ymax = 0.f;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float yp = fmaxf(fmaf(c, C[kb][qb][v], -thr[qb]), 0.f);
                        ymax = fmaxf(ymax, yp);
                        float pr;
                        if constexpr (AM == ALPHA_GEN) pr = (yp > 0.f) ? pow_r<AM>(yp, r) : 0.f;
                        else pr = pow_r<AM>(yp, r);
                        if constexpr (REFINE) rowsum[qb] += pr;
                        C[kb][qb][v] = pr;
                    }
            if (!__any(ymax > 0.f)) return;
            if (lane == 0) atomicOr(&fm[myrow * W + (j >> 5)], 1u << (j & 31));
            if constexpr (!MASK_ONLY) { stage2<E2, D, QB>(X, buf + SM::KBYTES, C, lane); ++npv_done; }
        });
    };

    float rowsum[QB];
    pv_pass(rowsum);
    if constexpr (REFINE) {
        int need = 0;
        float fval[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            fval[qb] = xhalf_sum(rowsum[qb]) - 1.f;
            if (!done[qb]) {
                iters[qb] += 1;
                const float chord = -fval[qb] / f1_prev[qb];
                if (fabsf(fval[qb]) <= p.tol) done[qb] = 1;
                else if (fabsf(chord) < step_tol(p.tol, thr[qb]) && f1_prev[qb] < 0.f && hc.alpha <= 2.f) {
                    thr[qb] = fminf(fmaxf(thr[qb] + chord, lo[qb]), hi[qb]);
                    done[qb] = 1;
                } else need = 1;
            }
        }
        if (__syncthreads_count(need) != 0) {
            // rare: finish those rows with scores-only sweeps over the tiles that held some P > 0
            // (a superset of the support at any larger tau), then form O once more.  For alpha > 2
            // the iterates come from both sides of the root, so the next tau may lie below this
            // one: the sweeps then walk the whole working mask, which was taken at tau_0 <= tau*.
            const bool below = hc.alpha > 2.f;
            bool have_f = true;          // the first sweep runs at the tau whose f is already known
            SecantPrev prev[QB];
            for (int sweep = 0; sweep < p.max_sweeps; ++sweep) {
                float F[QB], G[QB], Hs[QB];
                int cnt[QB];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) { F[qb] = G[qb] = Hs[qb] = 0.f; cnt[qb] = 0; }
                stream_tiles<NBUF>(*tl_count, set0, NBUF == 2 ? set1 : set0, issue_k, [&](int it, const char* buf) {
                    const int j = tl[it];
                    if (!mask_bit(below ? wm : fm, W, myrow, j)) return;
                    stage1<E, D, QB>(C, buf, qf, lane);
                    if (p.causal && (long)j * 64 + 63 > qw0) causal_hide<QB, true>(C, j * 64, (int)qw0, lane);
                    ++nstat_done;
                    eval_scores<AM, QB>(C, thr, c, r, F, G, Hs, cnt);
                });
                int pending = 0;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    if constexpr (AM == ALPHA_15) Hs[qb] = (float)cnt[qb];
                    if constexpr (AM == ALPHA_20) G[qb] = (float)cnt[qb];
                    const float g = xhalf_sum(G[qb]), hs = xhalf_sum(Hs[qb]);
                    const float f = have_f ? fval[qb] : xhalf_sum(F[qb]) - 1.f;
                    if (!done[qb]) {
                        if (!have_f) iters[qb] += 1;
                        if (!have_f && fabsf(f) <= p.tol) done[qb] = 1;
                        else {
                            const float stol = step_tol(p.tol, thr[qb]);
                            const float cand = hybrid_step<AM>(thr[qb], f, g, hs, r, hc.alpha, lo[qb], hi[qb], prev[qb], stol);
                            if (fabsf(cand - thr[qb]) < stol) done[qb] = 1;
                            thr[qb] = cand;
                        }
                        pending |= !done[qb];
                    }
                }
                have_f = false;
                if (__syncthreads_count(pending) == 0) break;
            }
            __syncthreads();
            for (int i = tid; i < MR * W; i += THREADS) fm[i] = 0u;
            __syncthreads();
            float unused[QB];
            pv_pass(unused);
        }
    }
    if constexpr (REFINE) {
        if (active && (lane >> 5) == 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const long g = (long)bh * N + qw0 + 32 * qb + n;
                p.tau[g] = thr[qb];
                if (p.iters) p.iters[g] = iters[qb];
            }
        }
    }

    if constexpr (!MASK_ONLY)
        if (active) store_owned_T<D, QB>(p.O + (long)bh * N * D, qw0, X, 1.f, lane);
    for (int i = tid; i < MR * W; i += THREADS)
        if (I * MR + i / W < T) p.mask[((long)bh * T + (long)I * MR + i / W) * W + (i % W)] = (int32_t)fm[i];
    {
        const int slot[3] = {MASK_ONLY ? 6 : 1, 7, 0};
        const unsigned long long val[3] = {ntile_done * QB, npv_done * QB, nstat_done * QB};
        flush_counters<3>(blk_stats, p.stats, slot, val, tid, lane);
    }
}

// Phase 4 for sparse row groups: O_r = sum over the row's support of p_j V_j, from the support
// entries (raw score, key index) that tau_list_kernel left at the front of the row's two lists.
// With a handful of non-zeros per row this is a gather of a few rows of V, not a matrix product:
// sixteen lanes per row (GatherLanes).  V is read in the caller's element type.
template <class E, int D, int AM>
__global__ __launch_bounds__(256) void gather_out_kernel(Params p) {
    using elem = typename E::elem;
    using L = GatherLanes<E, D>;
    using vec = typename L::vec;
    constexpr int EPT = L::EPT, BT = 4;               // rows of V in flight per lane
    const int tid = threadIdx.x, sub = tid & 15, rsel = tid >> 4;
    // a work-group takes GATHER_ROWS rows of a row group (one per 16 lanes): the rows are
    // chains of dependent loads, so many short work-groups hide their latency better than few long ones
    const int N = p.N, G = (N + p.grows - 1) / p.grows, parts = p.grows / GATHER_ROWS;
    int bh, I;
    map_block(blockIdx.x, p.BH, G * parts, bh, I);
    const int part = I % parts;
    I /= parts;
    if (!p.gflag[(long)bh * G + I]) return;
    const int row = I * p.grows + part * GATHER_ROWS + rsel;
    if (row >= N) return;                             // (N is a multiple of 64: whole work-groups)
    const HeadConsts hc = head_consts(p, bh);
    const float c = hc.c, r = hc.r;
    const HeadRows<E, D> Vh(p.V, (long)bh * N, N, sub);
    const long gi = (long)bh * N + row;
    const float tau = p.tau[gi];
    const int s0 = p.scnt[gi * 2], tot = s0 + p.scnt[gi * 2 + 1];
    const char* l0 = (const char*)p.lists + (size_t)gi * (2 * LIST_CAP * 8);      // the second list follows the first
    const int nmax = longest_list(tot);
    float acc[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) acc[k] = 0.f;
    for (int i0 = 0; i0 < nmax; i0 += 16) {
        const int i = i0 + L::entry_of(sub);
        uint2 e = make_uint2(0u, NO_ENTRY);
        if (i < tot) e = *(const uint2*)(l0 + (i < s0 ? i * 8 : LIST_CAP * 8 + (i - s0) * 8));
        const float y = fmaf(c, __uint_as_float(e.x), -tau);
        const float pr = (i < tot && y > 0.f) ? pow_r<AM>(y, r) : 0.f;
        unroll_steps<L::STEPS / BT>([&](auto b) {
            constexpr int S0 = decltype(b)::value * BT;
            if (S0 * L::PAR >= nmax - i0) return;
            vec v[BT];
            unroll_steps<BT>([&](auto u) { v[decltype(u)::value] = Vh.load(L::template of_step<S0 + decltype(u)::value>(e.y)); });
            unroll_steps<BT>([&](auto u) { add_scaled<EPT>(acc, L::template of_step<S0 + decltype(u)::value>(pr), v[decltype(u)::value]); });
        });
    }
#pragma unroll
    for (int k = 0; k < EPT; ++k) acc[k] = L::halves_sum(acc[k]);
    L::store(p.O + gi * D, acc, sub);
}

// All causally visible tiles set: the working mask handed to out_kernel<MASK_ONLY>.
static __global__ void full_mask_kernel(int32_t* wmask, int BH, int T, int W, int causal) {
    const long total = (long)BH * T * W;
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
        const int m = (int)(i % W), row = (int)((i / W) % T);
        const int last = causal ? row : T - 1;       // last visible tile
        uint32_t w = 0;
        const int lo = 32 * m;
        if (last >= lo) {
            const int nb = min(last - lo + 1, 32);
            w = (nb == 32) ? 0xffffffffu : ((1u << nb) - 1u);
        }
        wmask[i] = (int32_t)w;
    }
}

// Element-wise copy into another element type, optionally divided by a (bits of a float a >= 0).
// A value whose magnitude the narrower type cannot hold (fp16: 65504) is copied as the largest finite
// value of its sign and counted in *clamped (so that the caller can see that the result is not the
// one of its inputs: the fp16 copies are the operands of every second-stage product).
template <class Ein, class Eout>
__global__ __launch_bounds__(256) void convert_kernel(const typename Ein::elem* in, typename Eout::elem* out, long n,
                                                      const unsigned int* amax_bits, const int32_t* needed,
                                                      unsigned long long* clamped) {
    if (needed && *needed == 0) return;     // nobody will read the copy
    float mul = 1.f;
    if (amax_bits) {
        const float a = __uint_as_float(*amax_bits);
        if (a > 0.f) mul = 1.f / a;
    }
    constexpr bool NARROW = std::is_same<Eout, F16>::value && !std::is_same<Ein, F16>::value;
    int nclamped = 0;
    for (long i = (blockIdx.x * 256L + threadIdx.x) * 8; i < n; i += (long)gridDim.x * 256 * 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float x = (float)in[i + e] * mul;
            if constexpr (NARROW) {
                if (fabsf(x) > 65504.f) { x = copysignf(65504.f, x); ++nclamped; }     // (NaN compares false and stays NaN)
            }
            out[i + e] = Eout::from_float(x);
        }
    }
    if constexpr (NARROW) {
        if (__any(nclamped != 0)) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) nclamped += __shfl_xor(nclamped, off);
            if ((threadIdx.x & 63) == 0 && clamped) atomicAdd(clamped, (unsigned long long)nclamped);
        }
    }
}

// The backward's fp16 copies, limited to the rows its matrix kernels will read: one work-group per
// 64 rows of a head and tensor (blockIdx.y picks the tensor).  Query side (Q, dO): the rows of row
// groups that are not served by the gather kernels (gflag = 0).  Key side (K, V): every row such a
// group can see - with a causal mask the rows up to the head's last such group, else all rows when
// the head has one.  gflag null: all rows.
struct ConvertJob { const void* in; void* out; const unsigned int* amax_bits; int query_side; };
struct ConvertJobs { ConvertJob j[4]; };
template <class Ein, class Eout, int D>
__global__ __launch_bounds__(256) void convert_rows_kernel(ConvertJobs jobs, int N, const int32_t* needed,
                                                           const int32_t* gflag, int grows, int causal,
                                                           unsigned long long* clamped) {
    if (needed && *needed == 0) return;     // nobody will read the copies
    __shared__ int last_plain;
    const ConvertJob job = jobs.j[blockIdx.y];
    const typename Ein::elem* in = (const typename Ein::elem*)job.in;
    typename Eout::elem* out = (typename Eout::elem*)job.out;
    const unsigned int* amax_bits = job.amax_bits;
    const int tiles = N / 64, bh = blockIdx.x / tiles, rt = blockIdx.x % tiles;
    if (gflag) {
        const int ng = (N + grows - 1) / grows;
        const int32_t* gf = gflag + (long)bh * ng;
        if (job.query_side) {
            if (gf[(rt * 64) / grows]) return;
        } else {
            if (threadIdx.x == 0) last_plain = -1;
            __syncthreads();
            int mine = -1;
            for (int g = threadIdx.x; g < ng; g += 256)
                if (!gf[g]) mine = g;
            if (mine >= 0) atomicMax(&last_plain, mine);
            __syncthreads();
            if (last_plain < 0 || (causal && rt * 64 >= (last_plain + 1) * grows)) return;
        }
    }
    float mul = 1.f;
    if (amax_bits) {
        const float a = __uint_as_float(*amax_bits);
        if (a > 0.f) mul = 1.f / a;
    }
    constexpr bool NARROW = std::is_same<Eout, F16>::value && !std::is_same<Ein, F16>::value;
    int nclamped = 0;
    const long base = ((long)bh * N + (long)rt * 64) * D;
    for (int i = threadIdx.x * 8; i < 64 * D; i += 256 * 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float x = (float)in[base + i + e] * mul;
            if constexpr (NARROW) {
                if (fabsf(x) > 65504.f) { x = copysignf(65504.f, x); ++nclamped; }     // (NaN compares false and stays NaN)
            }
            out[base + i + e] = Eout::from_float(x);
        }
    }
    if constexpr (NARROW) {
        if (__any(nclamped != 0)) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) nclamped += __shfl_xor(nclamped, off);
            if ((threadIdx.x & 63) == 0 && clamped) atomicAdd(clamped, (unsigned long long)nclamped);
        }
    }
}

static __global__ void zero_stats_kernel(unsigned long long* stats, int n, unsigned int* scal) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) stats[i] = 0ull;
    if (scal && threadIdx.x < 4) scal[threadIdx.x] = 0u;
}

// max |x| over a tensor, rounded up to a power of two -> atomicMax on the float's bit pattern
// (non-negative floats order as unsigned ints); n is a multiple of 8.  One atomic per block: thousands of them on one word
// would take longer than reading the tensor.
template <class E>
__global__ __launch_bounds__(256) void amax_kernel(const typename E::elem* x, long n, unsigned int* out_bits, const int32_t* needed) {
    __shared__ float part[4];
    if (needed && *needed == 0) return;     // nobody will read the maximum
    float m = 0.f;
    const long stride = (long)gridDim.x * 256 * 8;
    long i = (blockIdx.x * 256L + threadIdx.x) * 8;
    if constexpr (sizeof(typename E::elem) == 2) {
        // four 16-byte loads in flight per thread: one at a time leaves the read latency-bound
        for (; i + 3 * stride < n; i += 4 * stride) {
            u32x4 w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = *(const u32x4*)(x + i + u * stride);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf((float)((const typename E::elem*)&w[u])[e]));
        }
    }
    for (; i < n; i += stride) {
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf((float)x[i + e]));
    }
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        // rounded up to a power of two: dividing by it is exact, so the fp16 copy of dO / max|dO|
        // holds the caller's bf16 values exactly (a scale with mantissa bits would round every
        // element, and dP - delta, a difference of nearly equal sums, multiplies that rounding)
        unsigned int bits = __float_as_uint(fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3])));
        if ((bits & 0x007fffffu) && bits < 0x7f000000u) bits = (bits & 0x7f800000u) + 0x00800000u;
        atomicMax(out_bits, bits);
    }
}

}  // namespace ea
