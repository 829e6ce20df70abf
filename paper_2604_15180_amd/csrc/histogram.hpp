// The histogram of a row's scores (Eq. 6-9): bounds and root of its objective f_h.  Included after
// common.hpp, of which it takes the power functions and lane helpers (a host program that supplies those can run
// the one-lane form).
#pragma once
#include <stdint.h>

namespace ea {

// ---- histogram solve (App. C.3) -----------------------------------------------------------------
// The row's histogram is a window of SLOTS = NB + 1 consecutive bins of an absolute grid of width
// h = 1 / NB, kept in a circular buffer: bin k of the window (left edge k h above the window's origin)
// is H[(rot + k) % SLOTS], BITS bits at bit `shift` of each word (two rows share a word when BITS == 16).
// PAIRED: the two lanes (n, n + 32) of a row hold the same arguments and read half of the bins each.
//
// The sums S0, S1, S2 (count, sum and sum of squares of the distance t = NB - k from the top bin, in bins) of a
// set of bins give a lower bound of f_h that has a closed-form root.  With y_k = k h - tau, r = 1/(alpha-1),
// and 0 < y <= 1 inside the window:
//   MOM 1:  sum y^r >= sum y                          (r <= 1; equality at alpha = 2)
//   MOM 2:  sum y^r >= sum y^2                        (r <= 2; equality at alpha = 1.5)
//   MOM 3:  sum y^r >= S0 (sum y^2 / S0)^(r/2)        (r >= 2, power means), which reaches 1 where sum y^2 does S0^(1 - 2/r)
// The active set is the largest one, from the top, whose root lies below the left edge of its lowest
// non-empty bin, i.e. the largest one whose bound at that edge is below 1: a polynomial in the three
// sums.  Whole chunks of eight bins are tried first and the bins of one chunk then; the root is formed once, from
// the sums of the set.  (MOM 1 and 2 only rise towards lower edges.  MOM 3 falls again where many bins join far
// below the others, S0^(1 - r/2): any set that passes gives a lower bound, the largest not always the best one, and
// for large r it can lie far below the root.)
// The sums are integers, so that they do not depend on the order of
// summation; a scan in fp32 over all 64 bins by each lane took three times the instructions.  Steps, together
// with the general solve below: alpha = 1.25, 32 heads of 8192 tokens 1633 -> 1447 us, 64 heads of 4096 tokens at
// alpha = 1.5 907 -> 858 us (d = 64).
// Returns the root in units above the origin - the root tau_h of f_h (Eq. 9) itself where equality
// holds, else a value below it; -h for an empty histogram.  *active, if wanted: the counts of the active set.
template <int BITS> EA_DEV uint32_t histogram_count(const uint32_t* H, int slot, int shift) {
    const uint32_t w = H[slot];
    if constexpr (BITS == 32) return w;
    else return (w >> shift) & ((1u << (BITS & 31)) - 1u);
}
template <int MOM, int SLOTS, int BITS, bool PAIRED>
EA_DEV float histogram_moment_root(const uint32_t* H, int rot, int shift, float h, float r, int* active = nullptr) {
    using I = int;                                     // (at most 2^17 counts: S2 stays below 2^30)
    constexpr int NB = SLOTS - 1, NCH = SLOTS / 8;
    static_assert(NCH % 2 == 0, "chunks are shared by the two lanes of a row");
    const float q = 1.f - 2.f / r;
    // bound at the edge t bins below the top, less its target, of a non-empty set (negative: the set may grow)
    auto inside = [&](I S0, I S1, I S2, int t) {
        if constexpr (MOM == 1) return (I)t * S0 - S1 < (I)NB;
        const I d = (I)t * ((I)t * S0 - 2 * S1) + S2;
        if constexpr (MOM == 2) return d < (I)(NB * NB);
        return (float)d * (h * h) < __builtin_amdgcn_exp2f(q * __builtin_amdgcn_logf((float)S0));
    };
    const int half = PAIRED ? (int)(__lane_id() >> 5) : 0;
    I S0 = 0, S1 = 0, S2 = 0, B0 = 0, B1 = 0, B2 = 0;
    int full = 0;                                      // chunks wholly inside the set
    bool grows = true;
    auto try_chunk = [&](int m, I a0, I a1, I a2) {
        S0 += a0; S1 += a1; S2 += a2;
        grows = grows && (S0 == 0 || inside(S0, S1, S2, 8 * m + 7));
        if (grows) { B0 = S0; B1 = S1; B2 = S2; full = m + 1; }
    };
#pragma unroll 1
    for (int m = 0; m < NCH; m += PAIRED ? 2 : 1) {    // (unrolled, the loads of all chunks cost registers that the caller's score tile holds)
        const int t0 = 8 * (m + half);
        I a0 = 0, a1 = 0, a2 = 0;                      // (distances inside the chunk at first)
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const I c = (I)histogram_count<BITS>(H, (rot + NB - t0 - b) & (SLOTS - 1), shift);
            a0 += c; a1 += (I)b * c; a2 += (I)(b * b) * c;
        }
        a2 += (I)t0 * (2 * a1 + (I)t0 * a0);
        a1 += (I)t0 * a0;
        if constexpr (PAIRED) {
            const auto x0 = __builtin_amdgcn_permlane32_swap((uint32_t)a0, (uint32_t)a0, false, false);
            const auto x1 = __builtin_amdgcn_permlane32_swap((uint32_t)a1, (uint32_t)a1, false, false);
            const auto x2 = __builtin_amdgcn_permlane32_swap((uint32_t)a2, (uint32_t)a2, false, false);
            try_chunk(m, (int)x0[0], (int)x1[0], (int)x2[0]);
            try_chunk(m + 1, (int)x0[1], (int)x1[1], (int)x2[1]);
        } else try_chunk(m, a0, a1, a2);
        if (!__any(grows)) break;
    }
    S0 = B0; S1 = B1; S2 = B2;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const int t = 8 * full + b;                    // (full = NCH: bins past the window, not counted)
        const I c = full < NCH ? (I)histogram_count<BITS>(H, (rot + NB - t) & (SLOTS - 1), shift) : (I)0;
        S0 += c; S1 += (I)t * c; S2 += (I)(t * t) * c;
        if (c > 0 && inside(S0, S1, S2, t)) { B0 = S0; B1 = S1; B2 = S2; }
    }
    if (active) *active = B0;
    if (B0 == 0) return -h;
    const float n = (float)B0, inv = 1.f / n;
    float t_root;
    if constexpr (MOM == 1) t_root = (float)(B1 + (I)NB) * inv;
    else {
        // about the bin nearest the mean, where the variance has no cancellation left
        const int t0 = (int)((float)B1 * inv + 0.5f);
        const float m1 = (float)(B1 - (I)t0 * B0) * inv, m2 = (float)(B2 - (I)t0 * (2 * B1 - (I)t0 * B0)) * inv;
        const float target = MOM == 2 ? 1.f : __builtin_amdgcn_exp2f(q * __builtin_amdgcn_logf(n));
        t_root = (float)t0 + (m1 + sqrtf(fmaxf(target * (float)(NB * NB) * inv - (m2 - m1 * m1), 0.f)));
    }
    return ((float)NB - t_root) * h;
}
// A lower bound of the histogram's root for general alpha, from the closed forms alone
template <int SLOTS, int BITS, bool PAIRED>
EA_DEV float histogram_lower_bound(const uint32_t* H, int rot, int shift, float h, float r, int* active = nullptr) {
    if (r >= 2.f) return histogram_moment_root<3, SLOTS, BITS, PAIRED>(H, rot, shift, h, r, active);
    if (r >= 1.f) return histogram_moment_root<2, SLOTS, BITS, PAIRED>(H, rot, shift, h, r, active);
    return histogram_moment_root<1, SLOTS, BITS, PAIRED>(H, rot, shift, h, r, active);
}
// Newton steps from the left for f = F - 1, F(tau) = sum_k c_k [y_k]_+^r with r >= 1: f is convex and falls with tau,
// so the iterates rise and stay at or below the root.  eval(tau, F, G) gives F and G = sum c y^(r-1).
// A step on f itself takes F down by about e at a time while F is large (by the power mean's bound F starts at
// thousands for r = 30 and more).  N = F^(1/r) is a norm of y, so convex as well and 1 at the same root, and its step,
// (N - 1) / -N' = (F - F^(1 - 1/r)) / G, is the longer one: with one bin it is the root.  Near the root, where the
// two agree and this one cancels, f's own step is taken.  Evaluations needed, r = 1 - 1000, 1 - 131072 counts: at most 5.
// `gap`: how far above the returned value the root can lie - nothing if the steps have died down, else by
// convexity f / |f'| at the root, which is at most (F - 1) / r as G >= 1 there (y <= 1).
constexpr int NEWTON_MAX = 24;
template <class Eval> EA_DEV float newton_from_left(Eval eval, float tau, float hi, float r, float& gap) {
    gap = 0.f;
    for (int i = 0; i < NEWTON_MAX; ++i) {
        float F, G;
        eval(tau, F, G);
        const float e = F > 2.f ? F - __builtin_amdgcn_exp2f((1.f - 1.f / r) * __builtin_amdgcn_logf(F)) : (F - 1.f) / r;
        const float nt = tau + e / G;                  // (G = 0, an empty histogram: NaN or inf, not taken)
        const bool moves = F > 1.f && nt > tau && nt <= hi;
        const bool far = moves && (nt - tau > 1e-7f || F > 1.001f);
        gap = far || !(F < 3e38f) ? fmaxf(F - 1.f, 0.f) / r : 0.f;
        if (moves) tau = nt;
        if (!__any(far)) break;
    }
    gap = fminf(gap, fmaxf(hi - tau, 0.f));
    return tau;
}

// The root tau_h of f_h(tau) = -1 + sum_k H_k [k h - tau]_+^r (Eq. 9) in units above the origin;
// -h for an empty histogram.  general alpha: `start` is a point known to lie at or below tau* (the row's maximum
// - 1), and tau* is at most h + gap above the result; otherwise neither is used.  `active`: closed forms only.
template <int AM, int SLOTS, int BITS, bool PAIRED>
EA_DEV float solve_histogram(const uint32_t* H, int rot, int shift, float h, float r, float start, float& gap, int* active = nullptr) {
    gap = 0.f;
    if constexpr (AM == ALPHA_15) return histogram_moment_root<2, SLOTS, BITS, PAIRED>(H, rot, shift, h, r, active);
    else if constexpr (AM == ALPHA_20) return histogram_moment_root<1, SLOTS, BITS, PAIRED>(H, rot, shift, h, r, active);
    else {
        // PAIRED: a lane takes every other bin.  Eight bins are read together (one at a time, each read
        // waits for the one before), down to the chunk that no lane's threshold reaches.
        constexpr int STEP = PAIRED ? 2 : 1;
        const int first = SLOTS - 1 - (PAIRED ? (int)(__lane_id() >> 5) : 0);
        auto eval = [&](float tau, float& F, float& G) {
            float f = 0.f, g = 0.f;
            for (int k8 = first; k8 >= 0; k8 -= 8 * STEP) {
                if (!__any(k8 * h > tau)) break;
                float cnt[8];
#pragma unroll
                for (int b = 0; b < 8; ++b) cnt[b] = (float)histogram_count<BITS>(H, (rot + k8 - b * STEP) & (SLOTS - 1), shift);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const float y = (k8 - b * STEP) * h - tau;
                    const float pr1 = y > 0.f && cnt[b] > 0.f ? cnt[b] * pow_r1<AM>(y, r) : 0.f;
                    f = fmaf(pr1, y, f);
                    g += pr1;
                }
            }
            if constexpr (PAIRED) { f = xhalf_sum(f); g = xhalf_sum(g); }
            F = f; G = g;
        };
        if (r < 1.f) {
            // alpha > 2: f_h is not convex; bisection of [-h, (SLOTS-1) h], whose left end, where f_h >= 0, is returned
            float lo = -h, hi = (SLOTS - 1) * h;
            for (int i = 0; i < 22; ++i) {
                const float mid = 0.5f * (lo + hi);
                float F, G;
                eval(mid, F, G);
                if (F - 1.f >= 0.f) lo = mid; else hi = mid;
            }
            return lo;
        }
        // from the closed-form bound Newton needs three or four steps at alpha = 1.25
        // (bisecting first took sixteen evaluations)
        return newton_from_left(eval, fmaxf(histogram_lower_bound<SLOTS, BITS, PAIRED>(H, rot, shift, h, r), fminf(start, (SLOTS - 1) * h)),
                                (SLOTS - 1) * h, r, gap);
    }
}

}  // namespace ea
