// Pieces of the gather kernels (output and gradients of sparse row groups, entry by entry): sixteen
// lanes work on one row (or key), in chunks of sixteen entries.
//
// What is needed once per entry - the list entry itself, P and U of its score, its slot in a key's
// list - is done by the lane that holds the entry, for sixteen entries at once; only the work on the
// entry's row of V, K, Q or dO is done by all of the row's lanes, 16 bytes of it per lane where the
// type allows.  A row of D elements then spans LPE lanes: with LPE = 8 (16-bit, D = 64) the two
// halves of the sixteen lanes take two entries side by side.
//   step s of a chunk: half p works on the entry held by lane LPE p + s (PAR = 1: lane s)
//   lane l holds list entry  l (PAR = 1)  or  2 (l % 8) + l / 8 (PAR = 2) of the chunk, so that the
//   entries of a short list fall into its first steps
// A lane past the end of its list holds NO_ENTRY and weight 0.  0 times what stands in some row is not 0 if that is
// infinite, so such a lane must get zeros: rows are read by buffer loads, whose bounds check returns zeros
// for an index past the head's rows (clearing the loaded values instead cost 1 us in each gather kernel at 256 tokens; steps:
// fp32, 256 tokens 110.2 -> 108.2 us, 16384 tokens, d = 128, sigma = 1 4525 -> 4481).
#pragma once
#include <type_traits>
#include <utility>

#include "common.hpp"

namespace ea {

constexpr uint32_t NO_ENTRY = MAX_T * 64;       // past the last row of every head

template <class F, int... I> EA_DEV void unroll_steps(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
// f(0), f(1), ... f(N-1) with the index as a compile-time constant (DPP controls are immediates)
template <int N, class F> EA_DEV void unroll_steps(F&& f) { unroll_steps(static_cast<F&&>(f), std::make_integer_sequence<int, N>{}); }

template <int CTRL, int BANKS = 0xf> EA_DEV uint32_t dpp_word(uint32_t old, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, 0xf, BANKS, BANKS == 0xf);
}

template <class E, int D> struct GatherLanes {
    using elem = typename E::elem;
    static constexpr int EPT = sizeof(elem) == 2 ? 8 : D / 16;     // elements of a row per lane
    static constexpr int LPE = D / EPT;                            // lanes per entry: 8 or 16
    static constexpr int PAR = 16 / LPE;                           // entries side by side
    static constexpr int STEPS = 16 / PAR;                         // steps of a chunk of sixteen entries
    static_assert(LPE == 8 || LPE == 16, "a row spans half or all of the sixteen lanes");
    typedef elem vec __attribute__((ext_vector_type(EPT)));
    // first element of a row that lane `sub` (0..15) works on, and the list entry it holds in a chunk
    static EA_DEV int column(int sub) { return (sub % LPE) * EPT; }
    static EA_DEV int entry_of(int sub) { return PAR == 1 ? sub : 2 * (sub & 7) + (sub >> 3); }
    // the value held by the lane whose entry a lane works on in step S
    template <int S> static EA_DEV uint32_t of_step(uint32_t v) {
        const uint32_t a = dpp_word<0x150 + S>(0u, v);             // row_newbcast: lane S of the sixteen
        if constexpr (PAR == 1) return a;
        else return dpp_word<0x150 + S + 8, 0xc>(a, v);            // upper eight lanes: lane S + 8
    }
    template <int S> static EA_DEV float of_step(float v) { return __uint_as_float(of_step<S>(__float_as_uint(v))); }
    // whether this lane holds (one of) the entries of step S
    template <int S> static EA_DEV bool holds(int sub) { return (sub % LPE) == S; }
    // sum over the lanes that work on one entry, in all of them
    static EA_DEV float entry_sum(float v) { return group_sum<LPE>(v); }
    // sum of the partial sums of the entries side by side, in both halves
    static EA_DEV float halves_sum(float v) {
        if constexpr (PAR == 2) v += __uint_as_float(dpp_word<0x128>(0u, __float_as_uint(v)));   // row_ror:8
        return v;
    }
    // store this lane's share of a row of sums (all halves hold the same sums)
    static EA_DEV void store(float* row, const float (&x)[EPT], int sub) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        if constexpr (PAR == 1) {
#pragma unroll
            for (int k = 0; k < EPT; k += 4) *(f4*)(row + column(sub) + k) = f4{x[k], x[k + 1], x[k + 2], x[k + 3]};
        } else {                                                   // each half stores four of the eight
            const bool up = sub >= LPE;
            *(f4*)(row + column(sub) + (up ? 4 : 0)) = f4{up ? x[4] : x[0], up ? x[5] : x[1], up ? x[6] : x[2], up ? x[7] : x[3]};
        }
    }
};

// <a, b> + c over a lane's share of two rows.  bf16: products of pairs summed in fp32 by the dot
// instruction (exact products; half the instructions of unpacking one side alone).
template <class E, int N, class V> EA_DEV float dot_share(const V& a, const V& b, float c) {
    if constexpr (std::is_same<E, Bf16>::value) {
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int k = 0; k < N; k += 2) c = __builtin_amdgcn_fdot2_f32_bf16(b2{a[k], a[k + 1]}, b2{b[k], b[k + 1]}, c, false);
    } else {
#pragma unroll
        for (int k = 0; k < N; ++k) c = fmaf((float)a[k], (float)b[k], c);
    }
    return c;
}
// The rows of one head, and this lane's share of row `index` (an entry's key or row): zeros for NO_ENTRY.
template <class E, int D> struct HeadRows {
    using L = GatherLanes<E, D>;
    using elem = typename E::elem;
    static constexpr int BYTES = L::EPT * (int)sizeof(elem);
    static_assert(BYTES == 16 || BYTES == 32, "one or two 16-byte loads");
    static_assert((long)MAX_T * 64 * D * (long)sizeof(elem) < (1l << 31), "32-bit offsets");
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t column;                                               // bytes
    EA_DEV HeadRows(const void* rows, long first, int N, int sub)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc((void*)((const elem*)rows + first * D), 0, N * D * (int)sizeof(elem), 0x00020000)),
          column((uint32_t)L::column(sub) * (uint32_t)sizeof(elem)) {}
    EA_DEV typename L::vec load(uint32_t index) const {
        const uint32_t at = index * (uint32_t)(D * sizeof(elem)) + column;
        const auto lo = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 0, 0);
        if constexpr (BYTES == 16) return __builtin_bit_cast(typename L::vec, lo);
        else {
            typedef uint32_t u8 __attribute__((ext_vector_type(8)));
            const auto hi = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at + 16, 0, 0);
            return __builtin_bit_cast(typename L::vec, u8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
        }
    }
};
// the longest list of the wave's four rows or keys
EA_DEV int longest_list(int n) {
    const auto x = __builtin_amdgcn_permlane16_swap((uint32_t)n, (uint32_t)n, false, false);
    n = max((int)x[0], (int)x[1]);
    const auto y = __builtin_amdgcn_permlane32_swap((uint32_t)n, (uint32_t)n, false, false);
    return __builtin_amdgcn_readfirstlane(max((int)y[0], (int)y[1]));
}
template <int N, class V> EA_DEV void add_scaled(float (&acc)[N], float w, const V& x) {
#pragma unroll
    for (int k = 0; k < N; ++k) acc[k] = fmaf(w, (float)x[k], acc[k]);
}

}  // namespace ea
