// Pieces shared by the forward and backward kernels: parameter block, block->work mapping,
// the entmax power functions, mask-word helpers, the tile streaming loop.
#pragma once
#include "tiles.hpp"

namespace ea {

constexpr int MAX_T = 2048;     // N <= 131072
constexpr int MAX_W = 64;       // mask words per row
// A row group's output comes from the gather kernel when its supports average at most GATHER_SUP_MAX keys per
// row: the gather takes about 0.02 ns per entry, the matrix kernel 3.2 ns per marked tile at head dim 128 (8192
// tokens, sigma = 0.8, about 60 keys per row: gather 105 us, matrix 292 us; near 200 keys per row, alpha = 1.25 at
// sigma = 1, the two are level: 343 and 315 us).
constexpr int GATHER_SUP_MAX = 96;
// Query tiles per part of a mask column in dkdv_kernel from 65536 tokens on (half that below;
// every part pays the column walk, the owned K, V fragments and atomic adds of its results, and an
// empty part a work-group's launch: parts of 32 or 16 tiles measured slower at every length).
constexpr int COL_PART = 128;
// Work-group sizes of the gather kernels: each 16 lanes take one row (or key), a chain of
// dependent loads; 16 rows or keys per work-group (one per 16 lanes) measured 10 - 20 % faster than
// 128 - 256 per work-group, whose lanes walked 8 - 16 such chains one after the other.
constexpr int GATHER_ROWS = 16;          // rows per work-group of gather_out / bwd_rows
constexpr int BWD_COLS_KEYS = 16;        // keys per work-group of bwd_cols_kernel
// Backward: support entries per lane list (two lists per row) and entries per key in the lists by key.
constexpr int BWD_LIST_CAP = 64, KEY_LIST_CAP = 128;
// Non-zeros per marked 64 x 64 tile up to which a row group's backward takes the gather path.  Gather
// and matrix time of both directions: about 0.09 ns per entry and 6.3 ns per tile at head dim 64, 0.13 and
// 13.4 ns at head dim 128, where the gather's rows are twice as long: level near 70 and 100 entries.  The lower limit
// holds for every group; up to the higher one a group goes by gather where leaving it to the matrix kernels costs more than its tiles:
// * it has at most a quarter of the mean marked tiles (the first rows of causal heads): with all others gathered the matrix
//   kernels would run for these alone, and make their fp16 copies and max |dO|.  Backward with the lower limit alone / the higher one, head dim
//   64: 32 heads of 8192 tokens, alpha = 2, sigma = 2, lists found again, 445 / 385 us, alpha = 1.25, sigma = 2, 549 / 531.  Higher for
//   every group: 64 heads of 2048, sigma = 0.8, 386 / 430, sigma = 1, 333 / 381, without a mask, sigma = 0.7, 509 / 703, 16
//   heads of 4096, sigma = 0.7, 282 / 384, sigma = 0.8, 304 / 393, 32 of 8192, sigma = 0.8, 1106 / 1250; lists found again, whose sweep
//   ends where the limit is out of reach, 64 of 2048, sigma = 0.7, 430 / 543, head dim 128, 32 of 4096, sigma = 0.7, 864 / 1198;
// * there are at most BWD_FEW_GROUPS row groups, so that a quarter of the CUs has none of the matrix kernels' work-groups, whose walks then set their
//   time: head dim 64, 16 heads of 1088 tokens, sigma = 1 / 1.5, 112 / 95 and 81 / 73, 8 of 2048, sigma = 1, 128 / 106; near the limit, where only a
//   few groups qualify, it costs: 8 of 2048, sigma = 0.7, 142 / 167;
// * head dim 128, forward's lists: its rows' keys would have at most BWD_KEY_ENTRIES entries each if all later rows attended to as many
//   keys (hub keys, with more than KEY_LIST_CAP, are several times the work): 32 heads of 8192 tokens, sigma = 0.7 / 0.8 / 1 (at most 72 entries):
//   2894 / 1980, 1902 / 1449, 1027 / 899; 16 of 16384, sigma = 0.7 / 0.8 (124, 100): 2880 / 3545, 1900 / 1943.
// The power functions of general alpha weigh on both sides alike.
// fp32 matrix products run at a sixteenth of the 16-bit rate, 72 ns per tile: 16 heads of 2048 tokens at d = 64,
// sigma = 1, backward with 40 / 128 / 512: 631 / 265 / 121 us.  Attention sinks do not change the picture: 32 heads
// of 4096 tokens at d = 64 with one, gather 149, matrix 311 us; with four 268 and 225.
constexpr int bwd_entries_per_tile(int d, int elem_bytes, bool higher) {
    return elem_bytes == 4 ? 512 : d == 64 ? (higher ? 128 : 64) : (higher ? 96 : 40);
}
constexpr int BWD_FEW_GROUPS = 192;
constexpr float BWD_KEY_ENTRIES = 80.f;
// ... or, in a group with at most BWD_FEW_TILES marked tiles, BWD_ENTRIES_PER_ROW per row (at head dim 128).
constexpr int BWD_ENTRIES_PER_ROW = 6, BWD_FEW_TILES = 40;
// The gather kernels' fixed cost is a few passes over dK and dV, 0.3 - 0.45 ns per row: what the matrix
// kernels need for about two tiles per 64-row block.  Below that the mask as a whole stays with them.
// (8192 tokens, d = 64, block-structured inputs with 5 tiles per block: matrix 773, gather 650 us a step.)
constexpr int BWD_MIN_TILES_PER_BLOCK = 2;

constexpr int MASK_PARTS = 64;

// An entry of a key's list: the query row and its dS and P there.
struct KeyEntry { uint32_t row; float dS, pr; };
// Keys that more rows attend to than a list holds (hub keys): what does not fit goes to a log, a segment of it
// per LOG_ROWS query rows of a head, with room for all entries those rows can have (gather_budget).
// key_slot holds the key and the low bits of the entry's slot in the key's list, row_slot the row and the high bits.
struct LogEntry { uint32_t key_slot, row_slot; float dS, pr; };
constexpr int LOG_ROWS = 1024, LOG_PER_ROW = GATHER_SUP_MAX, MAX_LOG_SEGMENTS = MAX_T * 64 / LOG_ROWS;
constexpr int ROW_BITS = 17, SLOT_LOW_BITS = 32 - ROW_BITS;

constexpr int ALPHA_15 = 0, ALPHA_20 = 1, ALPHA_GEN = 2;
constexpr int LIST_CAP = 256;   // candidate entries per (row, lane half)

// What depends on alpha, per head when alpha differs between heads (then a table of these, one per
// head, sits in the workspace; otherwise the copy inside Params is used).
struct HeadConsts {
    float alpha;
    float c;              // (alpha-1)/sqrt(d): x = c * <q,k>
    float r;              // 1/(alpha-1)
    // c = kappa * rho with kappa a power of two and 1 <= rho < 2 (dK/dV kernel: keys scaled by kappa,
    // which is exact, scores kept in units of rho); lrho_u = log2(rho^(r-1))
    float kappa, rho, lrho_u;
    float pad[2];
};

struct Params {
    const void* Q; const void* K; const void* V; const void* dO;
    const void* V2;       // forward: V in the stage-2 element type (fp16 copy for bf16 inputs)
    float* O;             // forward: output; backward: the forward's output (nullable)
    float* tau; float* delta;
    float* ntau;          // backward scratch [BH][N]: -tau / rho, the bias the dK/dV kernel starts its scores from
    float* dQ; float* dK; float* dV;
    int32_t* mask;        // exported / final mask   [BH][T][W]
    int32_t* wmask;       // working mask (superset) [BH][T][W]
    int32_t* iters;       // nullable
    float* rs_lo; float* rs_hi; float* rs_f1; int* rs_state;   // [BH][N] solver state handed from tau_kernel to out_kernel
    float* rs_t0; float* rs_up0;   // [BH][N] what the histogram stage alone gave: tau_0 and the bracket's upper end (read out by tests)
    _Float16* tmax;       // [BH][T][N] per-row key-tile maxima of the raw scores (forward scratch)
    void* lists;          // [BH][N][2][LIST_CAP] candidate scores (raw score, key index), 8 bytes each
    int32_t* scnt;        // [BH][N][2] entries at the front of each list that are in the support at the final tau
    int32_t* gflag;       // [BH][ceil(N / grows)] 1 = the rows of this row group get their output by the gather kernel
    int grows;            // rows per row group of the candidate-list kernel
    // backward: entries per lane list of p.lists (its own lists, or the forward's when the caller hands
    // them over), and then the forward's group flags and their row-group size
    int right_edge;      // forward: thresholds are the right-edge histogram roots, no refinement (Sec. 3.2)
    // dkdv_kernel: a key block's mask column (its list of query tiles) is worked off in parts of
    // col_part_len tiles: work-group blockIdx takes part blockIdx / (BH * key blocks), leaves at
    // once where colcnt (the columns' lengths, from col_count_kernel) says the list ends before its
    // part, and adds to dK, dV atomically where the column has several parts (col_count_kernel
    // cleared those rows).  col_part_len = 0: whole columns, one work-group each, no counts.
    int col_part_len;
    int32_t* colcnt;
    int list_cap;
    const int32_t* fwd_gflag; const unsigned int* fwd_scal;   // (fwd_scal[2] = rows per row group of the forward's flags)
    int32_t* kcnt;        // backward [BH][N]: entries in each key's list
    int32_t* nplain;      // backward: number of row groups that stay with dq_kernel / dkdv_kernel
    int32_t* mask_parts;  // backward [MASK_PARTS]: set bits of the whole mask, partial sums
    void* klist;          // backward [BH][N][KEY_LIST_CAP] KeyEntry
    LogEntry* klog;       // backward [BH][N][LOG_PER_ROW], in segments of LOG_ROWS rows (where the 16-bit copies were: they are read no more)
    int32_t* log_cnt;     // backward [BH][MAX_LOG_SEGMENTS]: entries in each segment
    int32_t* hub_cnt;     // backward [BH]: hub keys of the head
    int32_t* hub_key;     // backward [BH][N]: the hub keys
    int32_t* hub_off;     // backward [BH][N]: where a hub key's part of hub_index starts
    uint32_t* hub_index;  // backward [BH][N][LOG_PER_ROW]: log entries by key (where the backward's own row lists were)
    int32_t* oflag;       // [BH][T] 1 = some row of this 64-row block has more candidates than its lists hold
    unsigned long long* stats;
    // bits of non-negative floats kept in the workspace (atomicMax on the bit patterns):
    // scal[0] = max |dO| rounded up to a power of two (the backward uses dO divided by it: exact)
    // scal[1] = forward: number of row groups left to out_kernel (a plain counter)
    // scal[2] = forward: rows per row group of its gather flags (for a backward that is handed the forward's lists)
    unsigned int* scal;
    int BH, N, T, W;
    int causal;
    HeadConsts hc;        // the constants of the call's single alpha
    const HeadConsts* hc_table;   // [H] per-head constants, or null
    int H;
    float inv_sqrt_d;
    float tol;
    int max_sweeps;
};

EA_DEV HeadConsts head_consts(const Params& p, int bh) { return p.hc_table ? p.hc_table[bh % p.H] : p.hc; }

// Consecutive block ids are dealt round-robin to the 8 XCDs (each with its own L2).  When the
// number of heads divides by 8 every XCD gets whole heads, so the work-groups that run together
// on one XCD stream the same K/V tiles.  Within a head the longest (causal: last) tiles go first.
EA_DEV void map_block(int bid, int BH, int ntile, int& bh, int& I) {
    int lin = bid;
    if ((BH & 7) == 0) {
        const int per = (BH >> 3) * ntile;
        lin = (bid & 7) * per + (bid >> 3);
    }
    bh = lin / ntile;
    I = ntile - 1 - (lin % ntile);
}

// y > 0:  y^r, y^(r-1), y^(r-2)  with r = 1/(alpha-1)
template <int AM> EA_DEV float pow_r(float y, float r) {
    if constexpr (AM == ALPHA_15) return y * y;
    else if constexpr (AM == ALPHA_20) return y;
    else return __builtin_amdgcn_exp2f(r * __builtin_amdgcn_logf(y));
}
// (alpha > 2: the exponent r - 1 is negative, at least -1/2 for alpha <= 3, and y^(r-1) grows
// without limit as y falls to zero.  y is held at or above 1e-6, about the accuracy to which an fp32
// score difference is known anyway, so that the result stays below 1e3 and its products with dP - delta
// inside the range of the fp16 operands of the backward's second-stage products.)
template <int AM> EA_DEV float pow_r1(float y, float r) {
    if constexpr (AM == ALPHA_15) return y;
    else if constexpr (AM == ALPHA_20) return 1.f;
    else return __builtin_amdgcn_exp2f((r - 1.f) * __builtin_amdgcn_logf(r < 1.f ? fmaxf(y, 1e-6f) : y));
}
// U = (rho y)^(r-1) from a y in units of rho (general alpha; lrho_u = log2(rho^(r-1)))
EA_DEV float pow_r1_rho(float y, float r, float lrho_u) {
    return __builtin_amdgcn_exp2f(fmaf(r - 1.f, __builtin_amdgcn_logf(r < 1.f ? fmaxf(y, 1e-6f) : y), lrho_u));
}
template <int AM> EA_DEV float pow_r2(float y, float r) {
    if constexpr (AM == ALPHA_15) return 1.f;
    else if constexpr (AM == ALPHA_20) return 0.f;
    else return __builtin_amdgcn_exp2f((r - 2.f) * __builtin_amdgcn_logf(y));
}

// Walk over `ntiles` streamed tiles.  issue(it, buf) starts the direct global->LDS loads of tile
// `it` into the buffer set at `buf`; compute(it, buf) does the math on it.
// NBUF == 2: the loads of tile it+1 fly under the math of tile it, one barrier per tile.  The two
// buffer sets must be two distinct __shared__ variables: the compiler gives each LDS variable its
// own alias scope, and only then does it refrain from making every LDS read of the tile being
// worked on wait for the loads in flight into the other set.
// NBUF == 1: half the LDS; loads and math alternate (other work-groups on the CU fill the gaps).
template <int NBUF, class IssueF, class ComputeF>
EA_DEV void stream_tiles(int ntiles, char* buf0, char* buf1, IssueF issue, ComputeF compute) {
    if constexpr (NBUF == 2) {
        if (ntiles > 0) issue(0, buf0);
        for (int it = 0; it < ntiles; it += 2) {
            wait_loads();
            __syncthreads();     // tile `it` has landed for every wave; everyone is done with tile it-1
            if (it + 1 < ntiles) issue(it + 1, buf1);
            compute(it, buf0);
            if (it + 1 >= ntiles) break;
            wait_loads();
            __syncthreads();
            if (it + 2 < ntiles) issue(it + 2, buf0);
            compute(it + 1, buf1);
        }
        __syncthreads();
    } else {
        for (int it = 0; it < ntiles; ++it) {
            issue(it, buf0);
            wait_loads();
            __syncthreads();
            compute(it, buf0);
            __syncthreads();
        }
    }
}

// The same walk with two tile bodies: tiles [0, n1) go to compute1, tiles [n1, n) to compute2
// (n1 even, or n1 == n), as two loops one after the other that share the double buffer: the first
// tile of the second loop is loaded under the last tile of the first.  Two loops rather than a
// choice per tile because accumulators pinned to registers by assembly statements must not meet at
// a join inside the loop (the compiler then copies all of them on one of the two paths, every tile).
template <class IssueF, class Compute1, class Compute2>
EA_DEV void stream_tiles_split(int n1, int n, char* buf0, char* buf1, IssueF issue, Compute1 compute1, Compute2 compute2) {
    if (n > 0) issue(0, buf0);
    int it = 0;
    for (; it < n1; it += 2) {
        wait_loads();
        __syncthreads();
        if (it + 1 < n) issue(it + 1, buf1);
        compute1(it, buf0);
        if (it + 1 >= n1) { it = n1; break; }        // only when n1 == n is odd
        wait_loads();
        __syncthreads();
        if (it + 2 < n) issue(it + 2, buf0);
        compute1(it + 1, buf1);
    }
    for (; it < n; it += 2) {
        wait_loads();
        __syncthreads();
        if (it + 1 < n) issue(it + 1, buf1);
        compute2(it, buf0);
        if (it + 1 >= n) break;
        wait_loads();
        __syncthreads();
        if (it + 2 < n) issue(it + 2, buf0);
        compute2(it + 1, buf1);
    }
    __syncthreads();
}

// Waits until at most K vector-memory operations of the wave are outstanding (loads, direct loads to LDS and stores alike)
template <int K> EA_DEV void wait_vm_at_most() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(K) : "memory"); }

// Executed-work counters.  The workspace starts with STATS_COPIES copies of the STATS_WORDS
// counters (a counter's value is the sum over the copies).  The waves of a group first add into
// LDS; one thread per counter then issues one global atomic, aimed at the copy picked by the
// block id, so that the atomics of groups finishing together fall on different cache lines
// (tens of thousands of atomics on one line cost more than a small kernel's whole run time).
constexpr int STATS_WORDS = 16, STATS_COPIES = 64;
template <int K>
EA_DEV void flush_counters(unsigned long long* blk, unsigned long long* stats, const int (&slot)[K],
                           const unsigned long long (&val)[K], int tid, int lane) {
    __syncthreads();
    if (tid < K) blk[tid] = 0ull;
    __syncthreads();
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (val[k]) atomicAdd(&blk[k], val[k]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tid == k && blk[k]) atomicAdd(&stats[(blockIdx.x & (STATS_COPIES - 1)) * STATS_WORDS + slot[k]], blk[k]);
}

// Union of `rows` mask rows (LDS, `W` words each) -> ascending list of tile indices in LDS.
// Called by all threads; the first wave does the work.  Uses one wave-wide exclusive scan of
// the per-word popcounts (W <= 64).
template <class ListT>
EA_DEV void build_tile_list(const uint32_t* words, int rows, int W, ListT* list, int* count, int tid) {
    __syncthreads();
    if (tid < 64) {
        uint32_t u = 0;
        if (tid < W)
            for (int r = 0; r < rows; ++r) u |= words[r * W + tid];
        const int cnt = __popc(u);
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(incl, off);
            if (tid >= off) incl += t;
        }
        int pos = incl - cnt;
        while (u) {
            const int b = __ffs(u) - 1;
            u &= u - 1;
            list[pos++] = (ListT)(tid * 32 + b);
        }
        if (tid == 63) *count = incl;
    }
    __syncthreads();
}

EA_DEV bool mask_bit(const uint32_t* words, int W, int row, int j) {
    return (words[row * W + (j >> 5)] >> (j & 31)) & 1u;
}

// Hide keys above the diagonal: element (tile row, owned row) of a stage-1 result with
// streamed index s_idx = s0 + trow and owned index o_idx = o0 + 32 qb + n.
// KEYS_STREAMED: streamed rows are keys (hide when key > query), else streamed rows are queries.
template <int QB, bool KEYS_STREAMED>
EA_DEV void causal_hide(f32x16 (&C)[2][QB], int s0, int o0, int lane) {
    const int n = lane & 31, h = lane >> 5;
    // hide when (s0 + trow) > (o0 + 32 qb + n)   [keys streamed]   i.e. trow > lim
    //        or (o0 + 32 qb + n) > (s0 + trow)   [queries streamed] i.e. trow < lim
    const int lim0 = o0 + n - s0 - 8 * h;      // compare 32 kb + 16 (v/8) + v%8 against lim0 + 32 qb
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = 32 * kb + 16 * (v >> 3) + (v & 7) - 32 * qb;   // compile-time constant
                const bool hide = KEYS_STREAMED ? (t > lim0) : (t < lim0);
                if (hide) C[kb][qb][v] = -INFINITY;
            }
}

}  // namespace ea
