// Device-side helpers shared by the HIP kernels (gfx950 / CDNA4 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/infllmv2.h"

namespace infllmv2 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Geometry the kernels are specialised for ("Hyper-Parameter Recommendation": p=32, s=16; m=64).
constexpr int kHeadDim = 128;
constexpr int kBlock = 64;    // m
constexpr int kKernel = 32;   // p
constexpr int kStride = 16;   // s
constexpr int kMaxTopk = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kScoreFloor = 7.888609052210118e-31f;  // 2^-100, floor of a relevance score
constexpr float kScoreCeil = 1.2676506002282294e30f;   // 2^100, ceiling (only the approximate LSE can reach it)

// Host+device view of the call: everything a kernel needs besides its own buffers.
struct Dims {
    int32_t Hq, Hkv, G;
    int32_t topk, n_init, n_local;
    int32_t batch, max_seqlen;
    float scale_log2;   // softmax_scale * log2(e)
    int32_t rho;        // coarse / fine kernel stride of the approximate log-sum-exp; 1 = exact
    int32_t n_q;        // decode-side kernels: query tokens per sequence (1 = plain decode, n = draft verification)
    uint32_t n_q_inv;   // floor(2^32 / n_q) + 1: i / n_q = the high word of i * n_q_inv, for n_q > 1 and i < 65536
    int32_t shared_q;   // prefill selection: 1 = one block set per 64-token query block (comparison variant)
    int32_t fill;       // 1 = also clear the rows of sequences shorter than max_seqlen (see internal.h)
};

struct Tensor {          // strides in elements
    __bf16 *ptr;
    int64_t sb, sh, st;
};

struct AppendArgs {      // the cache append folded into the first kernel of a fused decode step
    Tensor k_new, v_new, k, v;
};
struct AttendArgs {      // the per-block attention folded into the top-k kernel of a fused decode step
    Tensor k, v;
    const uint64_t *tree_mask;                        // verification only, else null
    bool fused;                                       // out: false = only the top-k ran (too many rows to repeat it per block)
    float *o_part;
    float2 *ml_part;
};

// A kernel's arguments, asked for together before anything else is done: left to itself the compiler loads each where it is first used, one
// round trip to memory after another.
template <typename A, typename... T>
__device__ inline void arguments_arrive(const A &a, const T &...x) {
    if constexpr (sizeof...(x) < 11) arguments_arrive(a, x..., a);
    else [](const auto &x0, const auto &x1, const auto &x2, const auto &x3, const auto &x4, const auto &x5, const auto &x6, const auto &x7,
            const auto &x8, const auto &x9, const auto &x10, const auto &x11) __attribute__((always_inline)) {
        asm volatile("" ::"s"(x0), "s"(x1), "s"(x2), "s"(x3), "s"(x4), "s"(x5), "s"(x6), "s"(x7), "s"(x8), "s"(x9), "s"(x10), "s"(x11));
    }(a, x...);
}

// A word at a uniform address that nothing in the launch writes: a scalar load, also behind assembly, which the compiler takes to write memory.
__device__ inline int32_t uniform_load(const int32_t *p) {
    return *(const __attribute__((address_space(4))) int32_t *)(uintptr_t)p;
}

// Number of complete semantic kernels of a sequence of l tokens (p=32, s=16).
__host__ __device__ inline int32_t num_kernels(int32_t l) {
    return l < kKernel ? 0 : (l - kKernel) / kStride + 1;
}

// Number of coarse kernels (ratio rho) all of whose fine kernels rho*c + 2r, r < rho, lie among the
// first n fine kernels ("Efficient Top-K Implementation": coarse-grained semantic kernels).
__host__ __device__ inline int32_t num_coarse(int32_t n, int32_t rho) {
    return n < 2 * rho - 1 ? 0 : (n - (2 * rho - 1)) / rho + 1;
}

// fp64 -> bf16, round to nearest even with a single rounding: first round-to-odd to fp32
// (24 bits keep a sticky bit), then nearest-even to 8 bits.
__device__ inline uint16_t f64_to_bf16_rne(double x) {
    float f = (float)x;
    uint32_t u = __float_as_uint(f);
    double fd = (double)f;
    if (fd != x) {
        if (fabs(fd) > fabs(x)) u -= 1u;   // back to the truncated magnitude
        u |= 1u;                           // inexact: make the last bit odd
    }
    uint32_t r = u + 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(r >> 16);
}

// Two channels of a semantic kernel from their 32 rows, a bf16 pair each: the sum runs in fp64 in token order, exact for bf16 inputs, and is rounded
// once.  Wherever a kernel is built, by compress_keys or by the step whose token completes it, these are its bits.
__device__ __forceinline__ uint32_t kernel_mean(const uint32_t (&row)[kKernel]) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int t = 0; t < kKernel; ++t) {
        s0 += (double)__uint_as_float(row[t] << 16);
        s1 += (double)__uint_as_float(row[t] & 0xffff0000u);
    }
    return (uint32_t)f64_to_bf16_rne(s0 / (double)kKernel) | ((uint32_t)f64_to_bf16_rne(s1 / (double)kKernel) << 16);
}

// 16x16x32 bf16 MFMA, D = A*B + C.
//   A is 16(M) x 32(K): lane l holds row l%16, k = 8*(l/16) .. 8*(l/16)+7
//   B is 32(K) x 16(N): lane l holds column l%16, same k range
//   C/D is 16 x 16:     lane l holds column l%16, rows 4*(l/16) .. 4*(l/16)+3
__device__ inline f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ inline bf16x8 load8(const __bf16 *p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p));
}

__device__ inline bf16x8 zero8() {
    uint4 z = {0u, 0u, 0u, 0u};
    return __builtin_bit_cast(bf16x8, z);
}

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
// ln(2^m x), x > 0: the log-sum-exp of a row from its reference and sum.  The hardware's logarithm comes out low, on average by half a unit in
// its last place, which for x far from 1 counts as much as the result's own rounding; so x's exponent goes to m, and what that
// sum rounds off to the logarithm of the rest.  Against 64 bits, root mean square: 32K tokens,
// G = 16, 3.6e-7 -> 1.7e-7, of which the rounding of results from 4 to 8 is 1.4e-7 (4.2e-7 where the walks begin inside their lists: the
// sums are then referred to a block nearer the largest score).
__device__ inline float lse_of(float m, float x) {
    const float e = (float)__builtin_amdgcn_frexp_expf(x), s = m + e, b = s - m;
    const float rest = ((m - (s - b)) + (e - b)) + fast_log2(__builtin_amdgcn_frexp_mantf(x));
    return __builtin_fmaf(s, kLn2, rest * kLn2);
}

// Reduce over the four 16-lane groups of a wavefront (lanes l, l^16, l^32, l^48): two lane swaps, each of which puts
// the two halves to be combined side by side in every lane (a shuffle would be an LDS round trip of 60 to 70 ns).
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
template <typename F>
__device__ inline float xgroup_reduce(float v, F f) {
    const u32x2_t a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const u32x2_t b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ inline float xgroup_max(float v) {
    return xgroup_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ inline float xgroup_sum(float v) {
    return xgroup_reduce(v, [](float a, float b) { return a + b; });
}
// Sum of x w over the four groups, in the first of them only: one product of each pair unrounded (an fma).
__device__ inline float xgroup_dot(float x, float w) {
    const float p = x * w;
    const u32x2_t a = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(p), false, false);
    const float v = __builtin_fmaf(x, w, __uint_as_float(a[1]));              // even groups: with the next one's product
    const u32x2_t b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Reduce over the 16 lanes of a group (a DPP row): four rotations, every lane ends with the result.
template <int kCtrl>
__device__ inline float dpp_rotate(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, false));
}
template <typename F>
__device__ inline float row_reduce(float v, F f) {
    v = f(v, dpp_rotate<0x128>(v));
    v = f(v, dpp_rotate<0x124>(v));
    v = f(v, dpp_rotate<0x122>(v));
    return f(v, dpp_rotate<0x121>(v));
}

// Top-k by counting (used by the pick kernels).  An element is the 64-bit word
// key << 32 | ~block: larger word = better element, ties go to the lower block index.
constexpr uint64_t kPickValid = 1ull << 32;               // smallest word of a real candidate

// number of words in w[0..n) (n a multiple of 4, 16-byte aligned) that are larger than x; sixteen
// words per step, all loaded before any is compared (a step costs one LDS latency, not eight)
__device__ inline int count_larger(const uint64_t *w, int n, uint64_t x) {
    int c0 = 0, c1 = 0;
    int j = 0;
    for (; j + 16 <= n; j += 16) {
        ulonglong2 a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = *reinterpret_cast<const ulonglong2 *>(w + j + 2 * i);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            c0 += a[i].x > x ? 1 : 0;
            c1 += a[i].y > x ? 1 : 0;
        }
    }
    for (; j < n; j += 4) {
        const ulonglong2 a = *reinterpret_cast<const ulonglong2 *>(w + j);
        const ulonglong2 bq = *reinterpret_cast<const ulonglong2 *>(w + j + 2);
        c0 += (a.x > x ? 1 : 0) + (bq.x > x ? 1 : 0);
        c1 += (a.y > x ? 1 : 0) + (bq.y > x ? 1 : 0);
    }
    return c0 + c1;
}

// The word of block j with the given score: candidates are the blocks n_init .. jc_max; a candidate
// without any visible kernel (-inf) gets key 1, below every real score (>= 2^-100) and above "none".
__device__ inline uint64_t pick_element(float score, int j, int n_init, int jc_max) {
    const uint32_t kj = score == -INFINITY ? 1u : __float_as_uint(score);
    const uint32_t key = (j >= n_init && j <= jc_max) ? kj : 0u;
    return ((uint64_t)key << 32) | (uint32_t)~j;
}

// Wavefront top-n of distinct 64-bit words, no serial rounds.  Lane l brings NE words; words below
// kPickValid are not candidates.  Returns in lane c < n the c-th largest candidate (0 when there are
// fewer than c + 1); n <= 64.  An element of the top n can only sit in a lane whose own maximum is
// among the n largest lane maxima, and it is at least tau, the n-th largest lane maximum: rank the 64
// lane maxima by counting, let the n best lanes publish their words >= tau (a handful), rank those by
// counting.  lds: 64 + topk_cand_cap(n, NE) words that belong to this wavefront alone.
__host__ __device__ inline int topk_cand_cap(int n, int ne) { return (n * ne + 3) & ~3; }

template <int NE>
__device__ inline uint64_t wave_topk(const uint64_t (&el)[NE], int n, uint64_t *lds, int lane) {
    uint64_t *tmax = lds, *cand = lds + 64;
    uint64_t best = 0ull;
#pragma unroll
    for (int s = 0; s < NE; ++s) best = el[s] > best ? el[s] : best;
    tmax[lane] = best;
    __builtin_amdgcn_wave_barrier();
    const bool real = best >= kPickValid;
    const int lrank = count_larger(tmax, 64, best);
    const bool finalist = real && lrank < n;
    uint64_t tau = kPickValid;                            // when fewer than n lanes hold a candidate
    const uint64_t who = __ballot(real && lrank == n - 1);
    if (who) {
        const int src = __builtin_ctzll(who);
        tau = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(best >> 32), src) << 32) |
              (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)best, src);
    }
    int n_cand = 0;
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int s = 0; s < NE; ++s) {
        const bool pub = finalist && el[s] >= tau;
        const uint64_t m = __ballot(pub);
        if (pub) cand[n_cand + __popcll(m & below)] = el[s];
        n_cand += __popcll(m);
    }
    const int n_cand4 = (n_cand + 3) & ~3;                // <= topk_cand_cap(n, NE)
    if (lane < n_cand4 - n_cand) cand[n_cand + lane] = 0ull;
    tmax[lane] = 0ull;                                    // the ranks are known: reuse as the result row
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < n_cand; i += 64) {
        const uint64_t e = cand[i];
        const int beaten = count_larger(cand, n_cand4, e);
        if (beaten < n) tmax[beaten] = e;
    }
    __builtin_amdgcn_wave_barrier();
    const uint64_t res = lane < n ? tmax[lane] : 0ull;
    __builtin_amdgcn_wave_barrier();
    return res;
}

// Largest value over a wavefront (uniform).
__device__ inline uint32_t wave_max_u32(uint32_t x) {
    auto step = [&](uint32_t y) { x = y > x ? y : x; };
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false));   // rotations inside the 16-lane rows
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false));
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false));
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
    return max(max(r0, r1), max(r2, r3));
}

// The n largest of the keys a wavefront holds (one per lane; 0 = not a candidate, at least n candidates, n >= 1), as a bit
// mask; ties go to the lower lane.  top: the largest key.  Bisection on the key: a step is a vector compare and scalar
// counting, and it ends early once a threshold splits off exactly n keys.  The first threshold lies a factor of 8 below the
// largest key, which in practice leaves 2^25 patterns instead of 2^30: about ten steps on scores that differ in the second
// digit, 32 at most.
// Bound by the chain of a step, eleven instructions with one branch; a threshold that splits off exactly n closes the interval instead
// of leaving the loop, which took a second branch and six scalar instructions.  Selection: 777 tokens (top-k 8, G = 16)
// 7.3 -> 6.8 us, 2048 (G = 4) 8.2 -> 7.5, 2 x 4096 (G = 8) 23.0 -> 20.6; two or four steps per branch: the same.
__device__ inline void pick_by_bisection(uint32_t key, uint32_t top, int n, uint64_t &chosen) {
    uint32_t lo = 1u, hi = top + 1u;                      // count(key >= lo) >= n >= count(key >= hi)
    uint32_t mid = top > (3u << 23) + 1u ? top - (3u << 23) : lo + ((hi - lo) >> 1);
    while (hi - lo > 1u) {                                // (as uint32: 0 once lo = hi)
        const int cnt = __popcll(__ballot(key >= mid));
        lo = cnt >= n ? mid : lo;
        hi = cnt > n ? hi : mid;
        mid = lo + ((hi - lo) >> 1);
    }
    const uint64_t above = __ballot(key > lo), eq = __ballot(key == lo);      // the keys above lo, and the first of those equal to it
    const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(eq >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq, 0u));
    chosen = above | __ballot(key == lo && before < n - __popcll(above));
}

// Sorted 64-bit words, sixteen to a row of lanes, largest first.  A step is a move of both halves across the row, a compare and two selects, about 50
// cycles; nothing goes through LDS, and a wavefront that runs alone needs no barrier.  (Maxima and minima of the words as doubles: the same.)
template <int kCtrl>
__device__ inline uint64_t row_move64(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, kCtrl, 0xf, 0xf, false);      // (no value for lanes without a source: there are none)
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), kCtrl, 0xf, 0xf, false);
    return (uint64_t)hi << 32 | lo;
}
constexpr int kSwap1 = 0xb1, kSwap2 = 0x4e, kMirror4 = 0x1b, kMirror8 = 0x141, kMirror16 = 0x140, kSwap8 = 0x128;   // lanes i ^ 1, 2, 3, 7, 15, 8
__device__ inline uint64_t keep_larger(uint64_t x, uint64_t y, bool larger) { return (y > x) == larger ? y : x; }
__device__ inline uint64_t row_clean(uint64_t x, int lane) {               // two runs of four end to end, one descending, one ascending -> sorted, twice a row
    x = keep_larger(x, row_move64<kMirror8>(row_move64<kMirror4>(x)), (lane & 4) == 0);
    x = keep_larger(x, row_move64<kSwap2>(x), (lane & 2) == 0);
    return keep_larger(x, row_move64<kSwap1>(x), (lane & 1) == 0);
}
__device__ inline uint64_t row_sort64(uint64_t x, int lane) {
    x = keep_larger(x, row_move64<kSwap1>(x), (lane & 1) == 0);
    x = keep_larger(x, row_move64<kMirror4>(x), (lane & 2) == 0);
    x = keep_larger(x, row_move64<kSwap1>(x), (lane & 1) == 0);
    x = keep_larger(x, row_move64<kMirror8>(x), (lane & 4) == 0);
    x = keep_larger(x, row_move64<kSwap2>(x), (lane & 2) == 0);
    x = keep_larger(x, row_move64<kSwap1>(x), (lane & 1) == 0);
    x = keep_larger(x, row_move64<kMirror16>(x), (lane & 8) == 0);
    return row_clean(x, lane);
}
// the sixteen largest of two sorted rows
__device__ inline uint64_t row_merge64(uint64_t a, uint64_t b, int lane) {
    uint64_t x = keep_larger(a, row_move64<kMirror16>(b), true);
    x = keep_larger(x, row_move64<kSwap8>(x), (lane & 8) == 0);
    return row_clean(x, lane);
}
// the sixteen largest of rows 0 and 1, and of rows 2 and 3, in both
__device__ inline uint64_t row_pairs_merge64(uint64_t x, int lane) {
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32), false, false);
    return row_merge64((uint64_t)hi[0] << 32 | lo[0], (uint64_t)hi[1] << 32 | lo[1], lane);
}
// the sixteen largest of a wavefront's four sorted rows, in every row
__device__ inline uint64_t rows_merge64(uint64_t x, int lane) {
    x = row_pairs_merge64(x, lane);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32), false, false);
    return row_merge64((uint64_t)hi[0] << 32 | lo[0], (uint64_t)hi[1] << 32 | lo[1], lane);
}

// The running picks of one row, merged with a chunk of kVPL * 64 blocks by one wavefront: lane l brings the keys (0 = not a candidate)
// of blocks j0 + l + 64 s.  picks (LDS): the n_have best so far as key << 32 | block, all blocks below j0; afterwards the n_pick best in
// ascending order of their blocks.  Ties go to the lower block.  tmp: 64 + topk_cand_cap(n_pick, kVPL + 1) words of this wavefront's own.
template <int kVPL>
__device__ inline void merge_picks(const uint32_t (&key)[kVPL], int j0, int n_have, int n_pick, uint64_t *picks, uint64_t *tmp, int lane) {
    uint64_t el[kVPL + 1];
#pragma unroll
    for (int s = 0; s < kVPL; ++s) el[s] = (uint64_t)key[s] << 32 | (uint32_t)~(j0 + lane + 64 * s);
    el[kVPL] = lane < n_have ? picks[lane] ^ 0xffffffffull : 0ull;
    const uint64_t res = wave_topk<kVPL + 1>(el, n_pick, tmp, lane) ^ 0xffffffffull;
    int rank = 0;
    for (int e = 0; e < n_pick; ++e) rank += (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)res, e) < (uint32_t)res ? 1 : 0;
    if (lane < n_pick) picks[rank] = res;
    __builtin_amdgcn_wave_barrier();
}

// How many of the other 15 lanes of a group hold an x larger than this lane's y.
template <int kR = 15>
__device__ inline int row_count_larger(uint32_t x, uint32_t y) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + kR, 0xf, 0xf, false);
    int c = o > y ? 1 : 0;
    if constexpr (kR > 1) c += row_count_larger<kR - 1>(x, y);
    return c;
}
template <typename F>
__device__ inline uint32_t row_reduce_u32(uint32_t x, F f) {
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false));
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false));
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false));
    return f(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false));
}

// merge_picks for four rows at a time, one per 16-lane group, of up to 14 (kP = 1) or 32 (kP = 2) picks each.  R (LDS): the chunk's
// scores of this lane's row, 16 kE of them; first, count: the chunk's candidates; live: the row exists; picks, n_have, n_pick as above.
// tmp: 4 * 64 words.  Returns false, with nothing changed, if a row has more than 64 elements that could enter.
// The wavefront runs alone in this (its neighbour on the SIMD multiplies), at about ten cycles an instruction, so what counts is how many there are:
// 130 a row (kP = 1) instead of 430.  A few lanes' largest elements give a threshold that n_pick of them reach: the n_pick-th
// of the 16 lanes' (of 512 random scores 26 reach it for 13 picks; beyond 14 it says too little), or, by bisection, about that of the
// 64 quarter lanes'; counting over the elements that reach it gives the order.  Ranking a row's chunk 4500 -> 2000 cycles;
// selection, top-k 16, G = 16: 5000 tokens 64 -> 55 us, 32K 613 -> 579; G = 8: 8192 118 -> 75, 32K 925 -> 585; G = 1: 16000 176 -> 108.
constexpr int kGroupPicks = 32;
inline int pick_form(const Dims &dm) { return dm.topk - dm.n_init - dm.n_local <= 14 ? 1 : 2; }   // kP; a row has no more picks
template <int kE, int kP>
__device__ inline bool merge_picks_group(const float *R, int j0, int first, int count, bool live, int n_have, int n_pick, uint64_t *picks,
                                         uint64_t *tmp, int lane) {
    const auto larger = [](uint32_t x, uint32_t y) { return max(x, y); };
    const int l = lane & 15;
    uint64_t *mine = tmp + 64 * (lane >> 4);
    uint64_t old[kP];                                     // key << 32 | ~block: larger is better
    uint32_t lo = 0xffffffffu;
#pragma unroll
    for (int i = 0; i < kP; ++i) {
        old[i] = l + 16 * i < n_have ? picks[l + 16 * i] ^ 0xffffffffull : 0ull;
        if (l + 16 * i < n_have) lo = min(lo, (uint32_t)(old[i] >> 32));
    }
    lo = n_have == n_pick ? ~row_reduce_u32(~lo, larger) + 1u : 1u;          // larger than the smallest pick
    constexpr int kSub = kP == 1 ? 1 : 4;
    uint32_t key[kE], best[kSub];
#pragma unroll
    for (int i = 0; i < kSub; ++i) best[i] = 0u;
#pragma unroll
    for (int i = 0; i < kE / 4; ++i) {                    // (every lane holds some of a chunk that is not full)
        const int at = 4 * (l + 16 * i);
        const int4 x = *reinterpret_cast<const int4 *>(R + at);
        const uint32_t from = (uint32_t)(j0 + at - first);
        const int b[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {                     // (a block without a visible kernel, -inf, comes last)
            const uint32_t k = from + e < (uint32_t)(live ? count : 0) ? (uint32_t)max(b[e], 1) : 0u;
            key[4 * i + e] = k;
            best[e % kSub] = max(best[e % kSub], k);
        }
    }
    if constexpr (kP == 1) {
        lo = max(lo, ~row_reduce_u32(row_count_larger<>(best[0], best[0]) < n_pick ? ~best[0] : 0u, larger));
    } else {
        const uint32_t top = row_reduce_u32(max(max(best[0], best[1]), max(best[2], best[3])), larger);
        uint32_t hi = max(top, lo) + 1u, mid = top > lo + (3u << 23) ? top - (3u << 23) : lo;   // first an eighth of the largest
        for (int i = 0; i < 12; ++i) {
            uint32_t c = 0u;
#pragma unroll
            for (int e = 0; e < kSub; ++e) c += best[e] >= mid ? 1u : 0u;
            const bool ok = row_reduce_u32(c, [](uint32_t x, uint32_t y) { return x + y; }) >= (uint32_t)n_pick;
            lo = ok ? mid : lo;
            hi = ok ? hi : mid;
            mid = lo + ((hi - lo) >> 1);
        }
    }
    int c = 0;
#pragma unroll
    for (int i = 0; i < kE; ++i) c += key[i] >= lo ? 1 : 0;
    int incl = c;                                         // up to this lane of the group
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, true);
    const int r0 = __builtin_amdgcn_readlane(incl, 15), r1 = __builtin_amdgcn_readlane(incl, 31);
    const int r2 = __builtin_amdgcn_readlane(incl, 47), r3 = __builtin_amdgcn_readlane(incl, 63);
    const int most = max(max(r0, r1), max(r2, r3)) + n_have;
    if (most == n_have) return true;
    if (most > 64) return false;
    const int total = (lane < 32 ? (lane < 16 ? r0 : r1) : (lane < 48 ? r2 : r3)) + n_have;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (l + 16 * i >= total) mine[l + 16 * i] = 0ull;
#pragma unroll
    for (int i = 0; i < kP; ++i)
        if (l + 16 * i < n_have) mine[l + 16 * i] = old[i];
    int at = n_have + incl - c;
#pragma unroll
    for (int i = 0; i < kE; ++i)
        if (key[i] >= lo) mine[at++] = (uint64_t)key[i] << 32 | (uint32_t)~(j0 + 4 * (l + 16 * (i / 4)) + i % 4);
    __builtin_amdgcn_wave_barrier();                      // same wavefront: LDS keeps the order
    uint64_t w[4];
    int rank[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[i] = mine[l + 16 * i];
        rank[i] = 0;
    }
    auto count_from = [&](auto parts) __attribute__((always_inline)) {
        for (int e = 0; e < most; e += 4) {
            const ulonglong2 x = *reinterpret_cast<const ulonglong2 *>(mine + e), y = *reinterpret_cast<const ulonglong2 *>(mine + e + 2);
#pragma unroll
            for (int i = 0; i < decltype(parts)::value; ++i)
                rank[i] += ((x.x > w[i] ? 1 : 0) + (x.y > w[i] ? 1 : 0)) + ((y.x > w[i] ? 1 : 0) + (y.y > w[i] ? 1 : 0));
        }
    };
    if (most <= 32) count_from(std::integral_constant<int, 2>{});
    else count_from(std::integral_constant<int, 4>{});
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (w[i] != 0ull && rank[i] < n_pick) mine[rank[i]] = w[i];           // (no two words are equal)
    __builtin_amdgcn_wave_barrier();
    const int n = min(total, n_pick);
    uint64_t p[kP];
#pragma unroll
    for (int i = 0; i < kP; ++i) p[i] = l + 16 * i < n ? mine[l + 16 * i] : 0ull;
#pragma unroll
    for (int i = 0; i < kP; ++i) {                        // ~block: larger is a lower block; the unused ones are 0
        int place = 0;
#pragma unroll
        for (int j = 0; j < kP; ++j) place += row_count_larger<>((uint32_t)p[j], (uint32_t)p[i]) + ((uint32_t)p[j] > (uint32_t)p[i] ? 1 : 0);
        if (l + 16 * i < n) picks[place] = p[i] ^ 0xffffffffull;
    }
    __builtin_amdgcn_wave_barrier();
    return true;
}

// The row of selected blocks of one query, ascending, padded with -1 up to topk: the first n_init, the n_pick picks (ascending), and
// lo_local .. the own one, n_sel in all.
__device__ inline void write_picks_row(const uint64_t *picks, int n_pick, int n_sel, int n_init, int lo_local, int topk,
                                       int32_t *__restrict__ o, int lane) {
    if (lane >= topk) return;
    int x = lane;
    if (lane >= n_init) x = lane < n_init + n_pick ? (int)(uint32_t)picks[lane - n_init] : lo_local + (lane - n_init - n_pick);
    o[lane] = lane < n_sel ? x : -1;
}

// The row of selected blocks of one query: lane c < n_pick brings a picked candidate block, the forced
// blocks (the first n_init and lo_local .. b_own) are added, and the n_sel blocks are written in
// ascending order, padded with -1 up to topk.
__device__ inline void write_block_row(int picked, int n_pick, int n_sel, int n_init, int lo_local, int topk,
                                       int32_t *__restrict__ o, int lane) {
    int mine = 0x7fffffff;
    if (lane < n_pick) mine = picked;
    else if (lane < n_sel) {
        const int f = lane - n_pick;
        mine = f < n_init ? f : lo_local + (f - n_init);
    }
    int rank = 0;                                         // number of selected blocks below mine
    for (int e = 0; e < n_sel; ++e) rank += __builtin_amdgcn_readlane(mine, e) < mine ? 1 : 0;
    if (lane < n_sel) o[rank] = mine;
    else if (lane < topk) o[lane] = -1;
}

// Rows max(t0, L) .. t0 + n_tok - 1 of a block-list tensor (below max_seqlen) set to -1 by one wavefront.
__device__ inline void fill_block_rows(const Dims &dm, int b, int h, int t0, int n_tok, int L, int32_t *__restrict__ block_idx,
                                       int lane) {
    const int t1 = min(t0 + n_tok, dm.max_seqlen);
    for (int t = max(t0, L); t < t1; ++t)
        if (lane < dm.topk) block_idx[(((int64_t)b * dm.Hkv + h) * dm.max_seqlen + t) * dm.topk + lane] = -1;
}

// Per-kernel timing of the bench-only build (INFLLMV2_TIMING, see timing.hip): every launch is bracketed
// by HIP events on its stream while infllmv2_timing_enable is on.  The production build compiles the
// hooks away.
#ifdef INFLLMV2_TIMING
void timing_begin(const char *kernel_name, hipStream_t stream);
void timing_end(hipStream_t stream);
#else
inline void timing_begin(const char *, hipStream_t) {}
inline void timing_end(hipStream_t) {}
#endif

// Launchers implemented in the .hip files; each returns a hipError_t as int.
int launch_compress_keys(const Dims &dm, Tensor k, Tensor ck, const int32_t *seqlens,
                         int32_t n_new_tokens, hipStream_t stream);
int launch_append_kv(const Dims &dm, Tensor k_new, Tensor v_new, Tensor k, Tensor v, const Tensor *ck,
                     const int32_t *seqlens, hipStream_t stream);   // dm.n_q rows per sequence
int launch_select_prefill(const Dims &dm, Tensor q, Tensor ck, const int32_t *seqlens,
                          int32_t *block_idx, void *ws, hipStream_t stream, float *scores_out = nullptr,
                          int32_t scores_pitch = 0);
size_t select_prefill_ws_bytes(const Dims &dm);
int launch_select_prefill16(const Dims &dm, Tensor q, Tensor ck, const int32_t *seqlens,
                            int32_t *block_idx, void *ws, hipStream_t stream, float *scores_out = nullptr,
                            int32_t scores_pitch = 0);
size_t select_prefill16_ws_bytes(const Dims &dm);
constexpr int kShortPrefill = 4096;                        // tokens: up to 255 semantic kernels (select_short.hip)
bool select_short_fits(const Dims &dm);
int launch_select_short(const Dims &dm, Tensor q, Tensor ck, const int32_t *seqlens, int32_t *block_idx, hipStream_t stream,
                        float *scores_out = nullptr, int32_t scores_pitch = 0);
int32_t select_scores_pitch(const Dims &dm);
size_t select_scores_bytes(const Dims &dm);
size_t select_shared_scores_bytes(const Dims &dm);
int launch_select_pick(const Dims &dm, const int32_t *seqlens, const float *R, int32_t nb_cap,
                       int32_t *block_idx, hipStream_t stream);
int launch_select_decode(const Dims &dm, Tensor q, Tensor ck, const int32_t *seqlens,
                         int32_t *block_idx, void *ws, hipStream_t stream, const AppendArgs *append = nullptr,
                         AttendArgs *attend = nullptr);
int launch_decode_step(const Dims &dm, Tensor q, Tensor ck, const AppendArgs &append, const int32_t *seqlens,
                       int32_t *block_idx, Tensor out, float *lse, void *ws_select, void *ws_attn,
                       hipStream_t stream);
int launch_verify_step(const Dims &dm, Tensor q, Tensor ck, const AppendArgs &append, const int32_t *seqlens,
                       const uint64_t *tree_mask, int32_t *block_idx, Tensor out, float *lse, void *ws_select,
                       void *ws_attn, hipStream_t stream);
size_t select_decode_ws_bytes(const Dims &dm);
int launch_attn_prefill(const Dims &dm, Tensor q, Tensor k, Tensor v, const int32_t *seqlens,
                        const int32_t *block_idx, Tensor out, float *lse, void *ws, hipStream_t stream);
size_t attn_prefill_ws_bytes(const Dims &dm);
int launch_attn_decode(const Dims &dm, Tensor q, Tensor k, Tensor v, const int32_t *seqlens,
                       const int32_t *block_idx, const uint64_t *tree_mask, Tensor out, float *lse, void *ws,
                       hipStream_t stream);
size_t attn_decode_ws_bytes(const Dims &dm);
int launch_attn_bwd(const Dims &dm, Tensor q, Tensor k, Tensor v, Tensor out, Tensor dout, const float *lse,
                    const int32_t *seqlens, const int32_t *block_idx, Tensor dq, Tensor dk, Tensor dv, void *ws,
                    hipStream_t stream);
size_t attn_bwd_ws_bytes(const Dims &dm);
int32_t validate_attn_decode(const infllmv2_params *prm, const infllmv2_tensor *q, const infllmv2_tensor *k,
                             const infllmv2_tensor *v, const int32_t *seqlens, int32_t batch, int32_t max_seqlen,
                             const int32_t *block_idx, const infllmv2_tensor *out, const float *lse, Dims *dm,
                             Tensor *tq, Tensor *tk, Tensor *tv, Tensor *tout);
int launch_probes(void *buf, size_t buf_bytes, double *mfma_flops, double *stream_bytes, hipStream_t stream);
int launch_probes_detail(void *buf, size_t buf_bytes, double *work, hipStream_t stream);

}  // namespace infllmv2
