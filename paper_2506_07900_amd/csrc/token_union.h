// Union of the block lists of a few consecutive query tokens, built by one wavefront in its own piece of LDS.
// Shared by the prefill attention and its backward: a wavefront that owns several tokens fetches every block
// that any of them selected once.
#pragma once
#include "common.h"

namespace infllmv2 {

constexpr int kRun = 4;                                  // tiles of a sequence that go to one XCD together

// Inclusive prefix sum over the 64 lanes (row shifts, then the row totals broadcast: no LDS round trips).
__device__ inline int wave_inclusive_sum(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// LDS of one wavefront: a bitmap of 2048 blocks with the rank of every word, then the list itself.
struct UnionLds {
    uint32_t *words, *prefix;                            // [64] each
    uint2 *list;                                         // [cap]: {block, member bits: bit t = token t selected it}
    __host__ __device__ static int cap(int n_tok, int topk) { return (n_tok * topk + 63) & ~63; }
    __host__ __device__ static size_t bytes(int n_tok, int topk) { return 512 + (size_t)cap(n_tok, topk) * sizeof(uint2); }
    __device__ explicit UnionLds(unsigned char *p)
        : words(reinterpret_cast<uint32_t *>(p)), prefix(words + 64), list(reinterpret_cast<uint2 *>(p + 512)) {}
};

// A lane's first entries of the tokens' rows, asked for before anything else is done.  A workgroup with direct fetches does so before it
// knows the sequence's length: n_ent are those that lie within the tensor (max_seqlen rows per sequence and head).
template <int NT>
struct UnionRows {
    static constexpr int kE = NT >= 4 ? NT / 4 : 1;      // entries per lane kept in registers: top-k 16; more are re-read
    int ent[kE];
    __device__ UnionRows(const int32_t *__restrict__ rows, int n_ent, int lane) {
#pragma unroll
        for (int i = 0; i < kE; ++i) ent[i] = lane + 64 * i < n_ent ? rows[lane + 64 * i] : -1;
    }
};

// Ascending union of the lists of n_tok <= NT <= 32 consecutive tokens.  rows: their n_tok * topk entries, contiguous;
// entries < 0 or > b_own are dropped, a block that a row lists twice counts once.  Returns the number of distinct
// blocks.  An entry's place is the number of set bits before its own in the bitmap, so nothing is sorted and the
// order of the rows' entries does not matter; sequences of more than 2048 blocks take several rounds.
template <int NT>
__device__ inline int build_union(const UnionRows<NT> &head, const int32_t *__restrict__ rows, int topk, int n_tok, int b_own,
                                  const UnionLds &u, int lane) {
    constexpr int kE = UnionRows<NT>::kE;
    const int n_ent = n_tok * topk;
    const uint32_t inv = (1u << 20) / (uint32_t)topk + 1u;   // entry i belongs to token i / topk (exact for i < 2048)
    int ent[kE];
#pragma unroll
    for (int i = 0; i < kE; ++i) {
        ent[i] = lane + 64 * i < n_ent && head.ent[i] <= b_own ? head.ent[i] : -1;
    }
    auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kE; ++i)
            if (ent[i] >= 0) f(ent[i], (int)(((uint32_t)(lane + 64 * i) * inv) >> 20));
        for (int at = lane + 64 * kE; at < n_ent; at += 64) {
            const int x = rows[at];
            if (x >= 0 && x <= b_own) f(x, (int)(((uint32_t)at * inv) >> 20));
        }
    };
    const int cap = UnionLds::cap(NT, topk);
    for (int i = lane; i < cap; i += 64) u.list[i] = uint2{0u, 0u};
    int cnt = 0;
    for (int base = 0; base <= b_own; base += 2048) {
        u.words[lane] = 0u;
        __builtin_amdgcn_wave_barrier();                 // same wavefront throughout: LDS keeps the order
        each([&](int x, int) {
            const uint32_t r = (uint32_t)(x - base);
            if (r < 2048u) atomicOr(&u.words[r >> 5], 1u << (r & 31u));
        });
        __builtin_amdgcn_wave_barrier();
        const int mine = __popc(u.words[lane]);
        const int incl = wave_inclusive_sum(mine);
        u.prefix[lane] = (uint32_t)(cnt + incl - mine);
        __builtin_amdgcn_wave_barrier();
        each([&](int x, int t) {
            const uint32_t r = (uint32_t)(x - base);
            if (r < 2048u) {
                const uint32_t at = u.prefix[r >> 5] + __popc(u.words[r >> 5] & ((1u << (r & 31u)) - 1u));
                u.list[at].x = (uint32_t)x;
                atomicOr(&u.list[at].y, 1u << t);
            }
        });
        cnt += __builtin_amdgcn_readlane(incl, 63);
        __builtin_amdgcn_wave_barrier();
    }
    return cnt;
}

// Where in its list of n blocks a workgroup begins its walk (which goes round).  Once a head's packed keys and values are more than an XCD's
// L2 holds, what a block costs depends on who asked for it last: workgroups that begin one after another and all walk upwards are spread
// over the whole sequence.  The `resident` workgroups of an XCD begin one walk's time / resident apart, so beginning slot / resident
// into the list puts them all near the same blocks.  The slot is counted back from a fixed tile (the launches deal tiles last first, in runs to
// the XCDs), so in one form of the kernel the order of a token's sums depends
// neither on the capacity nor on the other sequences.  Lines past L2, attention, 128K tokens,
// 2 x 16 heads: 219 -> 159 million, 4250 -> 3950 us; top-k 64, 64K 9550 -> 6740; G = 8, 32K 768 -> 688; G = 4, 32K 775 -> 630; G = 16, 32K 803
// -> 790, 16K and below: the same.  Half as many residents, or the other way round: 4310 for the first.  dq: 64K, G = 4 3490 -> 2975 us
// for the whole backward, top-k 64, G = 16 18.7 -> 16.8 ms; G = 16, top-k 16: the same.
constexpr int kFarBlocks = 128;                          // 4 MiB of packed blocks
__device__ inline int walk_start(int n, int tile, uint32_t resident, int b_own) {
    if (b_own < kFarBlocks) return 0;
    const uint32_t r = 0x40000000u - (uint32_t)tile, slot = r / (8 * kRun) * kRun + r % kRun;
    return __builtin_amdgcn_readfirstlane((int)((uint32_t)n * (slot % resident) / resident));
}

// Rows of 128 channels in LDS: a row's sixteen 16-byte pieces are stored XOR-swizzled with the row's two bit pairs exchanged.  An
// operand load takes one piece from each of 16 or 32 rows, a transposing load 32 bytes from each of 4 consecutive rows, and
// both then touch every bank once.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int row_swizzle(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }
// 4 rows x 16 channels per 16-lane group, transposed: lane i of the group gets channel i of the four rows its
// group addressed (source lane s: row s/4, channels 4(s%4) .. +3)
__device__ __forceinline__ s16x4 lds_read_tr16(const char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
}

// A tile whose columns belong to several tokens multiplies a block that only some of them selected with zeros for the
// others, and 0 * inf or 0 * NaN reaches their sums.  Such a sum is not finite, so the kernels look at their results and, when
// one is not, take the walk again once per token of a tile, with that token's blocks alone.  (A select per accumulator
// would cost every call: 487 -> 565 us for a training step on 2 x 4096 tokens, G = 8; a second copy of the walk spills.)
__device__ inline bool not_finite(const f32x4 &x) {
    const float s = (x[0] * 0.f + x[1] * 0.f) + (x[2] * 0.f + x[3] * 0.f);
    return s != s;
}

}  // namespace infllmv2
