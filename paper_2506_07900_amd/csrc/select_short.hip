// Stage 2, prefill, for sequences of up to kShortPrefill tokens: one pass over the compressed keys, one
// kernel, straight from the compressed keys to the block lists.
//
// The two-pass kernels (select_prefill16.hip, select_prefill.hip) compute every logit and its exponential
// twice, because a score 2^(z - lse) needs the log-sum-exp over all visible kernels first.  Up to 256
// semantic kernels the exponentials e = 2^(z - m) of a 16-row tile of (token, head) rows stay in the
// registers of the wavefront that computed them, and the scores follow as sum_heads e * w with one weight
// w = 1 / sum e per row: half the matrix work, half the exponentials, no log-sum-exps, packed keys or
// second and third launch in between.  Tokens that attend all of their blocks anyway (own block < top-k)
// are not scored at all.
//
// The compressed keys of a (sequence, key-value head) -- 64 KiB at most -- are copied into LDS once per
// workgroup, in MFMA operand order; its eight wavefronts then take tile after tile of tokens, each on its own.
// Reading the keys from L2 for every tile instead was bound by the half-line reads of the row-major keys
// (16 rows x 64 bytes per load): 8 tiles of 16 kernels took 10 us with every wavefront at it.
// Selection alone, us, two passes -> this: 777 tokens (top-k 8) 33 -> 6.8, 2048 42 -> 11, 4096 53 -> 21 (G = 16, 2 heads);
// 2048 G = 4 27 -> 7.5.
// Its scores are nearer to 64-bit ones than the two passes' (largest relative error over 300 to 4096 tokens and every G 2.5e-7
// against 8.4e-7; no rounded log-sum-exp in between), but not theirs: blocks whose scores tie to fp32 rounding change places, in
// 4 of 983040 rows of 8192 tokens against 1 of 921600 of 1500 to 4096.  Up to 8192 tokens it would still be faster (113 -> 51,
// G = 1 59 -> 37); longer prompts keep the lists they had.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace infllmv2 {

constexpr int kShortWaves = 8;

template <int kG, int kKT>
struct ShortCfg {
    static constexpr int kTok = 16 / kG;                  // tokens per tile
    static constexpr int kPitch = 16 * kKT + 16;          // floats of the one token a wavefront ranks at a time
    static constexpr int kStep = kKT >= 16 ? kKT / 4 : 4; // kernel tiles between the sizes the code is unrolled for
    static size_t lds_bytes(int n_c) { return (size_t)((n_c + 15) / 16) * 4096 + (size_t)kShortWaves * kPitch * sizeof(float); }
};

// kScores: the scores of every candidate block go to `scores` (infllmv2_block_scores) instead of being ranked.
template <int kG, int kKT, bool kScores>
__global__ __launch_bounds__(64 * kShortWaves, 4) void select_short_kernel(
    Dims dm, Tensor q, Tensor ck, const int32_t *__restrict__ seqlens, int32_t *__restrict__ block_idx, int32_t n_units,
    int32_t wgs, int32_t share_log2, float *__restrict__ scores, int32_t scores_pitch) {
    using C = ShortCfg<kG, kKT>;
    static_assert(64 % C::kTok == 0, "one own block per tile");
    static_assert(4 * kKT <= 64, "a block per lane in the ranking");
    extern __shared__ __align__(16) unsigned char short_smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = blockIdx.x % wgs, h = (blockIdx.x / wgs) % dm.Hkv, b = blockIdx.x / (wgs * dm.Hkv);
    const int n = lane & 15, g = lane >> 4;
    const float c = dm.scale_log2;
    int32_t L = __builtin_amdgcn_readfirstlane(seqlens[b]);
    L = L < 0 ? 0 : (L > dm.max_seqlen ? dm.max_seqlen : L);
    const int n_c = num_kernels(L);
    float *rs = reinterpret_cast<float *>(short_smem) + wave * C::kPitch;     // slot 1 + jh: score of kernel jh
    uint4 *cks = reinterpret_cast<uint4 *>(short_smem + kShortWaves * C::kPitch * sizeof(float));

    // ---- compressed keys to LDS: tile t, piece p = 4ks + g of row n at [t][ks][16g + (n ^ p)] (an operand read covers 1 KiB
    // in some order, a write's 16 pieces of a row go to 16 different bank groups) -------------------------------
    if (kScores || dm.topk <= (L - 1) / kBlock) {         // (else every token attends everything)
        const __bf16 *ckh = ck.ptr + b * ck.sb + h * ck.sh + 8 * (tid & 15);
#pragma unroll 1
        for (int r0 = tid >> 4; r0 < n_c; r0 += 4 * 4 * kShortWaves) {
            bf16x8 x[4];                                  // (rows past the last one copy it again, to its own place)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = load8(ckh + (int64_t)min(r0 + 4 * kShortWaves * i, n_c - 1) * ck.st);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = min(r0 + 4 * kShortWaves * i, n_c - 1), p = tid & 15;
                cks[(r >> 4) * 256 + (p >> 2) * 64 + (p & 3) * 16 + ((r & 15) ^ p)] = __builtin_bit_cast(uint4, x[i]);
            }
        }
    }
    for (int i = lane; i < C::kPitch; i += 64) rs[i] = -INFINITY;             // (slot 0 stays: no kernel)
    __syncthreads();

    // ---- tiles of tokens, the longest rows first ----------------------------------------------------------------
    // (with fewer than a chipful of tiles, 2^share_log2 wavefronts compute the same tile and rank a part of its tokens each)
    for (int unit = (n_units << share_log2) - 1 - (wg * kShortWaves + wave); unit >= 0; unit -= wgs * kShortWaves) {
        const int t0 = (unit >> share_log2) * C::kTok;
        const int sub = unit & ((1 << share_log2) - 1), sub_mask = (1 << share_log2) - 1;
        if (dm.fill && sub == 0) fill_block_rows(dm, b, h, t0, C::kTok, L, block_idx, lane);
        if (t0 >= L) continue;
        const int b_own = t0 / kBlock, n_blk = b_own + 1;
        const int n_sel = dm.topk < n_blk ? dm.topk : n_blk;
        const int n_init = dm.n_init < n_blk ? dm.n_init : n_blk;             // forced leading blocks
        const int lo_local = max(n_init, b_own - dm.n_local + 1);             // forced trailing: lo_local..b_own
        const int n_pick = n_sel - (n_init + (b_own - lo_local + 1));         // from the candidates n_init..lo_local-1
        int32_t *row0 = block_idx + (((int64_t)b * dm.Hkv + h) * dm.max_seqlen + t0) * dm.topk;
        const int n_tok = min(C::kTok, L - t0);
        const int n_vis_lo = num_kernels(t0 + 1), n_vis_hi = num_kernels(t0 + n_tok);
        if constexpr (kScores) {
            if (lo_local <= n_init) continue;             // no candidate
            if (n_vis_hi == 0) {                          // nothing to score: all within the first block
                for (int u = sub; u < n_tok; u += sub_mask + 1)
                    if (lane == 0) scores[(((int64_t)b * dm.Hkv + h) * dm.max_seqlen + t0 + u) * scores_pitch] = -INFINITY;
                continue;
            }
        } else if (n_sel == n_blk || n_pick <= 0) {              // every block, or the forced ones only: nothing to score
            for (int u = sub; u < n_tok; u += sub_mask + 1)
                if (lane < dm.topk) {
                    int x = lane;
                    if (n_sel < n_blk && lane >= n_init) x = lo_local + (lane - n_init);
                    row0[u * dm.topk + lane] = lane < n_sel ? x : -1;
                }
            continue;
        }
        // row n of the tile: token t0 + n / kG, head n % kG
        bf16x8 qf[4];
        {
            const __bf16 *qr = q.ptr + b * q.sb + (int64_t)min(t0 + n / kG, L - 1) * q.st + (int64_t)(h * kG + n % kG) * q.sh + 8 * g;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) qf[ks] = load8(qr + 32 * ks);
        }

        // Straight-line code for kNT kernel tiles (those past the end are masked), so that the products of one tile run
        // under the LDS reads of the next.  (All products first and the masks after them: 20.6 -> 19.4 us for 2 x 4096 tokens, G = 8, but
        // the kernels that follow it then run at a lower clock: a training step on them 480 -> 496 us back to back.)  Z = Q . CK^T: lane = kernel, accumulator entries = rows 4g .. 4g+3.
        auto run = [&](auto nt) __attribute__((always_inline)) {
            constexpr int kNT = decltype(nt)::value;
            f32x4 z[kNT];
            float m[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) m[j] = -INFINITY;
            const int t_last = (n_vis_hi - 1) >> 4;
#pragma unroll
            for (int t = 0; t < kNT; ++t) {
                const uint4 *src = cks + min(t, t_last) * 256 + 16 * g;
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc = mfma16(qf[ks], __builtin_bit_cast(bf16x8, src[64 * ks + (n ^ (4 * ks + g))]), acc);
                z[t] = acc;
                if (16 * t + 16 > n_vis_lo) {             // causal edge: some token does not see the whole tile
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (16 * t + n >= num_kernels(t0 + (4 * g + j) / kG + 1)) z[t][j] = -INFINITY;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) m[j] = fmaxf(m[j], z[t][j]);
            }
            // ---- exponentials, in place of the logits, and the row weights 1 / (G sum) ------------------------------
            float wgt[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float mr = row_reduce(m[j], [](float x, float y) { return fmaxf(x, y); }) * c;
                const float neg = mr == -INFINITY ? 0.f : -mr;
                float s = 0.f;
#pragma unroll
                for (int t = 0; t < kNT; ++t) {
                    const float e = fast_exp2(__builtin_fmaf(z[t][j], c, neg));
                    z[t][j] = e;
                    s += e;
                }
                wgt[j] = 1.f / (row_reduce(s, [](float x, float y) { return x + y; }) * kG);
            }
            // ---- scores: mean over the heads of a token.  Lane (n, g) ends up with
            //   G <= 4: entry p of tile t = kernel 16t + n for token (4g + 4p/kPer) / G
            //   G = 8:  entry 0 of tile t (t even) = kernel 16(t + g%2) + n for token g/2
            //   G = 16: entry 0 of tile t (4 | t) = kernel 16(t + g) + n
            constexpr int kPer = kG >= 4 ? 1 : 4 / kG, kRows = 4 / kPer;
#pragma unroll
            for (int t = 0; t < kNT; ++t)
#pragma unroll
                for (int p = 0; p < kPer; ++p) {
                    float v = 0.f;
#pragma unroll
                    for (int j = 0; j < kRows; ++j) v = __builtin_fmaf(z[t][p * kRows + j], wgt[p * kRows + j], v);
                    z[t][p] = v;
                }
            constexpr int kPack = kG == 16 ? 4 : kG == 8 ? 2 : 1;                  // tiles side by side in the lane groups
            if constexpr (kG >= 8) {
#pragma unroll
                for (int t = 0; t < kNT; t += 2) {
                    const u32x2_t x = __builtin_amdgcn_permlane16_swap(__float_as_uint(z[t][0]), __float_as_uint(z[t + 1][0]), false, false);
                    z[t][0] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
                }
            }
            if constexpr (kG == 16) {
#pragma unroll
                for (int t = 0; t < kNT; t += 4) {
                    const u32x2_t x = __builtin_amdgcn_permlane32_swap(__float_as_uint(z[t][0]), __float_as_uint(z[t + 2][0]), false, false);
                    z[t][0] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
                }
            }
            // ---- token by token: scores to LDS, 5/4 max over kernels, top-k, the row ---------------------------------
#pragma unroll
            for (int u = 0; u < C::kTok; ++u) {
                if (u >= n_tok) break;                    // uniform
                if (C::kTok > 1 && (u & sub_mask) != sub) continue;
                const int n_vis = num_kernels(t0 + u + 1);
                const bool mine = kG == 16 || (kG == 8 ? g >> 1 == u : g == u / kPer);
                const int off = 16 * (kG == 16 ? g : kG == 8 ? g & 1 : 0) + n;
                if (mine) {
#pragma unroll
                    for (int t = 0; t < kNT; t += kPack) {
                        const int jh = 16 * t + off;
                        const float v = fminf(fmaxf(z[t][kPer > 1 ? u % kPer : 0], kScoreFloor), kScoreCeil);
                        rs[1 + jh] = jh < n_vis ? v : -INFINITY;
                    }
                }
                __builtin_amdgcn_wave_barrier();          // same wavefront: LDS keeps the order
                // The n_pick best by bisection on the scores' bit patterns (positive floats order like integers).
                uint32_t key = 0u;                        // of block `lane`
                if (lane >= n_init && lane < lo_local) {  // kernels 4 lane - 1 .. 4 lane + 3 = slots 4 lane .. 4 lane + 4
                    const f32x4 x = *reinterpret_cast<const f32x4 *>(&rs[4 * lane]);
                    const float r = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), rs[4 * lane + 4]);
                    key = (uint32_t)max(__float_as_int(r), 1);                // a block without a visible kernel (-inf) comes last
                    if constexpr (kScores) scores[(((int64_t)b * dm.Hkv + h) * dm.max_seqlen + t0 + u) * scores_pitch + lane] = r;
                }
                __builtin_amdgcn_wave_barrier();
                if constexpr (kScores) continue;
                uint64_t chosen;
                pick_by_bisection(key, wave_max_u32(key), n_pick, chosen);
                const int at = n_init + __popcll(chosen);
                int32_t *o = row0 + u * dm.topk;
                if ((chosen >> lane) & 1ull) o[n_init + __popcll(chosen & ((1ull << lane) - 1ull))] = lane;
                if (lane < n_init) o[lane] = lane;
                if (lane >= at && lane < dm.topk) o[lane] = lane < n_sel ? lo_local + (lane - at) : -1;
            }
        };
        // every kernel that meets a block up to the tokens' own, visible or not: what the pooling looks at
        const int steps = ((4 * b_own + 4 + 15) / 16 + C::kStep - 1) / C::kStep;
        if (steps <= 1) run(std::integral_constant<int, C::kStep>{});
        else if (steps == 2 || kKT <= 2 * C::kStep) run(std::integral_constant<int, 2 * C::kStep>{});
        else if (steps == 3) run(std::integral_constant<int, kKT <= 2 * C::kStep ? C::kStep : 3 * C::kStep>{});
        else run(std::integral_constant<int, kKT <= 2 * C::kStep ? C::kStep : 4 * C::kStep>{});
    }
}

template <int kG, int kKT, bool kScores>
static int launch_variant(const Dims &dm, Tensor q, Tensor ck, const int32_t *seqlens, int32_t *block_idx, hipStream_t stream,
                          float *scores, int32_t scores_pitch) {
    using C = ShortCfg<kG, kKT>;
    const int32_t n_units = (dm.max_seqlen + C::kTok - 1) / C::kTok;
    const size_t lds = C::lds_bytes(num_kernels(dm.max_seqlen));              // at most 73 KiB: two fit a compute unit
    // as many workgroups as the chip holds at a time (each copies the keys once), no more than there are tiles to go round
    constexpr int resident = 2;
    const int64_t rows = (int64_t)dm.batch * dm.Hkv;
    int share = 0;
    while ((1 << share) < C::kTok && ((int64_t)n_units * rows << share) * 2 <= 2048 * resident) ++share;
    const int32_t wgs = std::max<int32_t>(1, std::min<int32_t>(((n_units << share) + kShortWaves - 1) / kShortWaves,
                                                              (int32_t)(256 * resident / rows)));
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)select_short_kernel<kG, kKT, kScores>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL((select_short_kernel<kG, kKT, kScores>), dim3((uint32_t)((int64_t)wgs * dm.Hkv * dm.batch)), dim3(64 * kShortWaves),
                       lds, stream, dm, q, ck, seqlens, block_idx, n_units, wgs, share, scores, scores_pitch);
    return 0;
}

template <int kG>
static int launch_group(const Dims &dm, Tensor q, Tensor ck, const int32_t *seqlens, int32_t *block_idx, hipStream_t stream,
                        float *scores, int32_t pitch) {
    const int n_blocks = (dm.max_seqlen + kBlock - 1) / kBlock;
    if (scores)
        return n_blocks <= 32 ? launch_variant<kG, 8, true>(dm, q, ck, seqlens, block_idx, stream, scores, pitch)
                              : launch_variant<kG, 16, true>(dm, q, ck, seqlens, block_idx, stream, scores, pitch);
    return n_blocks <= 32 ? launch_variant<kG, 8, false>(dm, q, ck, seqlens, block_idx, stream, nullptr, 0)
                          : launch_variant<kG, 16, false>(dm, q, ck, seqlens, block_idx, stream, nullptr, 0);
}

bool select_short_fits(const Dims &dm) { return dm.rho == 1 && !dm.shared_q && dm.max_seqlen <= kShortPrefill; }

int launch_select_short(const Dims &dm, Tensor q, Tensor ck, const int32_t *seqlens, int32_t *block_idx, hipStream_t stream,
                        float *scores, int32_t scores_pitch) {
    if (dm.max_seqlen <= 0 || dm.batch <= 0) return 0;
    int err = (int)hipErrorInvalidValue;
    timing_begin("select_short_kernel", stream);
    switch (dm.G) {
        case 1: err = launch_group<1>(dm, q, ck, seqlens, block_idx, stream, scores, scores_pitch); break;
        case 2: err = launch_group<2>(dm, q, ck, seqlens, block_idx, stream, scores, scores_pitch); break;
        case 4: err = launch_group<4>(dm, q, ck, seqlens, block_idx, stream, scores, scores_pitch); break;
        case 8: err = launch_group<8>(dm, q, ck, seqlens, block_idx, stream, scores, scores_pitch); break;
        case 16: err = launch_group<16>(dm, q, ck, seqlens, block_idx, stream, scores, scores_pitch); break;
    }
    timing_end(stream);
    return err ? err : (int)hipGetLastError();
}

}  // namespace infllmv2
