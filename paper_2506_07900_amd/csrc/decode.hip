// Decode step, stages 2 and 3 for ONE query token per sequence at position seqlens[b]-1
// (section 2.1.3 "Different Granularity for Query and Key-Value Tokens": token-level queries
// keep the method usable in decoding; section 5.4: per step the attended blocks stay constant
// and only the semantic-kernel representations grow), and for the n drafted tokens of a
// speculative-verification step (section 4.1, "InfLLM v2 for Target Model"): the same kernels
// over n query rows per sequence, with the causal test of the last n x n region replaced by a
// bit-packed tree mask.
//
// A step of a few sequences moves a few megabytes, so it is bound by launch and memory latency, not by
// bandwidth: every kernel below spreads its reads over many workgroups and issues all the loads
// of a thread before using any of them.
//
// Selection (the softmax needs the log-sum-exp over ALL visible kernels before any score exists):
//   decode_logits_kernel   128 or 256 kernels per workgroup: MFMA logits, one partial (max, sum) per head
//                          and workgroup
//   decode_scores_*kernel  merges the partials into the log-sum-exp, group-mean scores, 5/4 max-pool
//                          -> block scores; the logits come from scratch (plain decode) or are
//                          computed again on the matrix cores (verification)
//   decode_pick_kernel     two-level top-k of the block scores (sorted lists of 128 blocks, or a row)
// Caches of up to 8192 tokens (verification: 4096): decode_short_kernel does all of this, and the attention, in one workgroup per block.
// Attention: one workgroup per selected block (split-KV) writes an unnormalised partial
// (o, max, sum); decode_merge_kernel combines the k partials per query head.  The one-call steps
// run the top-k inside the attention kernel (decode_pick_partial_kernel): one launch fewer.
#include "common.h"

namespace infllmv2 {

__device__ inline int clamp_len(int32_t L, int32_t cap) { return L < 0 ? 0 : (L > cap ? cap : L); }

// Every kernel below works on "query rows": row bv = b * n_q + qi is query token qi of sequence b.
// Plain decode has n_q = 1.  Draft verification (section 4.1, "InfLLM v2 for Target Model") has the
// n_q drafted tokens in the last n_q cache rows; token qi sits at position seqlens[b] - n_q + qi and
// selects blocks like any query at that position.  Returns the number of cache rows up to and
// including the query (0: the row is skipped; a sequence shorter than n_q is skipped as a whole).
__device__ inline int query_row(const Dims &dm, const int32_t *__restrict__ seqlens, int bv, int &b, int &qi) {
    if (dm.n_q == 1) {
        b = bv;
        qi = 0;
        return clamp_len(uniform_load(seqlens + b), dm.max_seqlen);
    }
    b = (int)__umulhi((uint32_t)bv, dm.n_q_inv);
    qi = bv - b * dm.n_q;
    const int L_all = clamp_len(uniform_load(seqlens + b), dm.max_seqlen);
    return L_all < dm.n_q ? 0 : L_all - (dm.n_q - 1 - qi);
}

// Query operands of parts 1 and 2.  MFMA operand layout: lane (n, g) holds head n, channels
// 32*ks + 8*g .. +7.  One query per workgroup: straight from memory.  Several (verification): every
// wave needs the same rows and every workgroup of the launch the same few cache lines, so the
// workgroup fetches them once into LDS (row pitch 272 bytes: conflict-free 16-byte reads).
constexpr int kQsPitch = kHeadDim + 8;
template <int kQT, int kThreads = 256>
struct QueryOperands {
    static constexpr int kEach = kQT == 1 ? 1 : kQT * 256 / kThreads;    // 256 threads take a query row's 16 heads x 16 chunks of 16 bytes
    static_assert(kQT == 1 || kEach * kThreads == kQT * 256, "every thread as many");
    bf16x8 x[kQT == 1 ? 4 : kEach];
    __device__ QueryOperands(const Dims &dm, const Tensor &q, int b, int h, int qi0) {      // asked for
        const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
        const int G = dm.G;
        if constexpr (kQT == 1) {
            const __bf16 *qr = q.ptr + (b * q.sb + qi0 * q.st + (int64_t)(h * G) * q.sh) + (min(n, G - 1) * q.sh + 8 * g);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) x[ks] = load8(qr + 32 * ks);
        } else {
            const int row = (threadIdx.x >> 4) & 15, c16 = threadIdx.x & 15, t0 = (int)(threadIdx.x >> 8) * kEach;
            const __bf16 *qr = q.ptr + (b * q.sb + (int64_t)(h * G) * q.sh) + (min(row, G - 1) * q.sh + 8 * c16);
#pragma unroll
            for (int t = 0; t < kEach; ++t) x[t] = load8(qr + min(qi0 + t0 + t, dm.n_q - 1) * q.st);
        }
    }
    __device__ void get(uint16_t *qs, bf16x8 (&bq)[kQT][4]) const {       // a barrier inside when kQT > 1
        const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
        if constexpr (kQT == 1) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) bq[0][ks] = x[ks];
        } else {
            const int row = (threadIdx.x >> 4) & 15, c16 = threadIdx.x & 15, t0 = (int)(threadIdx.x >> 8) * kEach;
#pragma unroll
            for (int t = 0; t < kEach; ++t) *reinterpret_cast<uint4 *>(&qs[((t0 + t) * 16 + row) * kQsPitch + 8 * c16]) = __builtin_bit_cast(uint4, x[t]);
            __syncthreads();
#pragma unroll
            for (int t = 0; t < kQT; ++t)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    bq[t][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&qs[(t * 16 + n) * kQsPitch + 32 * ks + 8 * g]));
        }
    }
};

// Candidates and counts of a query at cache row L - 1 (L >= 1).
struct RowRange {
    int n_sel, n_init, lo_local, jc_max, n_pick;
    __device__ RowRange(const Dims &dm, int L) {
        const int b_own = (L - 1) / kBlock, n_blk = b_own + 1;
        n_sel = dm.topk < n_blk ? dm.topk : n_blk;
        n_init = dm.n_init < n_blk ? dm.n_init : n_blk;                       // forced leading blocks
        lo_local = max(n_init, b_own - dm.n_local + 1);                       // forced trailing: lo_local..b_own
        jc_max = lo_local - 1;                                                // candidates: n_init..jc_max
        n_pick = n_sel - (n_init + (b_own - lo_local + 1));                   // at most topk - n_init - n_local
    }
};

// ---- selection, parts 1 and 2 -------------------------------------------------------------------
// Both parts score semantic kernels against kQT consecutive query tokens of one sequence on the
// matrix cores.  kQT = 1 is plain decode; verification uses kQT = kVerifyQT.  A workgroup of part 1
// covers kTW tiles of 16 kernels per wave, one of part 2 verify_tiles2 (plus one halo tile).  More
// tiles per wave mean fewer workgroups and fewer log-sum-exp partials for part 2 to merge (every
// workgroup of part 2 reads all partials of its heads); fewer tiles spread a lone step over more compute
// units.  Measured at 128K context, plain decode in a graph, 2 / 4 tiles: 14.2 / 15.0 us per step for
// one sequence, 14.5 / 15.4 for two, 16.6 / 16.1 for three, 20.7 / 19.9 for the ragged batch of 8, 49.9 / 50.9 for 32;
// one sequence of 32K 13.5 / 14.5.
constexpr int kVerifyQT = 4;
constexpr int kVerifyTiles = 2;                                                          // part 1, verification
// Part 1, plain decode: two for up to three sequences; for more, four where workgroups of two tiles are neither few enough for a compute unit each
// nor enough to fill the chip several times over (two / four tiles, us per step: 4 sequences of 60K, 240 workgroups, 15.1 / 15.8; 8 of 60K, 480,
// 17.4 / 16.8; 8 of 16K to 128K, 1024 by the capacity, 20.0 / 19.3; 16 of 128K, 2048, 31.6 / 32.0; 32 of 128K, 4096, 56.6 / 58.0, G = 4
// 38.2 / 40.9).  The scratch holds two sets of partials of `decode_tiles_scratch` tiles each; the exact log-sum-exp needs one, which may be twice as long.
static inline int decode_tiles_scratch(const Dims &dm) { return dm.batch >= 4 ? 4 : 2; }
static inline int decode_tiles_per_wave(const Dims &dm) {
    const int64_t n = (int64_t)dm.batch * dm.Hkv * ((num_kernels(dm.max_seqlen) + 127) / 128);
    return dm.batch < 4 || (dm.rho == 1 && (n <= 256 || n >= 2048)) ? 2 : 4;
}

// Part 1, verification: how many columns the grid has for a row's chunks.  A multiple of eight runs all query tiles of a chunk on one XCD, so that its
// kernels come from memory once; the columns that are added are empty, and the XCDs without them have up to twice the others' work.  It pays for
// few tiles per chunk, and while these do not fill the chip.  us, chunks' number / a multiple: 8 tiles per chunk (16 drafted, 2 heads), 10 chunks 6.2 / 5.8, 50
// 7.3 / 6.8, 90 9.1 / 8.3, 106 9.8 / 10.0; 16 tiles, 18 chunks 7.2 / 6.7, 42 8.6 / 8.4, 50 9.6 / 9.8, 58 10.1 / 11.5; 24 tiles, 10 chunks 6.2 / 7.1, 30 8.6 / 10.0,
// 58 12.9 / 14.3; 96 tiles (3 sequences, 32 drafted, 4 heads), 10 chunks 10.3 / 13.5; 128 tiles, 26 chunks 19.9 / 27.0.
__host__ __device__ inline int verify_columns(const Dims &dm, int n_qt, int n_part) {
    const int wide = (n_part + 7) & ~7;
    const int64_t tiles = (int64_t)dm.Hkv * dm.batch * n_qt;
    return n_qt > 1 && tiles <= 16 && tiles * wide <= 768 ? wide : n_part;
}

// length of the cache up to and including query token qi of sequence b (0: no such row)
__device__ inline int row_len(const Dims &dm, int L_all, int qi) {
    return (L_all < dm.n_q || qi >= dm.n_q) ? 0 : L_all - (dm.n_q - 1 - qi);
}

// Channels c0 .. c0+7 of the semantic kernel that the token appended at position L-1 completes: rows
// L-32 .. L-2 from the cache, row L-1 from the step's new key; fp64 sum in token order, one rounding
// (the bits compress_keys_kernel produces once the row is in the cache).
__device__ inline bf16x8 fresh_kernel_row8(const AppendArgs &ap, int b, int h, int L, int c0) {
    const __bf16 *kc = ap.k.ptr + b * ap.k.sb + h * ap.k.sh + c0;
    double acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0;
#pragma unroll 1
    for (int t0 = 0; t0 < kKernel; t0 += 8) {            // eight rows in flight at a time
        bf16x8 rows[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            rows[i] = t0 + i < kKernel - 1 ? load8(kc + (int64_t)(L - kKernel + t0 + i) * ap.k.st)
                                           : load8(ap.k_new.ptr + b * ap.k_new.sb + h * ap.k_new.sh + c0);
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += (double)(float)rows[i][e];
    }
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        w[e] = (uint32_t)f64_to_bf16_rne(acc[2 * e] / (double)kKernel) |
               ((uint32_t)f64_to_bf16_rne(acc[2 * e + 1] / (double)kKernel) << 16);
    return __builtin_bit_cast(bf16x8, uint4{w[0], w[1], w[2], w[3]});
}

// ---- part 1: partial (max, sum) of the relevance softmax ---------------------------------------------
// grid (n_c_cap / (64*kTW), Hkv, B * ceil(n_q/kQT)); wave w owns kernels chunk + 16*kTW*w .. +16*kTW-1.
// Z^T = CK . Q^T: lane = query head, 4 accumulator entries = 4 consecutive kernels.
// With kAppend (the one-call steps) the kernel also opens the step: workgroups behind the chunks (of a row, or of all) copy the new tokens' key and value
// rows into the caches (nothing before the attention kernel reads them; done by the first chunk's, those held up the launch: 16 drafted
// tokens at 128K, 12800 of its 13000 cycles), and the wave that owns the semantic kernel the new token completes builds its
// representation itself -- 31 cached rows and the new one, fp64 sum in token order, one rounding, the same bits as
// compress_keys_kernel -- uses it, and stores it for the steps to come.  Verification: the same for the n_q new tokens and the up to
// four kernels they complete, which every workgroup whose chunk holds one builds for itself; the last query tile's stores them.
// A launch fewer: 16 drafted tokens at 128K 31.5 -> 27.7 us per step, 4 22.4 -> 20.6, 2 x 60K tokens 31.7 -> 27.6.
template <int kQT, bool kAppend, int kTW>
__global__ __launch_bounds__(256) void decode_logits_kernel(Dims dm, Tensor q, Tensor ck,
                                                             const int32_t *__restrict__ seqlens,
                                                             float *__restrict__ zbuf, int32_t n_c_cap,
                                                             float2 *__restrict__ part,
                                                             float2 *__restrict__ part_c, int32_t n_part,
                                                             AppendArgs ap, uint32_t n_qt_inv) {
    constexpr int kChunk = 64 * kTW;
    constexpr int kNewKernels = 5;                    // at most, that the new tokens complete (64 drafted tokens: 4)
    __shared__ float2 wpart[kQT][4][16];
    __shared__ float2 wpart_c[kQT][4][16];
    __shared__ __align__(16) uint16_t qs[kQT > 1 ? kQT * 16 * kQsPitch : 8];
    __shared__ __align__(16) uint32_t newrow[kAppend ? 64 : 1];
    __shared__ __align__(16) uint16_t newrows[kAppend && kQT > 1 ? kNewKernels * kQsPitch : 8];
    arguments_arrive(dm.Hkv, dm.G, dm.max_seqlen, dm.n_q, seqlens, ck.ptr, ck.sb, ck.sh, ck.st, zbuf, n_c_cap, part);
    arguments_arrive(q.ptr, q.sb, q.sh, q.st, dm.scale_log2, n_part, dm.rho);
    const int n_qt = kQT == 1 ? 1 : (dm.n_q + kQT - 1) / kQT;            // query tiles per sequence (kQT = 1 is only launched with n_q = 1)
    int h = blockIdx.y, bx = blockIdx.x, b = blockIdx.z, qi0 = 0;
    bool appends = kAppend && kQT == 1 && bx >= n_part;
    if (kAppend && (int)blockIdx.z >= dm.batch * n_qt) {  // behind all chunks: one appends up to eight tokens to a (sequence, key-value head)
        const int n_app = kQT == 1 ? 1 : (dm.n_q + 7) / 8;
        const int wide = verify_columns(dm, n_qt, n_part);               // (the grid's)
        const int at = (((int)blockIdx.z - dm.batch * n_qt) * dm.Hkv + h) * wide + bx, unit = at / n_app;
        if (unit >= dm.batch * dm.Hkv) return;
        b = unit / dm.Hkv;
        h = unit - b * dm.Hkv;
        bx = n_part + at - unit * n_app;
        appends = true;
    } else if (n_qt > 1) {
        if (bx >= n_part) return;
        b = (int)__umulhi(blockIdx.z, n_qt_inv);
        qi0 = ((int)blockIdx.z - b * n_qt) * kQT;
    }
    const int32_t L_raw = uniform_load(seqlens + b);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int G = dm.G;
    __builtin_amdgcn_sched_barrier(0);
    // (queries and kernels are cold, 3200 cycles away from an idle unit: both are asked for before anything else is worked out)
    const QueryOperands<kQT> query(dm, q, b, h, kQT == 1 ? 0 : qi0);      // heads >= G repeat head G-1: their columns are never used
    __builtin_amdgcn_sched_barrier(0);
    const int jw = blockIdx.x * kChunk + wave * 16 * kTW; // first kernel of this wave
    int64_t ck_wave_at = b * ck.sb + h * ck.sh + (int64_t)jw * ck.st, ck_lane = n * ck.st + 8 * g;   // (worked out while the length is on its way)
    asm volatile("" : "+s"(ck_wave_at), "+v"(ck_lane));
    const int L_all = clamp_len(L_raw, dm.max_seqlen);
    bool closes = false;                              // the new token completes semantic kernel n_vis - 1
    int new_from = 0x7fffffff;                        // several tokens: the kernels from here on are completed by them
    if constexpr (kAppend) {
        const bool live = L_raw >= dm.n_q && L_raw <= dm.max_seqlen;  // as the stand-alone append: others are skipped
        if (appends) {                                // copies the rows of eight new tokens into the caches
            const int qi = (bx - n_part) * 8 + (threadIdx.x >> 5), c8 = (threadIdx.x & 15) * 8;
            if (!live || qi >= dm.n_q) return;
            const int64_t at = L_raw - dm.n_q + qi;
            if (threadIdx.x & 16)
                *reinterpret_cast<uint4 *>(ap.v.ptr + b * ap.v.sb + h * ap.v.sh + at * ap.v.st + c8) =
                    *reinterpret_cast<const uint4 *>(ap.v_new.ptr + b * ap.v_new.sb + h * ap.v_new.sh + qi * ap.v_new.st + c8);
            else
                *reinterpret_cast<uint4 *>(ap.k.ptr + b * ap.k.sb + h * ap.k.sh + at * ap.k.st + c8) =
                    *reinterpret_cast<const uint4 *>(ap.k_new.ptr + b * ap.k_new.sb + h * ap.k_new.sh + qi * ap.k_new.st + c8);
            return;
        }
        if (kQT > 1 && live) new_from = num_kernels(L_raw - dm.n_q);
        if (kQT == 1) closes = live && L_raw >= kKernel && (L_raw - kKernel) % kStride == 0;
    }
    if (!kAppend && (int)blockIdx.x >= n_part) return;
    int n_vis[kQT], n_vis_max = 0;                    // query slot t sits at L-1: n_c((L-1)+1); 0 = no such row
#pragma unroll
    for (int t = 0; t < kQT; ++t) {
        n_vis[t] = num_kernels(row_len(dm, L_all, qi0 + t));
        n_vis_max = max(n_vis_max, n_vis[t]);
    }
    if ((int)blockIdx.x * kChunk >= n_vis_max) return;    // uniform over the workgroup
    bf16x8 a[kTW][4];
    // Rows past the last kernel repeat it, and those that this launch completes may or may not be there yet: their scores are masked or their
    // operands replaced below.
    const __bf16 *ck_wave = ck.ptr + ck_wave_at;
    if (jw + 16 * kTW <= n_vis_max) {                 // uniform over the wave
#pragma unroll
        for (int i = 0; i < kTW; ++i)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a[i][ks] = load8(ck_wave + 16 * i * ck.st + ck_lane + 32 * ks);
    } else {
#pragma unroll
        for (int i = 0; i < kTW; ++i) {
            const int64_t at = min(16 * i + n, n_vis_max - 1 - jw) * ck.st + 8 * g;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a[i][ks] = load8(ck_wave + at + 32 * ks);
        }
    }
    const int build_from = max(new_from, (int)blockIdx.x * kChunk), build_to = min(n_vis_max, (int)(blockIdx.x + 1) * kChunk);
    const bool builds = kAppend && kQT > 1 && build_from < build_to;   // uniform over the workgroup
    if constexpr (kAppend && kQT > 1)
        if (builds) {
            // A wave per kernel, lane = channels 2*lane, 2*lane + 1; new rows from the call's inputs, older ones from the cache.  Rows' addresses are
            // scalar.  (A workgroup that builds ends last: with 32 lanes of four channels and addresses per lane it took 14000 cycles, so 9000.)
            for (int jh = build_from + wave; jh < build_to; jh += 4) {
                const int t_new = L_all - dm.n_q - jh * kStride;          // rows t_new .. of the kernel are new ones
                const int64_t old_at = b * ap.k.sb + h * ap.k.sh + (int64_t)jh * kStride * ap.k.st;
                const int64_t new_at = b * ap.k_new.sb + h * ap.k_new.sh - (int64_t)t_new * ap.k_new.st;
                uint32_t row[kKernel];
#pragma unroll
                for (int t = 0; t < kKernel; ++t) {
                    const __bf16 *p = t < t_new ? ap.k.ptr + (old_at + t * ap.k.st) : ap.k_new.ptr + (new_at + t * ap.k_new.st);
                    row[t] = reinterpret_cast<const uint32_t *>(p)[lane];
                }
                const uint32_t x = kernel_mean(row);
                *reinterpret_cast<uint32_t *>(&newrows[(jh - build_from) * kQsPitch + 2 * lane]) = x;
                if (qi0 + kQT >= dm.n_q)                  // the last query tile sees every kernel: it stores them
                    reinterpret_cast<uint32_t *>(ck.ptr + b * ck.sb + h * ck.sh + (int64_t)jh * ck.st)[lane] = x;
            }
        }
    bf16x8 bq[kQT][4];
    query.get(qs, bq);
    if constexpr (kAppend && kQT > 1)
        if (builds) {                                 // (a barrier lies between: the query rows went through LDS too)
#pragma unroll
            for (int i = 0; i < kTW; ++i) {
                const int x = jw + 16 * i + n;
                if (x >= build_from && x < build_to) {
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        a[i][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&newrows[(x - build_from) * kQsPitch + 32 * ks + 8 * g]));
                }
            }
        }
    if constexpr (kAppend && kQT == 1) {
        const int jh_new = n_vis_max - 1;             // = (L - p) / s when the new token closes a kernel
        if (closes && jh_new >= jw && jh_new < jw + 16 * kTW) {       // uniform over the wave
            // lane = channels 2*lane, 2*lane+1: rows L-32 .. L-2 from the cache, row L-1 from k_new
            const __bf16 *kc = ap.k.ptr + (b * ap.k.sb + h * ap.k.sh + (int64_t)(L_all - kKernel) * ap.k.st);
            uint32_t rowv[kKernel];
#pragma unroll
            for (int t = 0; t < kKernel - 1; ++t) rowv[t] = reinterpret_cast<const uint32_t *>(kc + t * ap.k.st)[lane];
            rowv[kKernel - 1] = reinterpret_cast<const uint32_t *>(ap.k_new.ptr + (b * ap.k_new.sb + h * ap.k_new.sh))[lane];
            const uint32_t packed = kernel_mean(rowv);
            newrow[lane] = packed;
            *reinterpret_cast<uint32_t *>(ck.ptr + b * ck.sb + h * ck.sh + (int64_t)jh_new * ck.st + 2 * lane) = packed;
            // same wavefront wrote newrow: LDS keeps the order.  The lanes whose operand row it is take it from there.
#pragma unroll
            for (int i = 0; i < kTW; ++i)
                if (jw + 16 * i + n == jh_new) {
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        a[i][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&newrow[16 * ks + 4 * g]));
                }
        }
    }
#pragma unroll
    for (int t = 0; t < kQT; ++t) {
        float x[kTW][4], mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < kTW; ++i) {
            f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) z = mfma16(a[i][ks], bq[t][ks], z);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[i][j] = z[j] * dm.scale_log2;
                if (jw + 16 * i + 4 * g + j >= n_vis[t]) x[i][j] = -INFINITY;
                mx = fmaxf(mx, x[i][j]);
            }
        }
        mx = xgroup_max(mx);
        const float m_use = mx == -INFINITY ? 0.f : mx;
        float sm = 0.f;
#pragma unroll
        for (int i = 0; i < kTW; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) sm += fast_exp2(x[i][j] - m_use);
        sm = xgroup_sum(sm);
        if (g == 0) wpart[t][wave][n] = float2{mx, sm};
        if constexpr (kQT == 1) {                     // plain decode keeps the logits for part 2
#pragma unroll
            for (int i = 0; i < kTW; ++i)
                if (n < G && jw + 16 * i < n_vis[0])
                    *reinterpret_cast<float4 *>(zbuf + (((int64_t)b * dm.Hkv + h) * G + n) * n_c_cap + jw + 16 * i + 4 * g) =
                        float4{x[i][0], x[i][1], x[i][2], x[i][3]};
        }
    }
    __syncthreads();
    if (threadIdx.x < 16 * kQT) {                     // merge the four waves: one partial per head and query
        const int t = threadIdx.x >> 4, head = threadIdx.x & 15;
        if (head < G && qi0 + t < dm.n_q) {
            float M = -INFINITY;
#pragma unroll
            for (int w = 0; w < 4; ++w) M = fmaxf(M, wpart[t][w][head].x);
            const float mu = M == -INFINITY ? 0.f : M;
            float S = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) S += wpart[t][w][head].y * fast_exp2(wpart[t][w][head].x - mu);
            const int64_t bv = (int64_t)b * dm.n_q + qi0 + t;
            part[((bv * dm.Hkv + h) * G + head) * n_part + blockIdx.x] = float2{M, S};
        }
    }
    // Approximate log-sum-exp ("Efficient Top-K Implementation", last paragraph): the same
    // partial (max, sum) over the coarse kernels kChunk/rho * bx .. of this chunk, each the bf16 mean
    // of its rho fine kernels rho*c + 2r (exact sum in fp64, one rounding).
    if (dm.rho > 1) {                                 // uniform over the launch
        const int tiles_c = 4 * kTW / dm.rho;         // 16-kernel tiles of coarse kernels per workgroup
        const int n_vis_c_max = num_coarse(n_vis_max, dm.rho);
        float Mc[kQT], Sc[kQT];                       // running partial of this wave, reduced over the wave
#pragma unroll
        for (int t = 0; t < kQT; ++t) {
            Mc[t] = -INFINITY;
            Sc[t] = 0.f;
        }
        for (int tc = wave; tc < tiles_c; tc += 4) {
            const int c0 = blockIdx.x * (kChunk / dm.rho) + tc * 16, cc = c0 + n;
            bf16x8 ac[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                ac[ks] = zero8();
                if (cc < n_vis_c_max) {
                    double acc[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] = 0.0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (r >= dm.rho) break;
                        const int jf = dm.rho * cc + 2 * r;
                        bf16x8 v;
                        if (kAppend && kQT == 1 && closes && jf == n_vis_max - 1)
                            // the kernel this step completes: another workgroup may be storing it right now,
                            // so its row is built here from the cache and the new key, never read back
                            v = fresh_kernel_row8(ap, b, h, L_all, 32 * ks + 8 * g);
                        else
                            v = load8(ck.ptr + b * ck.sb + h * ck.sh + (int64_t)jf * ck.st + 32 * ks + 8 * g);
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[e] += (double)(float)v[e];
                    }
                    uint32_t w[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w[e] = (uint32_t)f64_to_bf16_rne(acc[2 * e] / (double)dm.rho) |
                               ((uint32_t)f64_to_bf16_rne(acc[2 * e + 1] / (double)dm.rho) << 16);
                    ac[ks] = __builtin_bit_cast(bf16x8, uint4{w[0], w[1], w[2], w[3]});
                }
            }
#pragma unroll
            for (int t = 0; t < kQT; ++t) {
                const int n_vis_c = num_coarse(n_vis[t], dm.rho);
                f32x4 zc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) zc = mfma16(ac[ks], bq[t][ks], zc);
                float mc = -INFINITY, xc[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    xc[j] = c0 + 4 * g + j < n_vis_c ? zc[j] * dm.scale_log2 : -INFINITY;
                    mc = fmaxf(mc, xc[j]);
                }
                mc = xgroup_max(mc);
                const float Mn = fmaxf(Mc[t], mc), mu = Mn == -INFINITY ? 0.f : Mn;
                float sc = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) sc += fast_exp2(xc[j] - mu);
                sc = xgroup_sum(sc);
                Sc[t] = Sc[t] * fast_exp2(Mc[t] - mu) + sc;
                Mc[t] = Mn;
            }
        }
#pragma unroll
        for (int t = 0; t < kQT; ++t)
            if (g == 0) wpart_c[t][wave][n] = float2{Mc[t], Sc[t]};
        __syncthreads();
        if (threadIdx.x < 16 * kQT) {
            const int t = threadIdx.x >> 4, head = threadIdx.x & 15;
            if (head < G && qi0 + t < dm.n_q) {
                float M = -INFINITY;
#pragma unroll
                for (int w = 0; w < 4; ++w) M = fmaxf(M, wpart_c[t][w][head].x);
                const float mu = M == -INFINITY ? 0.f : M;
                float S = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) S += wpart_c[t][w][head].y * fast_exp2(wpart_c[t][w][head].x - mu);
                const int64_t bv = (int64_t)b * dm.n_q + qi0 + t;
                part_c[((bv * dm.Hkv + h) * G + head) * n_part + blockIdx.x] = float2{M, S};
            }
        }
    }
}

// ---- part 2, several queries per sequence: block scores ----------------------------------------------
// grid (n_lists, Hkv, B * ceil(n_q/kQT)), 512 threads (every block has a workgroup, also a
// last one too short to hold a complete kernel).  Workgroup bx pools blocks
// 16*kTW*bx .. +16*kTW-1 of kQT consecutive query tokens; block j needs kernels 4j-1 .. 4j+3, so the
// workgroup scores 4*kTW+1 tiles of 16 kernels starting one tile before its chunk (of that halo tile
// only the last kernel is used).  The logits are computed again rather than kept from part 1: a
// kernel's output has to reach memory before the next kernel starts, and megabytes of logits per
// query cost more than the matrix-core work to redo them.
// Z = Q . CK^T: lane = kernel (column), 4 accumulator entries = 4 consecutive heads.  A lane adds its 4
// heads; the four 16-lane groups leave their sums side by side in LDS and the pooling adds them, so
// no cross-lane traffic sits between the matrix cores and the scores.
// Eight wavefronts: a workgroup has a compute unit to itself, and one wavefront per SIMD issues an instruction every other slot.
template <int kQT, int kTW>
__global__ __launch_bounds__(512) void decode_scores_kernel(Dims dm, Tensor q, Tensor ck,
                                                             const int32_t *__restrict__ seqlens,
                                                             const float2 *__restrict__ part, int32_t n_part,
                                                             void *__restrict__ found, int32_t list_len, int32_t pitch, uint32_t n_qt_inv) {
    constexpr int kWaves = 8, kTiles = 4 * kTW + 1, kPerWave = 4 * kTW / kWaves;
    constexpr int kChunk = 64 * kTW;
    constexpr int kBlocks = 16 * kTW;                 // of a list
    static_assert(kBlocks <= 64 && kBlocks % 16 == 0 && kQT * kBlocks <= 256 && kPerWave >= 1, "a lane per block, a query within a wavefront");
    constexpr int kChunk1 = 64 * kVerifyTiles;  // kernels per partial of part 1
    constexpr int kLanesPerPair = 64 * kWaves / (16 * kQT);   // lanes that merge the partials of one (query, head)
    static_assert(kLanesPerPair == 8, "half a row of lanes");
    constexpr int kRound = 4 * 2 * kLanesPerPair;     // partials of a head that are merged at a time: 128K tokens' (of at most 262144 tokens')
    __shared__ __align__(16) float lse_h[kQT][16];
    __shared__ __align__(16) float4 rs[kQT][kTiles * 16];   // head sums of kernels chunk-16 .. chunk+kChunk-1, by 16-lane group
    __shared__ __align__(16) uint16_t qs[kQT * 16 * kQsPitch];
    __shared__ __align__(16) uint64_t words[kQT][16 * kTW];
    arguments_arrive(dm.Hkv, dm.G, dm.max_seqlen, dm.n_q, seqlens, ck.ptr, ck.sb, ck.sh, ck.st, part, n_part, n_qt_inv);
    arguments_arrive(q.ptr, q.sb, q.sh, q.st, dm.scale_log2, dm.rho, found, list_len, pitch, dm.topk, dm.n_init, dm.n_local);
    const int h = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int G = dm.G;
    const int n_qt = (dm.n_q + kQT - 1) / kQT;
    const int b = n_qt == 1 ? blockIdx.z : (int)__umulhi(blockIdx.z, n_qt_inv);
    const int qi0 = (blockIdx.z - b * n_qt) * kQT;
    const int32_t L_raw = uniform_load(seqlens + b);
    const int first = (int)blockIdx.x * kChunk - 16;  // kernel of rs[.][.][0]
    const int tile0 = 1 + wave * kPerWave;            // this wave's kernel tiles (tile 0 is the halo, taken by the last wave)
    int64_t ck_head = b * ck.sb + h * ck.sh, ck_wave_at = ck_head + (int64_t)(first + 16 * tile0) * ck.st, ck_lane = n * ck.st + 8 * g;
    asm volatile("" : "+s"(ck_wave_at), "+s"(ck_head), "+v"(ck_lane));
    const int L_all = clamp_len(L_raw, dm.max_seqlen);
    int L_max = 0;
#pragma unroll
    for (int t = 0; t < kQT; ++t) L_max = max(L_max, row_len(dm, L_all, qi0 + t));
    if (L_max < 1 || (int)blockIdx.x * kBlocks > (L_max - 1) / kBlock) return;    // no block of this chunk exists
    const int n_vis_max = num_kernels(L_max);
    // ---- operand loads: rows past the last kernel repeat it, and are left out of the pooling ----
    bf16x8 aq[kQT][4], bk[kPerWave + 1][4];
    if (n_vis_max > 0) {                              // uniform over the workgroup
        const int from = first + 16 * tile0;
        const __bf16 *ck_wave = ck.ptr + ck_wave_at;
        const bool all = from + 16 * kPerWave <= n_vis_max;                       // uniform over the wave
#pragma unroll
        for (int i = 0; i < kPerWave; ++i) {
            const int64_t at = all ? 16 * i * ck.st + ck_lane : min(16 * i + n, n_vis_max - 1 - from) * ck.st + 8 * g;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) bk[i][ks] = load8(ck_wave + at + 32 * ks);
        }
        if (wave == kWaves - 1) {
            const __bf16 *ck_halo = ck.ptr + ck_head + (int64_t)max(min(first + n, n_vis_max - 1), 0) * ck.st + 8 * g;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) bk[kPerWave][ks] = load8(ck_halo + 32 * ks);
        }
    } else {
#pragma unroll
        for (int i = 0; i <= kPerWave; ++i)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) bk[i][ks] = zero8();
    }
    __builtin_amdgcn_sched_barrier(0);
    const QueryOperands<kQT, 64 * kWaves> query(dm, q, b, h, qi0);
    // ---- log-sum-exp per (query, head): kLanesPerPair lanes each, two partials to a load ----
    {
        const int pair = tid / kLanesPerPair, sub = tid % kLanesPerPair;
        const int pt = pair >> 4, head = pair & 15;
        const int64_t bv = (int64_t)b * dm.n_q + min(qi0 + pt, dm.n_q - 1);
        const float2 *pr = part + ((bv * dm.Hkv + h) * G + min(head, G - 1)) * n_part;
        const int np = (num_kernels(row_len(dm, L_all, qi0 + pt)) + kChunk1 - 1) / kChunk1;  // valid partials
        float M = -INFINITY, S = 0.f;
        for (int p0 = 0; p0 < n_part; p0 += kRound) {
            float4 v[4];                              // (n_part is even, a row begins at a multiple of 16 bytes)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const float4 *>(pr + min(p0 + 2 * (sub + kLanesPerPair * i), n_part - 2));
            float m = M;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = p0 + 2 * (sub + kLanesPerPair * i);
                if (p >= np) v[i].x = -INFINITY, v[i].y = 0.f;
                if (p + 1 >= np) v[i].z = -INFINITY, v[i].w = 0.f;
                m = fmaxf(m, fmaxf(v[i].x, v[i].z));
            }
            const float mu = m == -INFINITY ? 0.f : m;
            S *= fast_exp2(M - mu);
#pragma unroll
            for (int i = 0; i < 4; ++i) S += v[i].y * fast_exp2(v[i].x - mu) + v[i].w * fast_exp2(v[i].z - mu);
            M = m;
        }
        float m = M;                                  // over the pair's eight lanes
        m = fmaxf(m, dpp_rotate<kSwap1>(m));
        m = fmaxf(m, dpp_rotate<kSwap2>(m));
        m = fmaxf(m, dpp_rotate<kMirror8>(m));
        const float mu = m == -INFINITY ? 0.f : m;
        float sm = S * fast_exp2(M - mu);
        sm += dpp_rotate<kSwap1>(sm);
        sm += dpp_rotate<kSwap2>(sm);
        sm += dpp_rotate<kMirror8>(sm);
        // approximate mode: rho times fewer kernels were summed; 0 when none is visible
        const float exact = m + fast_log2(sm), coarse = m == -INFINITY ? 0.f : exact + (float)(31 - __clz(dm.rho));
        if (sub == 0) lse_h[pt][head] = head >= G ? INFINITY : dm.rho > 1 ? coarse : exact;   // (heads that are not there score 0)
    }
    query.get(qs, aq);                                // (a barrier inside)
    // ---- head sums of exp(z - lse) ------------------------------------------------------------------------
#pragma unroll
    for (int t = 0; t < kQT; ++t) {
        const float4 l4 = *reinterpret_cast<const float4 *>(&lse_h[t][4 * g]);
        const float lh[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
        for (int i = 0; i <= kPerWave; ++i) {
            if (i == kPerWave && wave != kWaves - 1) break;   // uniform over the wave
            const int tile = i < kPerWave ? tile0 + i : 0;
            f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) z = mfma16(aq[t][ks], bk[i][ks], z);
            float acc = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc += fast_exp2(z[r] * dm.scale_log2 - lh[r]);
            reinterpret_cast<float *>(&rs[t][16 * tile + n])[g] = acc;
        }
    }
    __syncthreads();
    // ---- group mean, clamps, 5/4 max-pool: thread (t, jl) takes kernels 4j-1 .. 4j+3 = rs[..][4*jl+15 .. +19]; the list_len
    // best of a query's kBlocks go to a descending list, or (list_len = 0) the scores of all of them to the query's row ----
    const int t = tid / kBlocks, jl = tid % kBlocks, L = t < kQT ? row_len(dm, L_all, qi0 + t) : 0;
    if (L >= 1) {
        const int j = blockIdx.x * kBlocks + jl, n_vis = num_kernels(L);
        float v = -INFINITY;
#pragma unroll
        for (int x = 0; x < 5; ++x) {
            const int c = 4 * jl + 15 + x, jh = first + c;
            const float4 y = rs[t][c];
            const float sum = (y.x + y.y) + (y.z + y.w);
            v = fmaxf(v, jh >= 0 && jh < n_vis ? sum : -INFINITY);
        }
        v = max(first + 4 * jl + 15, 0) < n_vis ? fminf(fmaxf(v * (1.f / G), kScoreFloor), kScoreCeil) : -INFINITY;
        const int64_t row = ((int64_t)b * dm.n_q + qi0 + t) * dm.Hkv + h;
        if (list_len == 0) {
            if (j <= (L - 1) / kBlock) reinterpret_cast<float *>(found)[row * pitch + j] = v;
            return;                                   // (uniform over the wavefront, and nothing waits below)
        }
        const RowRange rr(dm, L);
        const uint64_t e = pick_element(v, j, rr.n_init, rr.jc_max);
        uint64_t *list = reinterpret_cast<uint64_t *>(found) + (row * gridDim.x + blockIdx.x) * list_len;
        if (list_len <= 16) {                         // by sorting networks, as in plain decode: a query's two or four rows of lanes
            uint64_t x = row_sort64(e, lane);
            x = kBlocks == 64 ? rows_merge64(x, lane) : row_pairs_merge64(x, lane);
            if (jl < list_len) list[jl] = x;
            return;
        }
        words[t][jl] = e;
        __builtin_amdgcn_wave_barrier();              // same wavefront: LDS keeps the order
        const int rank = count_larger(words[t], kBlocks, e);   // no two words are equal
        if (rank < list_len) list[rank] = e;
    }
}

// ---- part 2, plain decode: block scores from the logits part 1 kept ---------------------------------
// (One query per sequence: its logits are a quarter of the bytes of the compressed keys, so reading
// them back is cheaper than computing them again; with several queries per sequence the balance tips.)
// grid (n_lists, Hkv, B), 512 threads.  Thread t scores kernel 512*bx + t, and 16 lanes, a head each, the one before the first;
// waves 0 and 1 then pool blocks 128*bx + t and leave the list_len best of the 128 as a descending list of pick words:
// the top-k that follows merges nb/128 short lists, at most one word per thread up to 150K tokens, instead of ranking a
// row of nb scores -- which each of its topk workgroups per row would do again.
// Eight wavefronts, so that four workgroups fit a compute unit (with a ninth for the halo kernel, three: 32 sequences
// of 128K, 1024 workgroups, took two rounds).  kSorted: lists of up to 16, by sorting networks across the lanes instead of by counting.
constexpr int kMaxParts = 128;                        // partials per head (of >= 128 kernels): contexts up to 262144 tokens
constexpr int kListBlocks = 128;                      // blocks per list
constexpr int kScoreThreads = 4 * kListBlocks;
template <int kG, bool kSorted>
__global__ __launch_bounds__(kScoreThreads) void decode_scores_z_kernel(Dims dm, const int32_t *__restrict__ seqlens,
                                                             const float *__restrict__ zbuf,
                                                             const float2 *__restrict__ part,
                                                             int32_t n_c_cap, int32_t n_part, int32_t part_kernels,
                                                             uint64_t *__restrict__ lists, int32_t list_len) {
    __shared__ __align__(16) float lse_h[16], halo_e[16];
    __shared__ float rs[kScoreThreads + 4];
    __shared__ __align__(16) uint64_t words[2][64], best[2][64];
    arguments_arrive(dm.Hkv, dm.n_init, dm.n_local, dm.topk, dm.max_seqlen, dm.rho, seqlens, zbuf, part, n_c_cap, n_part, part_kernels);
    arguments_arrive(lists, list_len);
    const int h = blockIdx.y, bv = blockIdx.z;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int base = blockIdx.x * kScoreThreads;
    const int32_t L_raw = uniform_load(seqlens + bv);
    // Everything this thread reads lies in the workspace at places that do not depend on the sequence
    // length, so the loads go out before the length is known (one memory round trip less on the
    // critical path of the step); what turns out to be past the end is masked afterwards.
    const float *z_row = zbuf + ((int64_t)bv * dm.Hkv + h) * kG * n_c_cap;
    const float2 *p_row = part + ((int64_t)bv * dm.Hkv + h) * kG * n_part;
    const int head = tid >> 4, sub = tid & 15;        // 16 lanes per head merge its partials
    float2 v[kMaxParts / 16];
    if (tid < 16 * kG) {
#pragma unroll
        for (int i = 0; i < kMaxParts / 16; ++i) {
            v[i] = float2{-INFINITY, 0.f};
            if (16 * i < n_part) v[i] = p_row[head * n_part + min(sub + 16 * i, n_part - 1)];
        }
    }
    const uint32_t jh_c = min(base + tid, n_c_cap - 1);
    float zz[kG];
#pragma unroll
    for (int gq = 0; gq < kG; ++gq) zz[gq] = (z_row + (int64_t)gq * n_c_cap)[jh_c];
    const bool halo = wave == kScoreThreads / 64 - 1 && lane < kG;
    float z_halo = 0.f;
    if (halo) z_halo = z_row[lane * n_c_cap + max(base - 1, 0)];
    const int L = clamp_len(L_raw, dm.max_seqlen);
    const int n_vis = num_kernels(L);
    if (L < 1 || (int)blockIdx.x * kListBlocks > (L - 1) / kBlock) return;   // no block of this chunk exists
    const int np = (n_vis + part_kernels - 1) / part_kernels;   // valid partials
    // log-sum-exp per head
    if (tid < 16 * kG) {
#pragma unroll
        for (int i = 0; i < kMaxParts / 16; ++i)
            if (sub + 16 * i >= np) v[i] = float2{-INFINITY, 0.f};
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < kMaxParts / 16; ++i) m = fmaxf(m, v[i].x);
        m = row_reduce(m, [](float a, float c) { return fmaxf(a, c); });
        const float mu = m == -INFINITY ? 0.f : m;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < kMaxParts / 16; ++i)
            if (16 * i < np) s += v[i].y * fast_exp2(v[i].x - mu);
        s = row_reduce(s, [](float a, float c) { return a + c; });
        // approximate mode: rho times fewer kernels were summed; 0 when none is visible
        const float exact = m + fast_log2(s), coarse = m == -INFINITY ? 0.f : exact + (float)(31 - __clz(dm.rho));
        if (sub == 0) lse_h[head] = dm.rho > 1 ? coarse : exact;
    }
    // logits of this thread's kernel, all heads
    __syncthreads();
    {
        float acc = 0.f;
#pragma unroll
        for (int gq = 0; gq < kG; ++gq) acc += fast_exp2(zz[gq] - lse_h[gq]);
        rs[1 + tid] = base + tid < n_vis ? fminf(fmaxf(acc * (1.f / kG), kScoreFloor), kScoreCeil) : -INFINITY;
        if (halo) {                                   // (the heads are added in the same order)
            halo_e[lane] = fast_exp2(z_halo - lse_h[lane]);
            __builtin_amdgcn_wave_barrier();          // same wavefront: LDS keeps the order
            acc = 0.f;
#pragma unroll
            for (int gq = 0; gq < kG; ++gq) acc += halo_e[gq];
            if (lane == 0) rs[0] = base >= 1 && base - 1 < n_vis ? fminf(fmaxf(acc * (1.f / kG), kScoreFloor), kScoreCeil) : -INFINITY;
        }
    }
    __syncthreads();
    uint64_t e = 0ull;
    uint64_t *list = lists + (((int64_t)bv * dm.Hkv + h) * gridDim.x + blockIdx.x) * list_len;
    if (wave < 2) {
        const int j = blockIdx.x * kListBlocks + tid;     // kernels 4j-1 .. 4j+3 = rs[4*tid .. 4*tid+4]
        float r = rs[4 * tid];
#pragma unroll
        for (int x = 1; x < 5; ++x) r = fmaxf(r, rs[4 * tid + x]);
        const RowRange rr(dm, L);
        e = pick_element(r, j, rr.n_init, rr.jc_max);
    }
    if constexpr (kSorted) {
        if (wave < 2) {
            e = rows_merge64(row_sort64(e, lane), lane);
            if (wave == 1 && lane < 16) best[1][lane] = e;
        }
        __syncthreads();
        if (wave == 0) {
            e = row_merge64(e, best[1][lane & 15], lane);
            if (lane < list_len) list[lane] = e;
        }
    } else {
        int rank = 64;
        if (wave < 2) {
            words[wave][lane] = e;
            best[wave][lane] = 0ull;
            __builtin_amdgcn_wave_barrier();              // same wavefront: LDS keeps the order
            rank = count_larger(words[wave], 64, e);      // no two words are equal
            if (rank < list_len) best[wave][rank] = e;
        }
        __syncthreads();
        if (wave < 2 && rank < list_len) {
            rank += count_larger(best[wave ^ 1], (list_len + 3) & ~3, e);
            if (rank < list_len) list[rank] = e;
        }
    }
}

// ---- selection, part 3: top-k of one row of block scores ----------------------------------------
// grid (B*n_q*Hkv), 256 threads.  Candidates are the blocks n_init .. b_own - n_local; the forced ones
// are added afterwards (section 2.1.2 "Top-K Blocks Sharing": initial and local blocks are always
// attended).  Scores are positive floats, so their bit patterns order like unsigned integers.
// An element is the 64-bit word  key << 32 | ~block  with key = bits of the score (1 for a block
// without visible kernel, -inf): larger word = better element, ties go to the lower block index,
// and no two elements are equal.  Words below 2^32 (key 0) are "not a candidate".
//
// No serial rounds (a dependent chain per pick is what makes a small top-k slow on this machine);
// filters by counting instead, every comparison independent of the others.  Thread t keeps blocks
// t, t+256, ... in registers and `best`, the largest of them.  An element of the final top-k can
// only sit in a thread whose best is among the n_pick largest thread maxima (every better thread
// holds an element that beats it), and it is at least tau, the n_pick-th largest thread maximum
// (the n_pick largest thread maxima are n_pick distinct elements).
//   1a. rank of `best` inside its wavefront; the n_pick best of each wavefront survive
//   1b. rank of the survivors among all survivors = rank among all thread maxima; gives tau
//   2.  the n_pick best threads publish their elements >= tau; rank by counting among those
//   3.  every wavefront repeats the ranking of the survivors of all of them and orders the selected blocks
//
// The elements are the sorted lists, one per 128 blocks (verification: 32 or 64), the scoring kernel left, or a row of scores.
constexpr int kPickThreads = 256, kPickWaves = kPickThreads / 64, kPickMaxVPT = 16;
// LDS of the top-k, carved out of the kernel's dynamic shared memory (16-byte aligned) so that its size
// follows the call's top-k instead of the largest one supported.
struct PickShared {
    uint64_t *tmax;                                       // [kPickThreads] thread maxima, 64 per wavefront
    uint64_t *top;                                        // [kPickWaves][n_pick rounded up to 4] per wavefront: its best (0 = none)
    uint64_t *cand;                                       // [kPickWaves][cand_cap] per wavefront: elements that can still make it
    int cand_cap;
    __device__ PickShared(unsigned char *smem, int topk, int vpt) {
        tmax = reinterpret_cast<uint64_t *>(smem);
        top = tmax + kPickThreads;
        cand = top + kPickWaves * ((topk + 3) & ~3);
        cand_cap = (topk * vpt + 3) & ~3;
    }
};
static inline size_t pick_shared_bytes(int topk, int vpt) {
    const size_t words = (size_t)kPickThreads + (size_t)kPickWaves * ((topk + 3) & ~3) +
                         (vpt > 1 ? (size_t)kPickWaves * (((size_t)topk * vpt + 3) & ~(size_t)3) : 0);
    return words * sizeof(uint64_t);
}

// This thread's kVPT elements of row `row` of the top-k's input: words of the lists (kLists) or scores of a row.  Every
// load goes out before the sequence length is known; what lies past the end is dropped afterwards.
struct PickInput {
    const void *found;                                    // lists: uint64 [rows][n_lists][list_len]; scores: float [rows][pitch]
    int32_t n_lists, list_len, inv;                       // inv: i / n_lists = (i * inv) >> 20 for i < 4096
    int32_t blocks;                                       // of a list
    int32_t pitch;
};
template <bool kLists, int kVPT>
struct PickLoad {
    uint64_t w[kLists ? kVPT : 1];
    float r[kLists ? 1 : kVPT];
    __device__ PickLoad(const PickInput &in, int64_t row) {
#pragma unroll
        for (int s = 0; s < kVPT; ++s) {
            const int i = threadIdx.x + kPickThreads * s;
            if constexpr (kLists) {                       // element i = entry i / n_lists of list i % n_lists
                const int rank = ((uint32_t)i * (uint32_t)in.inv) >> 20, list = i - rank * in.n_lists;
                w[s] = reinterpret_cast<const uint64_t *>(in.found)[(row * in.n_lists + list) * in.list_len + min(rank, in.list_len - 1)];
            } else {
                r[s] = reinterpret_cast<const float *>(in.found)[row * in.pitch + min(i, in.pitch - 1)];
            }
        }
    }
    __device__ void elements(const PickInput &in, const RowRange &rr, int L, uint64_t (&el)[kVPT]) const {
#pragma unroll
        for (int s = 0; s < kVPT; ++s) {
            const int i = threadIdx.x + kPickThreads * s;
            if constexpr (kLists) {
                const int rank = ((uint32_t)i * (uint32_t)in.inv) >> 20, list = i - rank * in.n_lists;
                el[s] = (rank < in.list_len && list * in.blocks <= (L - 1) / kBlock) ? w[s] : 0ull;   // (later lists were not written)
            } else {
                el[s] = pick_element(r[s], i, rr.n_init, rr.jc_max);
            }
        }
    }
};

// Top-k of one row for a query at cache row L - 1 (L >= 1), by a whole workgroup of kPickThreads threads; a thread
// brings kVPT elements.  Leaves the selected blocks in this wavefront's `mine` (LDS, [64]): the picked ones, best first,
// then the forced ones; every wavefront gets its own copy.  Contains barriers: every thread calls it.
//
// Two levels.  Every wavefront finds the n_pick best of its own share on its own, synchronising with
// nobody: rank its 64 thread maxima by counting; an element of its top n_pick can only sit in a
// thread whose maximum is among the n_pick largest, and is at least tau, the n_pick-th largest
// maximum; those threads publish their elements >= tau (a handful) and the wavefront ranks them by
// counting (with one element per thread the first ranking is the answer).  Then every finalist is counted against the
// four short lists, one list per wavefront, and the counts are added.
// Clock stamps at 128K context, one sequence: 0.4 us first ranking, 0.1 barrier, 0.3 second; a row of 2048 scores cost
// 4.4 us in all.
template <int kVPT>
__device__ inline void pick_row(const RowRange &rr, const uint64_t (&el)[kVPT], const PickShared &sh, int *mine) {
    __shared__ int counts[kPickWaves][kPickWaves * kMaxTopk];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n_pick = rr.n_pick;
    if (n_pick > 0) {                                                         // uniform over the workgroup
        const int pitch = (n_pick + 3) & ~3, n_fin = kPickWaves * pitch;
        uint64_t *wtop = sh.top + wave * pitch, *wmax = sh.tmax + 64 * wave;
        if (lane < pitch) wtop[lane] = 0ull;
        uint64_t best = 0ull;
#pragma unroll
        for (int s = 0; s < kVPT; ++s) best = el[s] > best ? el[s] : best;
        const bool real = best >= kPickValid;
        wmax[lane] = best;
        __builtin_amdgcn_wave_barrier();                  // same wavefront: LDS keeps the order
        const int lrank = count_larger(wmax, 64, best);
        if constexpr (kVPT == 1) {
            if (real && lrank < n_pick) wtop[lrank] = best;
        } else {
            uint64_t *wcand = sh.cand + wave * sh.cand_cap;
            const bool finalist = real && lrank < n_pick;
            uint64_t tau = kPickValid;                    // the n_pick-th largest maximum, if there are that many real ones
            const uint64_t who = __ballot(real && lrank == n_pick - 1);
            if (who) {
                const int src = __builtin_ctzll(who);
                tau = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(best >> 32), src) << 32) |
                      (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)best, src);
            }
            int n_cand = 0;                               // <= n_pick * kVPT <= cand_cap
            const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
            for (int s = 0; s < kVPT; ++s) {
                const bool pub = finalist && el[s] >= tau;
                const uint64_t m = __ballot(pub);
                if (pub) wcand[n_cand + __popcll(m & below)] = el[s];
                n_cand += __popcll(m);
            }
            const int n_cand4 = (n_cand + 3) & ~3;
            if (lane < n_cand4 - n_cand) wcand[n_cand + lane] = 0ull;
            __builtin_amdgcn_wave_barrier();
            for (int i = lane; i < n_cand; i += 64) {
                const uint64_t e = wcand[i];
                const int beaten = count_larger(wcand, n_cand4, e);
                if (beaten < n_pick) wtop[beaten] = e;
            }
        }
        __syncthreads();
        for (int i = lane; i < n_fin; i += 64) counts[wave][i] = count_larger(wtop, pitch, sh.top[i]);
        __syncthreads();
        for (int i = lane; i < n_fin; i += 64) {
            const uint64_t e = sh.top[i];
            const int beaten = (counts[0][i] + counts[1][i]) + (counts[2][i] + counts[3][i]);
            if (e >= kPickValid && beaten < n_pick) mine[beaten] = (int)~(uint32_t)e;
        }
    }
    if (lane >= max(n_pick, 0) && lane < rr.n_sel) {      // the forced blocks
        const int f = lane - max(n_pick, 0);
        mine[lane] = f < rr.n_init ? f : rr.lo_local + (f - rr.n_init);
    }
    __builtin_amdgcn_wave_barrier();
}

// Puts a wavefront's n_sel selected blocks (`mine`, LDS) in ascending order: returns the place of this lane's block
// (lane < n_sel) and, if `o` is given, writes the row of the block_idx output, padded with -1.
__device__ inline int order_row(int *mine, int n_sel, int topk, int32_t *__restrict__ o) {
    const int lane = threadIdx.x & 63;
    const int x = lane < n_sel ? mine[lane] : 0x7fffffff;
    mine[lane] = x;
    __builtin_amdgcn_wave_barrier();
    int rank = 0;                                         // number of selected blocks below x
    for (int e = 0; e < n_sel; e += 16) {
        int4 y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = *reinterpret_cast<const int4 *>(mine + e + 4 * i);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            rank += (y[i].x < x ? 1 : 0) + (y[i].y < x ? 1 : 0) + (y[i].z < x ? 1 : 0) + (y[i].w < x ? 1 : 0);
    }
    if (o) {
        if (lane < n_sel) o[rank] = x;
        else if (lane < topk) o[lane] = -1;
    }
    return rank;
}

// The same for at most 16 picks from at most 16 kSlots (kShare) or 4 kSlots sorted lists: a row of lanes holds a list, rows are merged
// two at a time without LDS; with kShare the four wavefronts merge a quarter of the lists each and then each other's results.
// Returns the c-th best word in lane c of every row.  Against counting (32 LDS reads of 16 bytes and 64 compares of 64 bits per
// wavefront, two barriers): 3200 -> 1600 cycles for 16 lists of 13 on a compute unit of its own.
constexpr int kMergePicks = 16;
template <int kSlots, bool kShare>
struct ListMerge {
    uint64_t w[kSlots];
    static __device__ int list(int s) { return ((kShare ? (int)(threadIdx.x >> 6) : 0) * kSlots + s) * 4 + ((int)(threadIdx.x & 63) >> 4); }
    __device__ ListMerge(const PickInput &in, int64_t row) {
        const int64_t first = row * in.n_lists * in.list_len + min((int)(threadIdx.x & 15), in.list_len - 1);
#pragma unroll
        for (int s = 0; s < kSlots; ++s) w[s] = reinterpret_cast<const uint64_t *>(in.found)[first + min(list(s), in.n_lists - 1) * in.list_len];
    }
    __device__ uint64_t best(const PickInput &in, int L) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int s = 0; s < kSlots; ++s)                  // (lists past the sequence's end were not written)
            if ((lane & 15) >= in.list_len || list(s) >= in.n_lists || list(s) * in.blocks > (L - 1) / kBlock) w[s] = 0ull;
        uint64_t x = w[0];
#pragma unroll
        for (int s = 1; s < kSlots; ++s) x = row_merge64(x, w[s], lane);
        x = rows_merge64(x, lane);
        if constexpr (kShare) {
            __shared__ uint64_t of_wave[kPickWaves][16];
            if (lane < 16) of_wave[threadIdx.x >> 6][lane] = x;
            __syncthreads();
            x = rows_merge64(of_wave[lane >> 4][lane & 15], lane);
        }
        return x;
    }
};

// How a row's top-k is found: from its scores (kScores), from sorted lists by counting (kCount) or by merging (kMerge, kMergeShared); kN: elements per
// thread, or lists per row of lanes.
enum PickForm { kScores, kCount, kMerge, kMergeShared };
template <int kForm, int kN>
struct Picker {
    std::conditional_t<kForm <= kCount, PickLoad<kForm == kCount, kN>, ListMerge<kN, kForm == kMergeShared>> load;
    __device__ Picker(const PickInput &in, int64_t row) : load(in, row) {}
    // the selected blocks of the row, the picked ones first, best first, to this wavefront's `mine`; entry `at` (uniform) is returned.  Every thread calls it.
    __device__ int pick(const PickInput &in, const RowRange &rr, int L, unsigned char *smem, int topk, int *mine, int at) {
        if constexpr (kForm <= kCount) {
            uint64_t el[kN];
            load.elements(in, rr, L, el);
            pick_row<kN>(rr, el, PickShared(smem, topk, kN), mine);
            return __builtin_amdgcn_readfirstlane(mine[min(at, rr.n_sel - 1)]);
        } else {
            const int lane = threadIdx.x & 63, n_pick = max(rr.n_pick, 0);
            int x = 0;
            if (n_pick > 0) x = (int)~(uint32_t)load.best(in, L);                 // uniform over the workgroup
            const int f = lane - n_pick;
            if (f >= 0) x = f < rr.n_init ? f : rr.lo_local + (f - rr.n_init);    // the forced blocks
            if (lane < rr.n_sel) mine[lane] = x;
            __builtin_amdgcn_wave_barrier();
            return __builtin_amdgcn_readlane(x, min(at, rr.n_sel - 1));
        }
    }
};

template <int kForm, int kN>
__global__ __launch_bounds__(kPickThreads) void decode_pick_kernel(Dims dm, const int32_t *__restrict__ seqlens,
                                                                    PickInput in, int32_t *__restrict__ block_idx) {
    extern __shared__ __align__(16) unsigned char pick_smem[];
    arguments_arrive(dm.Hkv, dm.topk, dm.n_init, dm.n_local, dm.max_seqlen, dm.n_q, seqlens, in.found, in.n_lists, in.list_len, in.blocks, block_idx);
    const int row = blockIdx.x, bv = row / dm.Hkv, h = row - bv * dm.Hkv;
    Picker<kForm, kN> picker(in, row);
    int b, qi;
    const int L = query_row(dm, seqlens, bv, b, qi);
    int32_t *o = block_idx + (((int64_t)b * dm.Hkv + h) * dm.n_q + qi) * dm.topk;
    if (L < 1) {
        if ((int)threadIdx.x < dm.topk) o[threadIdx.x] = -1;
        return;
    }
    const RowRange rr(dm, L);
    __shared__ __align__(16) int mine[kPickWaves][64];
    picker.pick(in, rr, L, pick_smem, dm.topk, mine[threadIdx.x >> 6], 0);
    if (threadIdx.x < 64) order_row(mine[0], rr.n_sel, dm.topk, o);
}

// ---- attention, part 1: one workgroup per selected block --------------------------------------
// grid (topk, Hkv, B), 256 threads.  Every load of the block (64 key rows as MFMA operands, 64
// value rows for LDS, the query) is issued before anything is used.  Wave w: S^T = K . Q^T for
// keys 16w..16w+15; the probabilities go to LDS in bf16 as the B operand of the value product; then
// wave w owns value channels 32w..32w+31 and computes O^T = V^T . P^T on the matrix cores, reading
// V^T through the transposing LDS load from the row-major value tile.
constexpr int kVsPitch = kHeadDim + 4;               // bf16 elements per LDS value row: 4 rows of a transposing load in 4 bank groups
typedef short s16x4_t __attribute__((ext_vector_type(4)));

// What the fetch of a block does not need the block for: where the thread's rows lie, value rows tid/16 + 16i (channels
// 8(tid%16) ..), key row 16 wave + n (channels 32ks + 8g ..).  Worked out before the block is known: a wavefront alone spends 2000
// cycles on these arguments and products otherwise, and left to itself the compiler moves them to where the block is known.
struct BlockFetch {
    int64_t k_head, v_head;                              // uniform: the head's first row
    int64_t v[4], k;
    __device__ void set(const Dims &dm, const Tensor &kt, const Tensor &vt, int b, int h) {
        k_head = b * kt.sb + h * kt.sh;
        v_head = b * vt.sb + h * vt.sh;
        rows(kt, vt, kBlock - 1);
        asm volatile("" : "+s"(k_head), "+s"(v_head));
        asm volatile("" : "+v"(k), "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
    }
    __device__ void rows(const Tensor &kt, const Tensor &vt, int last) {                 // the block's rows 0 .. last exist
        const int tid = threadIdx.x, lane = tid & 63;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (int64_t)min((tid >> 4) + 16 * i, last) * vt.st + 8 * (tid & 15);
        k = (int64_t)min(16 * (tid >> 6) + (lane & 15), last) * kt.st + 8 * (lane >> 4);
    }
};

// Partial attention of query row bv = (b, qi), L cache rows up to and including the query, over
// selected block `blk` (< 0: none; uniform).  Whole workgroup of 256 threads.  `place()` returns the block's entry in
// the row's ascending list, where the partial result goes; it is called while the block's rows are on their way.
// kFresh: row fresh_row of the caches (-1: none) is being written by this very launch: it is taken from fresh.k_new / v_new.
template <bool kFresh, typename Place>
__device__ inline void attend_block(const Dims &dm, const Tensor &k, const Tensor &v, BlockFetch fetch, const bf16x8 (&bq)[4],
                                    int bv, int b, int qi, int h, int L, int blk, const uint64_t *__restrict__ tree_mask,
                                    float *__restrict__ o_part, float2 *__restrict__ ml_part, Place place,
                                    const AppendArgs *fresh = nullptr, int fresh_row = -1) {
    __shared__ __align__(16) uint16_t Vs[kBlock * kVsPitch];
    __shared__ __align__(16) uint4 Pb[2 * 4 * 16];       // [key half kk][key group g][head]: keys 32kk + 8g .. +7 in bf16
    __shared__ float wmax[4][16], wsum[4][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int G = dm.G;
    const int L_all = L + (dm.n_q - 1 - qi);             // cache rows of the sequence (when L >= 1)
    uint64_t mask_word = 0ull;
    if (tree_mask) mask_word = tree_mask[bv];
    // a tree mask may let a query attend drafted tokens that lie after it in the cache
    const bool valid = L >= 1 && blk >= 0 && (int64_t)blk * kBlock < (tree_mask ? L_all : L);
    if (!valid) {                                        // uniform over the workgroup
        const int cidx = place();
        const int head = tid & 15, chunk = tid >> 4;
        if (head < G) {
            const int64_t pbase = (((int64_t)bv * dm.Hq + h * G + head) * dm.topk + cidx);
            if (chunk == 0) ml_part[pbase] = float2{-INFINITY, 0.f};
            float4 zf = {0.f, 0.f, 0.f, 0.f};
            float4 *op = reinterpret_cast<float4 *>(o_part + pbase * kHeadDim + 8 * chunk);
            op[0] = zf;
            op[1] = zf;
        }
        return;
    }
    const int key0 = blk * kBlock;
    // ---- all loads --------------------------------------------------------------------------------
    // (rows the query may not see are read, in bounds, and masked)
    const int c8 = tid & 15, vr = tid >> 4;
    uint4 vrow[4];
    bf16x8 a[4];
    {
        if (key0 + kBlock > dm.max_seqlen) fetch.rows(k, v, dm.max_seqlen - 1 - key0);
        const __bf16 *kr = k.ptr + (fetch.k_head + (int64_t)key0 * k.st) + fetch.k;
        const __bf16 *vb = v.ptr + (fetch.v_head + (int64_t)key0 * v.st);
        // (its block is the last: all others' addresses are left alone)
        const bool fresh_here = kFresh && fresh_row >= key0 && fresh_row < key0 + kBlock;      // uniform
        if (fresh_here && key0 + 16 * wave + n == fresh_row) kr = fresh->k_new.ptr + b * fresh->k_new.sb + h * fresh->k_new.sh + 8 * g;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) a[ks] = load8(kr + 32 * ks);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const __bf16 *vp = vb + fetch.v[i];
            if (fresh_here && key0 + vr + 16 * i == fresh_row) vp = fresh->v_new.ptr + b * fresh->v_new.sb + h * fresh->v_new.sh + 8 * c8;
            vrow[i] = *reinterpret_cast<const uint4 *>(vp);
        }
    }
    const int cidx = place();
    // ---- which of the block's 64 keys the query attends: bit r = key key0 + r ------------------------
    // Causal: keys up to the query's own position.  Tree mask: every context key (before the drafted
    // tokens), and drafted token j iff bit j of the query's mask word is set.
    uint64_t allow;
    if (!tree_mask) {
        const int nv = L - key0;                         // >= 1
        allow = nv >= 64 ? ~0ull : (1ull << nv) - 1ull;
    } else {
        const int l_ctx = L_all - dm.n_q;                // >= 0
        const uint64_t mw = dm.n_q >= 64 ? mask_word : mask_word & ((1ull << dm.n_q) - 1ull);
        const int sh = key0 - l_ctx;                     // block offset of the first drafted token, negated
        if (sh >= 0) allow = sh < 64 ? mw >> sh : 0ull;
        else allow = sh > -64 ? (mw << -sh) | ((1ull << -sh) - 1ull) : ~0ull;
    }
    // ---- scores of this wave's 16 keys ---------------------------------------------------------------
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) s = mfma16(a[ks], bq[ks], s);
    float x[4], mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        x[j] = ((allow >> (16 * wave + 4 * g + j)) & 1ull) ? s[j] * dm.scale_log2 : -INFINITY;
        mx = fmaxf(mx, x[j]);
    }
    mx = xgroup_max(mx);
    if (g == 0) wmax[wave][n] = mx;
    // ---- value tile to LDS (masked rows as zeros: 0 * garbage must stay 0) ----------------------------
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = vr + 16 * i;
        uint4 y = vrow[i];
        if (!((allow >> r) & 1ull)) y = uint4{0u, 0u, 0u, 0u};
        *reinterpret_cast<uint2 *>(&Vs[r * kVsPitch + 8 * c8]) = uint2{y.x, y.y};
        *reinterpret_cast<uint2 *>(&Vs[r * kVsPitch + 8 * c8 + 4]) = uint2{y.z, y.w};
    }
    __syncthreads();
    const float m = fmaxf(fmaxf(wmax[0][n], wmax[1][n]), fmaxf(wmax[2][n], wmax[3][n]));
    const float m_sub = m == -INFINITY ? 0.f : m;       // -inf only when a tree mask hides the whole block
    float ps = 0.f;
    bf16x4 pv;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float p = fast_exp2(x[j] - m_sub);
        ps += p;
        pv[j] = (__bf16)p;
    }
    // keys 16 wave + 4g + j: half wave/2, group 2 (wave%2) + g/2, elements 4 (g%2) + j
    reinterpret_cast<uint2 *>(Pb)[2 * (((wave >> 1) * 4 + 2 * (wave & 1) + (g >> 1)) * 16 + n) + (g & 1)] = __builtin_bit_cast(uint2, pv);
    ps = xgroup_sum(ps);
    if (g == 0) wsum[wave][n] = ps;
    __syncthreads();
    // ---- O^T[channel, head] for channels 32*wave .. 32*wave+31 ---------------------------------------
    f32x4 o[2];
    o[0] = o[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 pb = __builtin_bit_cast(bf16x8, Pb[(kk * 4 + g) * 16 + n]);       // B: head n, keys 32kk + 8g .. +7
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {                 // A: channel 32 wave + 16ct + n, the same keys: 4 rows x 16 channels per read
            const uint16_t *vp = &Vs[(32 * kk + 8 * g + (n >> 2)) * kVsPitch + 32 * wave + 16 * ct + 4 * (n & 3)];
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)vp);
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(vp + 4 * kVsPitch));
            o[ct] = mfma16(__builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)), pb, o[ct]);
        }
    }
    if (n < G) {                                         // lane: head n, channels 32w + 16ct + 4g .. +3
        const int64_t pbase = (((int64_t)bv * dm.Hq + h * G + n) * dm.topk + cidx);
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
            *reinterpret_cast<float4 *>(o_part + pbase * kHeadDim + 32 * wave + 16 * ct + 4 * g) =
                float4{o[ct][0], o[ct][1], o[ct][2], o[ct][3]};
        if (wave == 0 && g == 0)
            ml_part[pbase] = float2{m, (wsum[0][n] + wsum[1][n]) + (wsum[2][n] + wsum[3][n])};
    }
}

__global__ __launch_bounds__(256) void decode_attn_partial_kernel(Dims dm, Tensor q, Tensor k, Tensor v,
                                                                   const int32_t *__restrict__ seqlens,
                                                                   const int32_t *__restrict__ block_idx,
                                                                   const uint64_t *__restrict__ tree_mask,
                                                                   float *__restrict__ o_part,
                                                                   float2 *__restrict__ ml_part) {
    const int cidx = blockIdx.x, h = blockIdx.y, bv = blockIdx.z;
    int b, qi;
    const int L = query_row(dm, seqlens, bv, b, qi);
    const int blk = block_idx[(((int64_t)b * dm.Hkv + h) * dm.n_q + qi) * dm.topk + cidx];
    bf16x8 bq[1][4];
    QueryOperands<1>(dm, q, b, h, qi).get(nullptr, bq);
    BlockFetch fetch;
    fetch.set(dm, k, v, b, h);
    attend_block<false>(dm, k, v, fetch, bq[0], bv, b, qi, h, L, __builtin_amdgcn_readfirstlane(blk), tree_mask, o_part, ml_part,
                        [cidx] { return cidx; });
}

// Top-k and partial attention in one launch (the one-call decode and verification steps): a step is
// a chain of dependent launches, each costing a launch gap and a memory round trip, and the block
// list is the only thing the attention waits for.  Every one of the k workgroups of a (query row,
// key-value head) repeats the top-k on the same input (same result; workgroup 0 writes it out) and goes on with one
// entry of the result as it stands, best first; the list's ascending order, which decides where the partial result goes,
// is worked out while the block's rows are on their way.  Those whose entry is a forced block rank nothing: their rows are on
// their way while the others rank (32 sequences of 128K: this kernel 12.1 -> 11.7 us, the step 63.6 -> 62.9).
template <int kForm, int kN>
__global__ __launch_bounds__(kPickThreads) void decode_pick_partial_kernel(Dims dm, Tensor q, Tensor k, Tensor v,
                                                                            const int32_t *__restrict__ seqlens,
                                                                            PickInput in,
                                                                            const uint64_t *__restrict__ tree_mask,
                                                                            int32_t *__restrict__ block_idx,
                                                                            float *__restrict__ o_part,
                                                                            float2 *__restrict__ ml_part) {
    extern __shared__ __align__(16) unsigned char pick_smem[];
    arguments_arrive(dm.Hkv, dm.max_seqlen, dm.n_q, seqlens, in.found, in.n_lists, in.list_len, in.blocks, q.ptr, q.sb, q.sh, q.st);
    arguments_arrive(dm.Hq, dm.topk, dm.n_init, k.ptr, k.sb, k.sh, k.st, v.ptr, v.sb, v.sh, v.st, tree_mask);
    arguments_arrive(dm.G, dm.n_local, dm.scale_log2, block_idx, o_part, ml_part);
    const int cidx = blockIdx.x, h = blockIdx.y, bv = blockIdx.z;
    Picker<kForm, kN> picker(in, (int64_t)bv * dm.Hkv + h);
    int b, qi;
    const int L = query_row(dm, seqlens, bv, b, qi);
    bf16x8 bq[1][4];
    QueryOperands<1>(dm, q, b, h, qi).get(nullptr, bq);
    BlockFetch fetch;
    fetch.set(dm, k, v, b, h);
    int32_t *orow = block_idx + (((int64_t)b * dm.Hkv + h) * dm.n_q + qi) * dm.topk;
    __shared__ __align__(16) int mine[kPickWaves][64];
    const int wave = threadIdx.x >> 6;
    int blk = -1, n_sel = 0, at = cidx;
    if (L < 1) {                                          // uniform over the workgroup
        if (cidx == 0 && (int)threadIdx.x < dm.topk) orow[threadIdx.x] = -1;
    } else {
        const RowRange rr(dm, L);
        const int f = cidx - rr.n_pick;
        if (rr.n_pick > 0 && f >= 0) {                    // a forced block, or no block: nothing to rank
            if (cidx < rr.n_sel) {
                blk = f < rr.n_init ? f : rr.lo_local + (f - rr.n_init);
                at = f < rr.n_init ? f : cidx;
            }
        } else {
            n_sel = rr.n_sel;
            const int mine_at = picker.pick(in, rr, L, pick_smem, dm.topk, mine[wave], cidx);
            if (cidx < n_sel) blk = mine_at;
        }
    }
    attend_block<false>(dm, k, v, fetch, bq[0], bv, b, qi, h, L, blk, tree_mask, o_part, ml_part, [&] {
        if (n_sel == 0) return at;
        const int rank = order_row(mine[wave], n_sel, dm.topk, cidx == 0 && wave == 0 ? orow : nullptr);
        return cidx < n_sel ? __builtin_amdgcn_readlane(rank, cidx) : cidx;
    });
}

// ---- short caches: selection, append and partial attention in one kernel -----------------------------------
// Up to kShortTokens cached tokens a row has at most 512 semantic kernels and 128 blocks: one workgroup scores them all
// in registers, so nothing of the selection has to pass through memory and the step is two launches, this one and the
// merge, instead of four -- each of which costs 1.3 to 1.9 us between kernels and a round trip to memory before it does
// anything.  Every one of the k workgroups of a (sequence, key-value head) repeats the selection (128 KB of compressed
// keys at most, from L2) and attends its own entry of the result; workgroup 0 writes the row.
// In a graph, us per step, four launches -> two: 2K G = 4 13.5 -> 8.3, one sequence of 4000 tokens 16.1 -> 11.5, 8000
// 16.1 -> 14.4; 32 sequences of 8000, three launches: 25.8 -> 23.9.
//   mode 0: block list only (infllmv2_select_blocks)       grid (1, Hkv, B n_q)
//   mode 1: append + block list (steps with many rows)      grid (2, Hkv, B)
//   mode 2: append + block list + partial attention         grid (topk, Hkv, B + ceil(B / topk))
// (Mode 2 appends in workgroups behind all others, so that these have the compute units first: behind each row's, 240 units and 20 that append
// took 13.8 us for 5 sequences of 4266, so 12.0; 256 and 32, 8 of 8000, 19.0 and 16.0.)
//   mode 3: block list + partial attention (verification)   grid (topk, Hkv, B n_q)
// Wave w scores kernels 16 kTW w .. +16 kTW - 1, Z = Q . CK^T: lane = kernel, accumulator entries = heads 4g .. 4g+3.
// Drafted tokens: a launch of its own appends them and builds the semantic kernels they complete, then a row is scored by every workgroup that
// attends a block of it (mode 3), or by one (mode 0).  Three or four launches instead of four longer ones, us per step in a graph, one
// sequence: 300 tokens, 4 drafted 14.6 -> 9.6, 900, 16 19.5 -> 15.8, 64 35.4 -> 28.6, 2000, 16 19.8 -> 17.0, 4000, 2 16.9 -> 14.0,
// 16 20.1 -> 18.7, 64 35.0 -> 30.2; at 8000 tokens they meet (8: 17.9 / 18.3, 16: 20.0 / 21.8).
constexpr int kShortTokens = 8192, kShortVerify = 4096;
template <int kTW, int kMode>
__global__ __launch_bounds__(256) void decode_short_kernel(Dims dm, Tensor q, Tensor ck, const int32_t *__restrict__ seqlens,
                                                            AppendArgs ap, int32_t *__restrict__ block_idx,
                                                            float *__restrict__ o_part, float2 *__restrict__ ml_part,
                                                            const uint64_t *__restrict__ tree_mask) {
    constexpr bool kOneRow = kMode == 1 || kMode == 2, kAttends = kMode >= 2;
    constexpr int kKernels = 64 * kTW, kWords = kTW > 4 ? 128 : 64;
    static_assert(16 * kTW <= kWords, "one word per block");
    __shared__ __align__(16) float2 wpart[4][16];
    __shared__ float rs[kKernels + 4];                    // slot 1 + jh: score of kernel jh; slot 0: no kernel
    __shared__ __align__(16) uint64_t words[kWords];
    __shared__ int counts[4][kWords];
    __shared__ int sel[4][64];                            // per wavefront: the selected blocks, ascending
    __shared__ __align__(16) uint32_t newrow[kOneRow ? 64 : 4];
    arguments_arrive(dm.Hkv, dm.G, dm.max_seqlen, dm.topk, dm.n_init, dm.n_local, seqlens, ck.ptr, ck.sb, ck.sh, ck.st, block_idx);
    arguments_arrive(q.ptr, q.sb, q.sh, dm.scale_log2, dm.Hq, o_part, ml_part, dm.batch);
    int cidx = blockIdx.x, h = blockIdx.y, bv = blockIdx.z;
    if (kMode == 2 && bv >= dm.batch) {                   // behind all others: one appends to each (sequence, key-value head)
        const int at = ((bv - dm.batch) * dm.Hkv + h) * dm.topk + cidx;
        if (at >= dm.batch * dm.Hkv) return;
        bv = at / dm.Hkv;
        h = at - bv * dm.Hkv;
        cidx = dm.topk;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int G = dm.G;
    const int b = kOneRow || dm.n_q == 1 ? bv : (int)__umulhi((uint32_t)bv, dm.n_q_inv), qi = kOneRow ? 0 : bv - b * dm.n_q;
    const int32_t L_raw = uniform_load(seqlens + b);
    __builtin_amdgcn_sched_barrier(0);
    const QueryOperands<1> query(dm, q, b, h, qi);
    const int jw = 16 * kTW * wave;                       // this wave's first kernel
    int64_t ck_wave_at = b * ck.sb + h * ck.sh + (int64_t)jw * ck.st, ck_lane = n * ck.st + 8 * g;       // (while the length is on its way)
    asm volatile("" : "+s"(ck_wave_at), "+v"(ck_lane));
    if (kOneRow && cidx == (kMode == 2 ? dm.topk : 1)) {  // copies the new rows into the caches
        const int c8 = (tid & 15) * 8;
        if (L_raw < 1 || L_raw > dm.max_seqlen || tid >= 32) return;
        if (tid < 16)
            *reinterpret_cast<uint4 *>(ap.k.ptr + b * ap.k.sb + h * ap.k.sh + (int64_t)(L_raw - 1) * ap.k.st + c8) =
                *reinterpret_cast<const uint4 *>(ap.k_new.ptr + b * ap.k_new.sb + h * ap.k_new.sh + c8);
        else
            *reinterpret_cast<uint4 *>(ap.v.ptr + b * ap.v.sb + h * ap.v.sh + (int64_t)(L_raw - 1) * ap.v.st + c8) =
                *reinterpret_cast<const uint4 *>(ap.v_new.ptr + b * ap.v_new.sb + h * ap.v_new.sh + c8);
        return;
    }
    const int L = kOneRow ? clamp_len(L_raw, dm.max_seqlen) : row_len(dm, clamp_len(L_raw, dm.max_seqlen), qi);
    const bool live = kOneRow && L_raw >= 1 && L_raw <= dm.max_seqlen;        // as the stand-alone append: others are skipped
    int32_t *orow = block_idx + (kOneRow ? (int64_t)b * dm.Hkv + h : ((int64_t)b * dm.Hkv + h) * dm.n_q + qi) * dm.topk;
    const int n_vis = num_kernels(L);
    const RowRange rr(dm, max(L, 1));
    bf16x8 a[kTW][4], bq[1][4];
    if (n_vis > 0 && rr.n_pick > 0) {                     // (otherwise every block is forced, or there is nothing to score)
        const __bf16 *ck_wave = ck.ptr + ck_wave_at;
        const bool all = jw + 16 * kTW <= n_vis;          // uniform over the wave; rows past the last kernel repeat it and are masked below
#pragma unroll
        for (int i = 0; i < kTW; ++i) {
            const int64_t at = all ? 16 * i * ck.st + ck_lane : min(16 * i + n, n_vis - 1 - jw) * ck.st + 8 * g;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a[i][ks] = load8(ck_wave + at + 32 * ks);
        }
    } else {
#pragma unroll
        for (int i = 0; i < kTW; ++i)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a[i][ks] = zero8();
    }
    __builtin_amdgcn_sched_barrier(0);
    query.get(nullptr, bq);
    std::conditional_t<kAttends, BlockFetch, int> fetch{};
    if constexpr (kAttends) fetch.set(dm, ap.k, ap.v, b, h);
    int blk = -1;
    if (L < 1) {                                          // uniform over the workgroup
        if (cidx == 0 && tid < dm.topk) orow[tid] = -1;
    } else {
        if constexpr (kOneRow) {
            // the semantic kernel the new token completes: rows L-32 .. L-2 from the cache, row L-1 from k_new; lane = channels
            // 2*lane, 2*lane+1
            const int jh_new = n_vis - 1;
            const bool closes = live && L >= kKernel && (L - kKernel) % kStride == 0;
            if (closes && jh_new >= jw && jh_new < jw + 16 * kTW && (rr.n_pick > 0 || cidx == 0)) {   // uniform over the wave
                const __bf16 *kc = ap.k.ptr + (b * ap.k.sb + h * ap.k.sh + (int64_t)(L - kKernel) * ap.k.st);
                uint32_t rowv[kKernel];
#pragma unroll
                for (int t = 0; t < kKernel - 1; ++t) rowv[t] = reinterpret_cast<const uint32_t *>(kc + t * ap.k.st)[lane];
                rowv[kKernel - 1] = reinterpret_cast<const uint32_t *>(ap.k_new.ptr + (b * ap.k_new.sb + h * ap.k_new.sh))[lane];
                const uint32_t packed = kernel_mean(rowv);
                newrow[lane] = packed;
                if (cidx == 0) *reinterpret_cast<uint32_t *>(ck.ptr + b * ck.sb + h * ck.sh + (int64_t)jh_new * ck.st + 2 * lane) = packed;
                __builtin_amdgcn_wave_barrier();          // same wavefront: LDS keeps the order
                // (the row's place in ck may or may not hold it yet: workgroup 0 is storing it)
#pragma unroll
                for (int i = 0; i < kTW; ++i)
                    if (jw + 16 * i + n >= jh_new) {
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks)
                            a[i][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&newrow[16 * ks + 4 * g]));
                    }
            }
        }
        uint64_t chosen[kWords / 64];                     // picked blocks as bits, 64 per word
#pragma unroll
        for (int i = 0; i < kWords / 64; ++i) chosen[i] = 0ull;
        if (rr.n_pick > 0) {
            f32x4 x[kTW];
            float m[4], s[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) m[j] = -INFINITY;
#pragma unroll
            for (int i = 0; i < kTW; ++i) {
                f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) z = mfma16(bq[0][ks], a[i][ks], z);
                const bool vis = jw + 16 * i + n < n_vis;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[i][j] = vis ? z[j] * dm.scale_log2 : -INFINITY;
                    m[j] = fmaxf(m[j], x[i][j]);
                }
            }
            // log-sum-exp per head: over the wave's kernels, then over the waves
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                m[j] = row_reduce(m[j], [](float u, float w) { return fmaxf(u, w); });
                const float mu = m[j] == -INFINITY ? 0.f : m[j];
                float t = 0.f;
#pragma unroll
                for (int i = 0; i < kTW; ++i) t += fast_exp2(x[i][j] - mu);
                s[j] = row_reduce(t, [](float u, float w) { return u + w; });
            }
            if (n == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) wpart[wave][4 * g + j] = float2{m[j], s[j]};
            }
            if (tid == 0) rs[0] = -INFINITY;
            __syncthreads();
            float lse_j[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float2 p[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) p[w] = wpart[w][4 * g + j];
                const float M = fmaxf(fmaxf(p[0].x, p[1].x), fmaxf(p[2].x, p[3].x)), mu = M == -INFINITY ? 0.f : M;
                float S = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) S += p[w].y * fast_exp2(p[w].x - mu);
                lse_j[j] = M + fast_log2(S);
            }
            // group mean of the kernel scores; 16-lane group i % 4 keeps tile i
#pragma unroll
            for (int i = 0; i < kTW; ++i) {
                float acc = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (4 * g + j < G) acc += fast_exp2(x[i][j] - lse_j[j]);
                acc = xgroup_sum(acc);
                const int jh = jw + 16 * i + n;
                if (g == (i & 3)) rs[1 + jh] = jh < n_vis ? fminf(fmaxf(acc * (1.f / G), kScoreFloor), kScoreCeil) : -INFINITY;
            }
            __syncthreads();
            if (tid < kWords) {                           // 5/4 max-pool: kernels 4j-1 .. 4j+3 = rs[4j .. 4j+4]
                uint64_t e = 0ull;
                if (tid < 16 * kTW) {
                    float r = rs[4 * tid];
#pragma unroll
                    for (int y = 1; y < 5; ++y) r = fmaxf(r, rs[4 * tid + y]);
                    e = pick_element(r, tid, rr.n_init, rr.jc_max);
                }
                words[tid] = e;
            }
            __syncthreads();
            // top-k by counting: every word against a quarter of the words on each wave; the words are in block order, so
            // the picked blocks come out ascending
#pragma unroll
            for (int i = 0; i < kWords / 64; ++i)
                counts[wave][64 * i + lane] = count_larger(words + wave * (kWords / 4), kWords / 4, words[64 * i + lane]);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kWords / 64; ++i) {
                const int at = 64 * i + lane;
                const int beaten = (counts[0][at] + counts[1][at]) + (counts[2][at] + counts[3][at]);
                chosen[i] = __ballot(words[at] >= kPickValid && beaten < rr.n_pick);
            }
        }
        // the row: forced leading blocks, picked blocks, forced trailing blocks -- ascending as they stand
        const uint64_t below = (1ull << lane) - 1ull;
        int *mine = sel[wave];
        int at = rr.n_init;
#pragma unroll
        for (int i = 0; i < kWords / 64; ++i) {
            if ((chosen[i] >> lane) & 1ull) mine[at + __popcll(chosen[i] & below)] = 64 * i + lane;
            at += __popcll(chosen[i]);
        }
        if (lane < rr.n_init) mine[lane] = lane;
        if (lane >= at && lane < rr.n_sel) mine[lane] = rr.lo_local + (lane - at);
        __builtin_amdgcn_wave_barrier();
        if (cidx == 0 && wave == 0 && lane < dm.topk) orow[lane] = lane < rr.n_sel ? mine[lane] : -1;
        if (cidx < rr.n_sel) blk = __builtin_amdgcn_readfirstlane(mine[cidx]);
    }
    if constexpr (kMode == 2)
        attend_block<true>(dm, ap.k, ap.v, fetch, bq[0], b, b, 0, h, L, blk, nullptr, o_part, ml_part, [cidx] { return cidx; }, &ap,
                           live ? L_raw - 1 : -1);
    if constexpr (kMode == 3)
        attend_block<false>(dm, ap.k, ap.v, fetch, bq[0], bv, b, qi, h, L, blk, tree_mask, o_part, ml_part, [cidx] { return cidx; });
}

// ---- attention, part 2: merge the k partials of every query head ---------------------------------
// grid (Hq, n_q, B), one wavefront: lane = two channels.  kTop is the top-k rounded up to 8, 16, 32 or 64; entries past the top-k lie
// outside the loads' resources and read 0.
// Bound by latency: arguments, one round trip for everything the partials say, and a chain of instructions.  So all arguments and
// all loads are asked for before anything is used and no branch lies between (the compiler sinks a load into the branch that
// uses it), and a lane works out one entry's weight, which the others read from it.
template <int kTop>
__global__ __launch_bounds__(64) void decode_merge_kernel(Dims dm, const float *__restrict__ o_part,
                                                           const float2 *__restrict__ ml_part, Tensor out,
                                                           float *__restrict__ lse) {
    arguments_arrive(dm.Hq, dm.topk, dm.n_q, o_part, ml_part, out.ptr, out.sb, out.sh, out.st, lse);
    const int hq = blockIdx.x, qi = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
    const int64_t row = ((int64_t)b * dm.n_q + qi) * dm.Hq + hq, pbase = row * dm.topk;
    const int mine = lane & (kTop - 1);
    const auto ml_rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float2 *>(ml_part + pbase), 0, dm.topk * (int)sizeof(float2), 0x00027000);
    const auto o_rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(o_part + pbase * kHeadDim), 0,
                                                          dm.topk * kHeadDim * (int)sizeof(float), 0x00027000);
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 ml2 = __builtin_amdgcn_raw_buffer_load_b64(ml_rows, mine * (int)sizeof(float2), 0, 0);
    u32x2 ov[kTop];
#pragma unroll
    for (int c = 0; c < kTop; ++c)
        ov[c] = __builtin_amdgcn_raw_buffer_load_b64(o_rows, lane * (int)sizeof(float2) + c * kHeadDim * (int)sizeof(float), 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    const float2 ml = {mine < dm.topk ? __uint_as_float(ml2[0]) : -INFINITY, __uint_as_float(ml2[1])};
    const auto larger = [](float x, float y) { return fmaxf(x, y); };
    const auto sum = [](float x, float y) { return x + y; };
    float M = row_reduce(ml.x, larger);
    if constexpr (kTop >= 32) M = xgroup_reduce(M, larger);
    M = M == -INFINITY ? 0.f : M;
    const float w = fast_exp2(ml.x - M);
    float den = lane < kTop ? w * ml.y : 0.f;
    den = row_reduce(den, sum);
    if constexpr (kTop >= 32) den = xgroup_reduce(den, sum);
    den = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(den)));
    float2 num = {0.f, 0.f};
#pragma unroll
    for (int c = 0; c < kTop; ++c) {
        const float wc = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), c));
        num.x += wc * __uint_as_float(ov[c][0]);
        num.y += wc * __uint_as_float(ov[c][1]);
    }
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 o;                                            // (quotients: a reciprocal for both would round once more, and saves under 0.1 us a step)
    o[0] = (__bf16)(den > 0.f ? num.x / den : 0.f);
    o[1] = (__bf16)(den > 0.f ? num.y / den : 0.f);
    *reinterpret_cast<bf16x2 *>(out.ptr + b * out.sb + qi * out.st + (int64_t)hq * out.sh + 2 * lane) = o;
    if (lane == 0) lse[row] = den > 0.f ? (M + fast_log2(den)) * kLn2 : -INFINITY;
}

// ---- host side -------------------------------------------------------------------------------------
static inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Part 2, verification: tiles per wave, and so blocks per list of the top-k: four where that leaves a workgroup for every compute
// unit, or for every second where lists of 32 blocks would be more than 32 and could not be merged as they are.  Measured (us per step, two / four):
// 128K, 4 drafted tokens 20.5 / 22.1, 16 27.9 / 27.6, 64 62.1 / 59.8; 120K, 16 (240 workgroups of four) 25.4 / 23.3, 70K, 16 (144) 24.5 / 23.3, 120K,
// 4 (60) 19.4 / 19.3; 64K, 16 (128) 22.0 / 22.9.
static int verify_tiles2(const Dims &dm) {
    const int64_t wide = (int64_t)((dm.max_seqlen + 64 * kBlock - 1) / (64 * kBlock)) * dm.Hkv * dm.batch * ((dm.n_q + kVerifyQT - 1) / kVerifyQT);
    return wide >= (dm.max_seqlen > 32 * 32 * kBlock ? 128 : 256) ? 4 : 2;
}

struct DecodeSelLayout {
    int32_t n_c_cap, n_part, nb_cap;
    int32_t list_blocks, n_lists, list_len;           // sorted lists of pick words, one per list_blocks blocks; 0: a row of scores
    size_t z_bytes, part_bytes, r_bytes;              // z: logits, plain decode only; r: those lists, or rows of nb_cap scores
    size_t found;                                     // where the lists, or the rows, begin
};
static DecodeSelLayout decode_sel_layout(const Dims &dm) {
    DecodeSelLayout l;
    int32_t n_c = num_kernels(dm.max_seqlen);
    l.n_c_cap = (n_c + 255) / 256 * 256;
    if (l.n_c_cap < 256) l.n_c_cap = 256;
    l.n_part = l.n_c_cap / (64 * (dm.n_q == 1 ? decode_tiles_per_wave(dm) : kVerifyTiles));
    l.nb_cap = ((dm.max_seqlen + kBlock - 1) / kBlock + 63) / 64 * 64;
    const size_t rows = (size_t)dm.batch * dm.n_q;
    l.z_bytes = dm.n_q == 1 ? align256(rows * dm.Hq * l.n_c_cap * sizeof(float)) : 0;
    l.part_bytes = align256(rows * dm.Hq * (dm.n_q == 1 ? l.n_c_cap / (64 * decode_tiles_scratch(dm)) : l.n_part) * sizeof(float2));
    l.list_blocks = dm.n_q == 1 ? kListBlocks : 16 * verify_tiles2(dm);
    l.n_lists = max(1, (dm.max_seqlen + kBlock * l.list_blocks - 1) / (kBlock * l.list_blocks));
    l.list_len = min(l.list_blocks, max(1, dm.topk - dm.n_init - dm.n_local));
    // Verification: two sets of partials and a row of scores, whatever the lists, so that the scratch grows with the rows alone.  Lists
    // that take more than the row begin in the second set (the approximate log-sum-exp's alone), or give way to the scores (128K
    // tokens, 16 drafted, G = 4, top-k 32: 24.9 us by lists, 24.5 by scores; top-k 64 43.1 and 49.5).
    const size_t lists = rows * dm.Hkv * l.n_lists * l.list_len * sizeof(uint64_t);
    l.r_bytes = align256(dm.n_q == 1 ? lists : rows * dm.Hkv * l.nb_cap * sizeof(float));
    l.found = l.z_bytes + 2 * l.part_bytes;
    if (lists > l.r_bytes) {
        if (dm.rho == 1 && lists <= l.r_bytes + l.part_bytes) l.found -= l.part_bytes;
        else l.list_len = 0;
    }
    return l;
}

size_t select_decode_ws_bytes(const Dims &dm) {
    DecodeSelLayout l = decode_sel_layout(dm);
    return l.z_bytes + 2 * l.part_bytes + l.r_bytes;
}

// One workgroup per row can score it all (see decode_short_kernel); the approximate log-sum-exp keeps the long path.
static bool short_cache(const Dims &dm) { return dm.rho == 1 && dm.max_seqlen <= (dm.n_q == 1 ? kShortTokens : kShortVerify); }
// Fused top-k and attention: every workgroup repeats the top-k of its row, which is free while compute units idle and
// costs throughput once the launch fills the machine many times over; merging sorted lists (up to 32 of up to 16 words: any context in plain decode,
// in verification up to 131072 tokens, or 65536 where its lists are of 32 blocks) costs less than counting.  Measured (us per step,
// fused / apart), merged: 1536 units 32.6 / 34.8 (48 sequences of 20K), 2048 37.4 / 39.2 (64), 34.0 / 36.0 and 33.2 / 34.8 (64 and 2 x 32 drafted
// tokens at 30K); counted: 1024 56.6 / 58.3, 42.3 / 44.0, 1920 31.5 / 30.1 (top-k 48) and 46.3 / 38.5 (30 drafted, top-k 64).
static bool fuse_units(const Dims &dm, bool merged) {  // by (row, key-value head, block) workgroups
    return (int64_t)dm.batch * dm.n_q * dm.Hkv * dm.topk <= (merged ? 2048 : 1024);
}

static int short_tiles(const Dims &dm) {              // tiles of 16 kernels (16 blocks) per wave
    const int n_blocks = (dm.max_seqlen + kBlock - 1) / kBlock;
    return n_blocks <= 16 ? 1 : n_blocks <= 32 ? 2 : n_blocks <= 64 ? 4 : 8;
}
// Repeating the whole selection in every attention workgroup beats a launch for it while the workgroups fit the chip a
// few times over; the more kernels there are to score, the earlier that ends.  Measured (us per step, fused / apart; a launch more costs an eager
// caller up to 3 us beside): 900 tokens 768 units 13.4 / 15.5, 2048 25.7 / 24.4; 2000 tokens 512 13.3 / 14.2 and 11.0 / 11.4, 768 15.8 / 16.0 and
// 13.2 / 12.9; 4000 tokens 256 11.3 / 12.8, 384 14.5 / 14.6, 512 15.2 / 15.2; 8000 tokens 256 14.4 / 15.9, 320 19.3 / 17.1.  Drafted tokens: 900
// tokens 512 units 15.8 / 17.1, 2048 29.4 / 28.6; 2000 tokens 512 17.0 / 17.8, 1024 22.7 / 22.3; 4000 tokens 512 18.7 / 19.2, 2048 38.3 / 30.2.
static bool fuse_short(const Dims &dm) {
    const int64_t units = (int64_t)dm.batch * dm.n_q * dm.Hkv * dm.topk;
    const int t = short_tiles(dm);
    return units <= (t == 1 ? 1024 : t == 2 ? 768 : t == 4 ? 512 : 256);
}

template <int kMode>
static int launch_short(const Dims &dm, Tensor q, Tensor ck, const AppendArgs &ap, const int32_t *seqlens, int32_t *block_idx,
                        float *o_part, float2 *ml_part, hipStream_t stream, const uint64_t *tree_mask = nullptr) {
    const dim3 grid(kMode >= 2 ? dm.topk : kMode + 1, dm.Hkv, dm.batch * dm.n_q + (kMode == 2 ? (dm.batch + dm.topk - 1) / dm.topk : 0)), block(256);
    timing_begin("decode_short_kernel", stream);
#define INFLLMV2_SHORT(TW) \
    hipLaunchKernelGGL((decode_short_kernel<TW, kMode>), grid, block, 0, stream, dm, q, ck, seqlens, ap, block_idx, o_part, ml_part, tree_mask)
    switch (short_tiles(dm)) {
        case 1: INFLLMV2_SHORT(1); break;
        case 2: INFLLMV2_SHORT(2); break;
        case 4: INFLLMV2_SHORT(4); break;
        default: INFLLMV2_SHORT(8); break;
    }
#undef INFLLMV2_SHORT
    timing_end(stream);
    return (int)hipGetLastError();
}

static auto scores_z_kernel(int G, bool sorted) {
    switch (G) {
        case 1: return sorted ? decode_scores_z_kernel<1, true> : decode_scores_z_kernel<1, false>;
        case 2: return sorted ? decode_scores_z_kernel<2, true> : decode_scores_z_kernel<2, false>;
        case 4: return sorted ? decode_scores_z_kernel<4, true> : decode_scores_z_kernel<4, false>;
        case 8: return sorted ? decode_scores_z_kernel<8, true> : decode_scores_z_kernel<8, false>;
        default: return sorted ? decode_scores_z_kernel<16, true> : decode_scores_z_kernel<16, false>;
    }
}

int launch_select_decode(const Dims &dm, Tensor q, Tensor ck, const int32_t *seqlens,
                         int32_t *block_idx, void *ws, hipStream_t stream, const AppendArgs *append,
                         AttendArgs *attend) {
    if (dm.batch <= 0) return 0;
    if (short_cache(dm) && !append) {
        const AppendArgs none = {q, q, q, q};                        // unused placeholders
        return launch_short<0>(dm, q, ck, none, seqlens, block_idx, nullptr, nullptr, stream);
    }
    DecodeSelLayout l = decode_sel_layout(dm);
    if (l.n_c_cap > 16384) return (int)hipErrorInvalidValue;         // rejected earlier by the C ABI
    char *wsb = reinterpret_cast<char *>(ws);
    float *zbuf = reinterpret_cast<float *>(wsb);
    float2 *part = reinterpret_cast<float2 *>(wsb + l.z_bytes);
    float2 *part_c = reinterpret_cast<float2 *>(wsb + l.z_bytes + l.part_bytes);
    void *found = wsb + l.found;
    const int rows = dm.batch * dm.n_q;                              // <= 65535, checked by the C ABI
    const int n_qt = (dm.n_q + kVerifyQT - 1) / kVerifyQT;
    const uint32_t n_qt_inv = n_qt > 1 ? (uint32_t)((1ull << 32) / (uint32_t)n_qt) + 1u : 0u;   // i / n_qt, as n_q_inv
    const float2 *part_lse = dm.rho > 1 ? part_c : part;
    timing_begin("decode_logits_kernel", stream);
    const AppendArgs no_append = {q, q, q, q};                       // unused placeholders
    const bool tw4 = decode_tiles_per_wave(dm) == 4;
    // Workgroups that append.  Plain decode: one per (sequence, key-value head), at the end of its chunks, or, where these fill the chip about once to
    // four times over, behind all others, so that no chunk waits for a compute unit that one of them has taken (4 sequences of 128K 19.3 -> 16.7 us per
    // step, 8 22.6 -> 20.3; 120 chunks 14.0 and 14.3, 4096 56.6 and 57.3).  Verification: always behind all.
    const int64_t chunks = (int64_t)l.n_part * dm.Hkv * dm.batch;
    const bool behind = append && (dm.n_q > 1 || (chunks > 240 && chunks <= 1024));
    const int32_t n_wg = verify_columns(dm, n_qt, l.n_part) + (append && !behind ? 1 : 0);
    const int32_t planes = behind ? (int32_t)(((int64_t)dm.batch * ((dm.n_q + 7) / 8) + n_wg - 1) / n_wg) : 0;
    const dim3 grid1(n_wg, dm.Hkv, dm.batch * n_qt + planes);
#define INFLLMV2_LOGITS(APPEND, TW, ARG)                                                                        \
    hipLaunchKernelGGL((decode_logits_kernel<1, APPEND, TW>), grid1, dim3(256), 0, stream, dm, q, ck, seqlens, \
                       zbuf, l.n_c_cap, part, part_c, l.n_part, ARG, 0u)
    if (dm.n_q == 1 && append) {
        if (tw4) INFLLMV2_LOGITS(true, 4, *append);
        else INFLLMV2_LOGITS(true, 2, *append);
    } else if (dm.n_q == 1) {
        if (tw4) INFLLMV2_LOGITS(false, 4, no_append);
        else INFLLMV2_LOGITS(false, 2, no_append);
    } else {
        if (append)
            hipLaunchKernelGGL((decode_logits_kernel<kVerifyQT, true, kVerifyTiles>), grid1, dim3(256), 0, stream, dm, q, ck, seqlens,
                               nullptr, 0, part, part_c, l.n_part, *append, n_qt_inv);
        else
            hipLaunchKernelGGL((decode_logits_kernel<kVerifyQT, false, kVerifyTiles>), grid1, dim3(256), 0, stream, dm, q, ck, seqlens,
                               nullptr, 0, part, part_c, l.n_part, no_append, n_qt_inv);
    }
#undef INFLLMV2_LOGITS
    timing_end(stream);
    timing_begin("decode_scores_kernel", stream);
    if (dm.n_q == 1)
        hipLaunchKernelGGL(scores_z_kernel(dm.G, l.list_len <= kMergePicks), dim3(l.n_lists, dm.Hkv, dm.batch), dim3(kScoreThreads), 0,
                           stream, dm, seqlens, zbuf, part_lse, l.n_c_cap, l.n_part, 64 * decode_tiles_per_wave(dm),
                           reinterpret_cast<uint64_t *>(found), l.list_len);
    else
        hipLaunchKernelGGL((l.list_blocks == 64 ? decode_scores_kernel<kVerifyQT, 4> : decode_scores_kernel<kVerifyQT, 2>),
                           dim3(l.n_lists, dm.Hkv, dm.batch * n_qt), dim3(512), 0, stream, dm, q, ck, seqlens, part_lse, l.n_part,
                           found, l.list_len, l.nb_cap, n_qt_inv);
    timing_end(stream);
    const bool lists = l.list_len > 0;
    const int n_elements = lists ? l.n_lists * l.list_len : (dm.max_seqlen + kBlock - 1) / kBlock;
    const int vpt = (n_elements + kPickThreads - 1) / kPickThreads;
    if (vpt > kPickMaxVPT) return (int)hipErrorInvalidValue;         // rejected earlier by the C ABI
    const PickInput in = {found, l.n_lists, l.list_len, (1 << 20) / l.n_lists + 1, l.list_blocks, l.nb_cap};
    const bool merged = lists && l.list_len <= kMergePicks && l.n_lists <= 32;
    if (attend) attend->fused = fuse_units(dm, merged);
    const bool fused = attend && attend->fused;
    timing_begin(fused ? "decode_pick_partial_kernel" : "decode_pick_kernel", stream);
#define INFLLMV2_PICK(FORM, N)                                                                                          \
    do {                                                                                                                \
        const size_t lds = FORM <= kCount ? pick_shared_bytes(dm.topk, N) : 0;                                          \
        if (fused)                                                                                                      \
            hipLaunchKernelGGL((decode_pick_partial_kernel<FORM, N>), dim3(dm.topk, dm.Hkv, rows), dim3(kPickThreads),  \
                               lds, stream, dm, q, attend->k, attend->v, seqlens, in, attend->tree_mask, block_idx,     \
                               attend->o_part, attend->ml_part);                                                        \
        else                                                                                                            \
            hipLaunchKernelGGL((decode_pick_kernel<FORM, N>), dim3(rows * dm.Hkv), dim3(kPickThreads), lds, stream, dm, \
                               seqlens, in, block_idx);                                                                 \
    } while (0)
    if (merged) {
        if (l.n_lists <= 4) INFLLMV2_PICK(kMerge, 1);
        else if (l.n_lists <= 8) INFLLMV2_PICK(kMerge, 2);
        else if (l.n_lists <= 16) INFLLMV2_PICK(kMergeShared, 1);
        else INFLLMV2_PICK(kMergeShared, 2);
    } else if (lists) {
        if (vpt <= 1) INFLLMV2_PICK(kCount, 1);
        else if (vpt <= 2) INFLLMV2_PICK(kCount, 2);
        else if (vpt <= 4) INFLLMV2_PICK(kCount, 4);
        else if (vpt <= 8) INFLLMV2_PICK(kCount, 8);
        else INFLLMV2_PICK(kCount, 16);
    } else {
        if (vpt <= 4) INFLLMV2_PICK(kScores, 4);
        else if (vpt <= 8) INFLLMV2_PICK(kScores, 8);
        else INFLLMV2_PICK(kScores, 16);
    }
#undef INFLLMV2_PICK
    timing_end(stream);
    return (int)hipGetLastError();
}

size_t attn_decode_ws_bytes(const Dims &dm) {
    const size_t o = align256((size_t)dm.batch * dm.n_q * dm.Hq * dm.topk * kHeadDim * sizeof(float));
    const size_t ml = align256((size_t)dm.batch * dm.n_q * dm.Hq * dm.topk * sizeof(float2));
    return o + ml;
}

static void attn_decode_ws(const Dims &dm, void *ws, float *&o_part, float2 *&ml_part) {
    const size_t o_bytes = align256((size_t)dm.batch * dm.n_q * dm.Hq * dm.topk * kHeadDim * sizeof(float));
    o_part = reinterpret_cast<float *>(ws);
    ml_part = reinterpret_cast<float2 *>(reinterpret_cast<char *>(ws) + o_bytes);
}

static void launch_decode_partial(const Dims &dm, Tensor q, Tensor k, Tensor v, const int32_t *seqlens,
                                  const int32_t *block_idx, const uint64_t *tree_mask, float *o_part, float2 *ml_part,
                                  hipStream_t stream) {
    timing_begin("decode_attn_partial_kernel", stream);
    hipLaunchKernelGGL(decode_attn_partial_kernel, dim3(dm.topk, dm.Hkv, dm.batch * dm.n_q), dim3(256), 0, stream,
                       dm, q, k, v, seqlens, block_idx, tree_mask, o_part, ml_part);
    timing_end(stream);
}

static int launch_decode_merge(const Dims &dm, const float *o_part, const float2 *ml_part, Tensor out, float *lse,
                               hipStream_t stream) {
    timing_begin("decode_merge_kernel", stream);
    const dim3 grid(dm.Hq, dm.n_q, dm.batch), block(64);
    if (dm.topk <= 8) hipLaunchKernelGGL(decode_merge_kernel<8>, grid, block, 0, stream, dm, o_part, ml_part, out, lse);
    else if (dm.topk <= 16) hipLaunchKernelGGL(decode_merge_kernel<16>, grid, block, 0, stream, dm, o_part, ml_part, out, lse);
    else if (dm.topk <= 32) hipLaunchKernelGGL(decode_merge_kernel<32>, grid, block, 0, stream, dm, o_part, ml_part, out, lse);
    else hipLaunchKernelGGL(decode_merge_kernel<64>, grid, block, 0, stream, dm, o_part, ml_part, out, lse);
    timing_end(stream);
    return (int)hipGetLastError();
}

int launch_attn_decode(const Dims &dm, Tensor q, Tensor k, Tensor v, const int32_t *seqlens,
                       const int32_t *block_idx, const uint64_t *tree_mask, Tensor out, float *lse, void *ws,
                       hipStream_t stream) {
    if (dm.batch <= 0) return 0;
    float *o_part;
    float2 *ml_part;
    attn_decode_ws(dm, ws, o_part, ml_part);
    launch_decode_partial(dm, q, k, v, seqlens, block_idx, tree_mask, o_part, ml_part, stream);
    return launch_decode_merge(dm, o_part, ml_part, out, lse, stream);
}

// One decode step for one query per sequence: cache append + selection + attention.  Four launches (five with the top-k in one of
// its own, see fuse_units); two or three up to kShortTokens (see fuse_short).
int launch_decode_step(const Dims &dm, Tensor q, Tensor ck, const AppendArgs &append, const int32_t *seqlens,
                       int32_t *block_idx, Tensor out, float *lse, void *ws_select, void *ws_attn,
                       hipStream_t stream) {
    if (dm.batch <= 0) return 0;
    AttendArgs at = {append.k, append.v, nullptr, false, nullptr, nullptr};
    attn_decode_ws(dm, ws_attn, at.o_part, at.ml_part);
    if (short_cache(dm)) {
        const bool fused = fuse_short(dm);
        const int err = fused ? launch_short<2>(dm, q, ck, append, seqlens, block_idx, at.o_part, at.ml_part, stream)
                                       : launch_short<1>(dm, q, ck, append, seqlens, block_idx, nullptr, nullptr, stream);
        if (err) return err;
        if (!fused) launch_decode_partial(dm, q, append.k, append.v, seqlens, block_idx, nullptr, at.o_part, at.ml_part, stream);
        return launch_decode_merge(dm, at.o_part, at.ml_part, out, lse, stream);
    }
    const int err = launch_select_decode(dm, q, ck, seqlens, block_idx, ws_select, stream, &append, &at);
    if (err) return err;
    if (!at.fused) launch_decode_partial(dm, q, append.k, append.v, seqlens, block_idx, nullptr, at.o_part, at.ml_part, stream);
    return launch_decode_merge(dm, at.o_part, at.ml_part, out, lse, stream);
}

// One verification step for n_q drafted tokens per sequence: append (+ completed semantic kernels),
// selection per drafted token, tree-masked attention; four launches (one more with the top-k in one of its own, and with the
// append in one of its own for the approximate log-sum-exp); three or four up to kShortVerify.
int launch_verify_step(const Dims &dm, Tensor q, Tensor ck, const AppendArgs &append, const int32_t *seqlens,
                       const uint64_t *tree_mask, int32_t *block_idx, Tensor out, float *lse, void *ws_select,
                       void *ws_attn, hipStream_t stream) {
    if (dm.batch <= 0) return 0;
    const bool brief = short_cache(dm);
    const bool folded = dm.n_q > 1 && dm.rho == 1 && !brief;     // (a coarse kernel would need rows that other workgroups are storing)
    int err = folded ? 0 : launch_append_kv(dm, append.k_new, append.v_new, append.k, append.v, &ck, seqlens, stream);
    if (err) return err;
    AttendArgs at = {append.k, append.v, tree_mask, false, nullptr, nullptr};
    attn_decode_ws(dm, ws_attn, at.o_part, at.ml_part);
    if (brief && fuse_short(dm)) {
        err = launch_short<3>(dm, q, ck, append, seqlens, block_idx, at.o_part, at.ml_part, stream, tree_mask);
        return err ? err : launch_decode_merge(dm, at.o_part, at.ml_part, out, lse, stream);
    }
    err = launch_select_decode(dm, q, ck, seqlens, block_idx, ws_select, stream, folded ? &append : nullptr, &at);
    if (err) return err;
    if (!at.fused) launch_decode_partial(dm, q, append.k, append.v, seqlens, block_idx, tree_mask, at.o_part, at.ml_part, stream);
    return launch_decode_merge(dm, at.o_part, at.ml_part, out, lse, stream);
}

}  // namespace infllmv2
