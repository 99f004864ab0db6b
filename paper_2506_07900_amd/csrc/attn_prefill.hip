// Stage 3, prefill: exact softmax attention of every query token over its own selected
// key-value blocks (section 2.1.1, second stage; section 2.1.3 "Different Granularity for
// Query and Key-Value Tokens": the query unit is a token, the key-value unit a 64-token block).
//
// Two kernels.
//
// pack_kv_kernel re-lays every 64-token block of the K and V caches into "fragment-major" order
// in the workspace: the 16 bytes a lane feeds to one 16x16x32 MFMA are contiguous and the 64
// lanes of a fragment are consecutive, so a wavefront fetches an operand fragment as one fully
// coalesced 1 KiB read straight into registers.  V is transposed on the way (the value product
// contracts over keys, which are the strided axis of the cache).
//
// attn_prefill_kernel: a wavefront owns the kTok consecutive query tokens of kTiles MFMA tiles of one
// key-value head; the 16 columns of a tile are the G query heads of 16 / G tokens, so no column is
// padding.  The wavefront walks the union of its tokens' block lists in ascending order; each
// fragment it loads is used for every tile with a token that selected the block (inside a tile the
// columns of the other tokens get probability zero).  Either every wavefront works alone, or the
// four of a workgroup own the same tokens, take every fourth block of the union and merge their
// partial results at the end.  Both contractions are computed
// transposed so that no register shuffles are needed:
//   S^T[key, head] = K[key, :] . Q[head, :]            A = K fragment,   B = Q (registers or LDS)
//   O^T[c,  head] += V^T[c, key] . P^T[key, head]       A = V^T fragment, B = P^T taken straight
// from the accumulator layout of S^T (lane = head column, 4 consecutive keys per 16-lane group),
// with the key order inside the packed V^T rows permuted to match.
#include "token_union.h"

namespace infllmv2 {

constexpr int kFragsPerOperand = 16;                     // 16 fragments of 1 KiB = one 16 KiB operand block
constexpr int kPackedBlockU4 = 2 * kFragsPerOperand * 64; // uint4 per packed (K, V) block: 32 KiB

// Consecutive virtual ids land on the same XCD (hardware deals workgroups round-robin over 8
// XCDs), so neighbouring query tiles -- which share blocks -- share an L2.
__device__ inline uint32_t xcd_contiguous_id(uint32_t bid, uint32_t n) {
    const uint32_t per = n >> 3, rem = n & 7u, x = bid & 7u, slot = bid >> 3;
    return x * per + (x < rem ? x : rem) + slot;
}

// ---- re-layout of one 64-token block per workgroup -------------------------------------------------
// K fragment (ks, mt), lane (g, m):  K[64j + 16mt + m][32ks + 8g .. +7]
// V fragment (dt, kk), lane (g, m), element e:  V[64j + 32kk + (e<4 ? 4g+e : 16+4g+e-4)][16dt + m]
__global__ __launch_bounds__(256) void pack_kv_kernel(Dims dm, Tensor k, Tensor v,
                                                       const int32_t *__restrict__ seqlens,
                                                       uint4 *__restrict__ kvp, int32_t nb_cap, Tensor out,
                                                       float *__restrict__ lse) {
    __shared__ __align__(16) __bf16 Ks[kBlock * 136];
    __shared__ __align__(16) __bf16 Vs[kBlock * 136];
    arguments_arrive(dm.Hkv, dm.G, dm.max_seqlen, dm.fill, seqlens, k.ptr, k.sb, k.sh, k.st, kvp, nb_cap);
    arguments_arrive(v.ptr, v.sb, v.sh, v.st);
    const int j = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    int32_t L = uniform_load(seqlens + b);
    const int tid = threadIdx.x, sc = tid & 15, sr = tid >> 4;
    const __bf16 *kb = k.ptr + (b * k.sb + h * k.sh + (int64_t)j * kBlock * k.st), *vb = v.ptr + (b * v.sb + h * v.sh + (int64_t)j * kBlock * v.st);
    L = L < 0 ? 0 : (L > dm.max_seqlen ? dm.max_seqlen : L);
    auto clear_rows = [&]() {                            // this head's rows of the block's tokens past the end: out = 0, lse = 0
        for (int t = max(j * kBlock, (int)L) + (tid >> 4); t < min((j + 1) * kBlock, dm.max_seqlen); t += 16)
            for (int hq = h * dm.G; hq < (h + 1) * dm.G; ++hq) {
                *reinterpret_cast<uint4 *>(out.ptr + b * out.sb + (int64_t)t * out.st + (int64_t)hq * out.sh + 8 * (tid & 15)) =
                    uint4{0u, 0u, 0u, 0u};
                if ((tid & 15) == 0) lse[((int64_t)b * dm.max_seqlen + t) * dm.Hq + hq] = 0.f;
            }
    };
    const int last = L - 1 - j * kBlock;                 // the block's last row; rows past it repeat it and are stored as zeros
    if (last < 0) {
        if (dm.fill) clear_rows();
        return;
    }
    uint4 xk[4], xv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        xk[i] = *reinterpret_cast<const uint4 *>(kb + min(sr + 16 * i, last) * k.st + 8 * sc);
        xv[i] = *reinterpret_cast<const uint4 *>(vb + min(sr + 16 * i, last) * v.st + 8 * sc);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (dm.fill && last < kBlock - 1) clear_rows();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (sr + 16 * i > last) xk[i] = xv[i] = uint4{0u, 0u, 0u, 0u};
        *reinterpret_cast<uint4 *>(&Ks[(sr + 16 * i) * 136 + 8 * sc]) = xk[i];
        *reinterpret_cast<uint4 *>(&Vs[(sr + 16 * i) * 136 + 8 * sc]) = xv[i];
    }
    __syncthreads();
    uint4 *dst = kvp + ((((int64_t)b * dm.Hkv + h) * nb_cap + j) * kPackedBlockU4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = tid + 256 * i;                 // K chunk: fragment f = c/64, lane = c%64
        const int f = c >> 6, lane = c & 63, m = lane & 15, g = lane >> 4;
        const int ks = f >> 2, mt = f & 3;
        dst[c] = *reinterpret_cast<const uint4 *>(&Ks[(16 * mt + m) * 136 + 32 * ks + 8 * g]);
    }
    const uint16_t *Vu = reinterpret_cast<const uint16_t *>(Vs);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = tid + 256 * i;                 // V chunk
        const int f = c >> 6, lane = c & 63, m = lane & 15, g = lane >> 4;
        const int dt = f >> 1, kk = f & 1;
        uint32_t w[4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            const int e = 2 * e2;                    // elements e, e+1 are consecutive keys
            const int key = 32 * kk + (e < 4 ? 4 * g + e : 16 + 4 * g + e - 4);
            const uint32_t lo = Vu[key * 136 + 16 * dt + m];
            const uint32_t hi = Vu[(key + 1) * 136 + 16 * dt + m];
            w[e2] = lo | (hi << 16);
        }
        dst[kFragsPerOperand * 64 + c] = uint4{w[0], w[1], w[2], w[3]};
    }
}

// ---- attention ---------------------------------------------------------------------------------------
// A block is processed as two halves of 32 keys.  The operand fragments of a block are fetched in
// 8 units of 4 fragments (4 KiB per wavefront), in the order they are consumed:
//   half hs:  K rows of key tile 2hs (all four 32-channel k-steps), K rows of key tile 2hs+1,
//             V^T of the half's 32 keys for channel tiles 0..3, then for channel tiles 4..7
// They rotate through a ring of kNU register buffers: as soon as the matrix cores have consumed
// a unit, the load of the unit kNU places further down the stream (same block, or the next block
// of the wavefront's list) is issued into the same registers, so loads stay in flight under the
// wavefront's own arithmetic.
//
// What bounds it: no unit on its own.  At 32K tokens (2 heads, G = 16, top-k 16) the matrix pipe is busy 32 % of the time, vector
// arithmetic 34 %, and 32 % of the wavefronts' time is waits: inside a wavefront a tile's products and its exponentials follow
// one another (11 % of the matrix time runs under vector work).  It takes 0.73 ms back to back (0.75 with events around
// every launch).  Leaving parts out was measured when it took 0.79, with 2.7 GB past L2, before walks began where the others are (1.9 GB):
// the loads alone 0.69, all but the loads 0.52, the matrix products alone 0.43; without the exponentials 0.74, without
// the value product 0.72, without misses (32 blocks in all) 0.73.  The loads are 16.6 GB, 0.46 ms at the
// 36 TB/s that a kernel of nothing but fragment loads reaches; here they run at 24 - 28, with two, four or eight units of 4 KiB per
// wavefront under way.
// The union of two tokens has 24 blocks, of four 33: four tokens per wavefront, their queries in LDS so that the accumulators
// (128 registers) and a ring of four units fit 256 registers, load 16.6 GB instead of 22.5: 1.00 -> 0.78 ms.
//
// The softmax keeps a per-head reference exponent taken from the data and re-bases it only when
// a partial sum leaves the safe range (or on first use, when it is still NaN): the common path is
// one fma, one exp2 and one add per probability, with no running maximum.  A tile of one token (G = 16) takes the reference before
// its first probabilities instead of after them (2000 of the 24000 cycles of a wavefront's walk at 1500 tokens: 23.0 -> 22.5 us
// at 777 tokens, 36.5 -> 35.7 at 1500, 98.2 -> 96.8 at 4096); with several tokens per tile the test for it costs what it saves.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr float kPsumLimit = 0x1p40f;
constexpr int kNone = 0x7fffffff;

// probabilities 2^(s*c + ne) of 32 keys (two key tiles) of one token in MFMA B layout, and their sum
__device__ __forceinline__ float half_probs(const f32x4 (&s)[2], float c, float ne, bf16x8 &p8) {
    float sum;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float p = fast_exp2(__builtin_fmaf(s[t][j], c, ne));
            sum = t + j ? sum + p : p;
            p8[4 * t + j] = (__bf16)p;
        }
    return sum;
}

template <int kG, int kTiles, int kSplit>
struct AttnCfg {
    // Queries in LDS: with four tiles the registers hold the accumulators.  With two, G = 16 then fits 168 registers and three
    // workgroups share a compute unit: 777 tokens 22.4 -> 20.5 us, 1020 28.1 -> 26.8, 2 x 700 with one head 18.9 -> 17.1 (G = 8:
    // 180 registers, 500 tokens 12.2 -> 11.9; G = 4 and 2: 22.6 -> 23.0 at 2000 tokens, 73.8 -> 75.5 at 7000).
    static constexpr bool kQLds = kTiles > 2 || (kTiles == 2 && kG >= 8);
    static constexpr int kWavesPerSimd = kTiles == 2 && kG == 16 ? 3 : 2;
    static constexpr int kTokPerTile = 16 / kG;           // tokens in the 16 columns of one MFMA tile
    static constexpr int kTok = kTiles * kTokPerTile;     // tokens of a wavefront (of the workgroup when its waves split the blocks)
    static constexpr int kTokPerWg = kSplit > 1 ? kTok : 4 * kTok;
    static constexpr int kCopies = kSplit > 1 ? 1 : 4;    // of the list and the queries: one per wavefront, or shared
    __host__ __device__ static size_t queries_at(int topk) { return kCopies * UnionLds::bytes(kTok, topk); }
    __host__ __device__ static size_t merge_at(int topk) {
        return queries_at(topk) + (kQLds ? (size_t)kCopies * kTiles * 4 * 64 * sizeof(uint4) : 0);
    }
    static size_t lds_bytes(int topk) {                   // merge area: one tile of every wavefront at a time
        return merge_at(topk) + (kSplit > 1 ? (size_t)4 * 64 * (8 * sizeof(float4) + sizeof(float2)) : 0);
    }
};

// kDirect (short prompts, one tile per workgroup): no packed copy, hence one launch and its round trip to memory less.  Whole
// rows come from the cache and take their operand form by way of 8 KiB of LDS per wavefront, V by the transposing load.
// (Rows fetched as the operand wants them, 16 x 64 bytes per load, were slower from 256 tokens on: half lines.  Two tiles
// spill with their queries in registers and lose more to LDS than the launch costs without: 2048 tokens, G = 4 19.1 / 21.6 us.)
template <int kG, int kTiles, int kSplit, bool kDirect>
__global__ __launch_bounds__(256, (AttnCfg<kG, kTiles, kSplit>::kWavesPerSimd)) void attn_prefill_kernel(Dims dm, Tensor q, Tensor k, Tensor v,
                                                            const uint4 *__restrict__ kvp, int32_t nb_cap,
                                                            const int32_t *__restrict__ seqlens,
                                                            const int32_t *__restrict__ block_idx,
                                                            Tensor out, float *__restrict__ lse) {
    using C = AttnCfg<kG, kTiles, kSplit>;
    constexpr int kNU = 4, kTPT = C::kTokPerTile, kTok = C::kTok;
    static_assert(64 % kTok == 0 && kTok <= 32, "one own block per wavefront; member bits in one word");
    extern __shared__ __align__(16) unsigned char attn_smem[];
    arguments_arrive(dm.Hkv, dm.topk, dm.max_seqlen, seqlens, block_idx, kvp, nb_cap, q.ptr, q.sb, q.sh, q.st, dm.scale_log2);
    // grid (8 XCDs x slots, key-value heads, sequences); see launch_attn_variant
    const int xcd = blockIdx.x & 7, sl = blockIdx.x >> 3, h = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Tiles are dealt last first, counted from the sequence's end.  Direct fetches, which are for short buffers, count them from the
    // capacity: their rows of block lists are asked for before the length has arrived (100 tokens 5.9 -> 5.4 us, 250 10.5 -> 9.9).  In
    // longer ones the workgroups of the tiles behind the sequence would all start, and wait for both, before the first real one:
    // 777 tokens in a buffer of 131072, G = 8, 33 us, counted from the capacity 57; in one of their own length, G = 16, 21.6 and 21.5.
    int32_t L = uniform_load(seqlens + b);
    const __bf16 *q_head = q.ptr + (b * q.sb + (int64_t)(h * kG) * q.sh);     // (while the length is on its way)
    if (!kDirect) L = L < 0 ? 0 : (L > dm.max_seqlen ? dm.max_seqlen : L);
    const int last = kDirect ? dm.max_seqlen : L;
    const int tile = (last + C::kTokPerWg - 1) / C::kTokPerWg - 1 - (((sl / kRun) * 8 + xcd) * kRun + sl % kRun);
    const int t0 = kSplit > 1 ? tile * kTok : (tile * 4 + wave) * kTok;   // this wavefront's first token
    if (tile < 0) return;
    const int32_t *idx_rows = block_idx + (((int64_t)b * dm.Hkv + h) * dm.max_seqlen + t0) * dm.topk;
    const UnionRows<kTok> idx_head(idx_rows, kSplit == 1 || wave == 0 ? min(kTok, last - t0) * dm.topk : 0, lane);
    if (kDirect) {
        __builtin_amdgcn_sched_barrier(0);
        L = L < 0 ? 0 : (L > dm.max_seqlen ? dm.max_seqlen : L);
    }
    if (kDirect && dm.fill)                              // rows past the end
        for (int i = threadIdx.x; i < kTok * kG * 16; i += 256) {
            const int tok = t0 + i / (kG * 16), hq = h * kG + i / 16 % kG;
            if (tok >= L && tok < dm.max_seqlen) {
                *reinterpret_cast<uint4 *>(out.ptr + b * out.sb + (int64_t)tok * out.st + (int64_t)hq * out.sh + 8 * (i & 15)) =
                    uint4{0u, 0u, 0u, 0u};
                if ((i & 15) == 0) lse[((int64_t)b * dm.max_seqlen + tok) * dm.Hq + hq] = 0.f;
            }
        }
    if (t0 >= L) return;                                 // (uniform over the workgroup when it splits the blocks)
    const int b_own = t0 / kBlock;                       // kTok divides 64: one own block per wavefront
    const int n = lane & 15, g = lane >> 4;              // MFMA column (token, query head) and 16-lane group
    const int tn = n / kG;                               // token of the column inside its tile
    const float c = dm.scale_log2;

    // The queries are asked for before the union is built, and go to LDS behind it.  (Columns of tokens past the end repeat the last one's and are
    // not written.)
    bf16x8 qf[C::kQLds ? 1 : kTiles][4];
    bf16x8 *ql = reinterpret_cast<bf16x8 *>(attn_smem + C::queries_at(dm.topk)) +                // [tile][ks][lane]
                 (kSplit > 1 ? 0 : wave * kTiles * 4 * 64) + lane;
    constexpr int kLoad = C::kQLds && kSplit > 1 ? 1 : kTiles;           // the waves that share their tokens load a tile each
    bf16x8 qx[kLoad][4];
    f32x4 o[kTiles][8];
    float neg_m[kTiles], l_run[kTiles];
#pragma unroll
    for (int i = 0; i < kLoad; ++i) {
        const int u = kLoad < kTiles ? min(wave, kTiles - 1) : i;
        const __bf16 *qr = q_head + ((int64_t)min(t0 + u * kTPT + tn, (int)L - 1) * q.st + (n % kG) * q.sh + 8 * g);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) qx[i][ks] = load8(qr + 32 * ks);
    }
    const UnionLds ul(attn_smem + (kSplit > 1 ? 0 : wave * UnionLds::bytes(kTok, dm.topk)));
    int cnt = 0;
    if (kSplit == 1 || wave == 0)
        cnt = build_union<kTok>(idx_head, idx_rows, dm.topk, min(kTok, (int)L - t0), b_own, ul, lane);
#pragma unroll
    for (int i = 0; i < kLoad; ++i)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if constexpr (!C::kQLds) qf[i][ks] = qx[i][ks];
            else if constexpr (kLoad == kTiles) ql[(i * 4 + ks) * 64] = qx[i][ks];
            else if (wave < kTiles) ql[(wave * 4 + ks) * 64] = qx[i][ks];
        }
    if constexpr (kSplit > 1) {
        __shared__ int cnt_s;
        if (threadIdx.x == 0) cnt_s = cnt;
        __syncthreads();
        cnt = __builtin_amdgcn_readfirstlane(cnt_s);
    }
    // (32 compute units per XCD, four wavefronts per workgroup; direct fetches are for short prompts)
    const int start = kDirect ? 0 : walk_start(cnt, tile, 32 * C::kWavesPerSimd, b_own);
    auto union_entry = [&](int i) __attribute__((always_inline)) {
        const int at = min(i, cnt - 1) + start;
        return ul.list[!kDirect && at >= cnt ? at - cnt : at];
    };

    // A block's address is uniform: fragments come by buffer loads (scalar base and offset, one vector register of lane
    // offsets), so that fetching them costs no vector instructions.
    const char *kv_head = reinterpret_cast<const char *>(kvp) + ((int64_t)b * dm.Hkv + h) * nb_cap * (kPackedBlockU4 * 16);
    const uint32_t lane16 = 16u * lane;
    u32x4 ring[kNU][4];
    // kDirect: 32-bit offsets from the head's first row; rows past the sequence's last one lie outside the resource and read 0
    const uint32_t kst = 2u * (uint32_t)k.st, vst = 2u * (uint32_t)v.st, last_row = (uint32_t)L - 1u;
    const __amdgpu_buffer_rsrc_t k_rows = __builtin_amdgcn_make_buffer_rsrc(k.ptr + b * k.sb + h * k.sh, 0, last_row * kst + 256u, 0x00027000);
    const __amdgpu_buffer_rsrc_t v_rows = __builtin_amdgcn_make_buffer_rsrc(v.ptr + b * v.sb + h * v.sh, 0, last_row * vst + 256u, 0x00027000);
    auto block_rsrc = [&](uint32_t blk) __attribute__((always_inline)) {
        if constexpr (kDirect) {
            return (uint32_t)__builtin_amdgcn_readfirstlane(blk) * kBlock;           // the block's first row
        } else {
            const int64_t at = (int64_t)(int)__builtin_amdgcn_readfirstlane(blk) * (kPackedBlockU4 * 16);
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(kv_head) + at, 0, kPackedBlockU4 * 16, 0x00027000);
        }
    };
    auto fragment = [&](__amdgpu_buffer_rsrc_t bp, int f) __attribute__((always_inline)) {
        return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(bp, lane16, f * 1024, 0));
    };
    auto issue = [&](int unit, auto bp) __attribute__((always_inline)) {
        const int hs = unit >> 2, r = unit & 3;
        if constexpr (kDirect) {                         // units of a half: K rows of key tiles 2hs, 2hs + 1, V rows of the same
            const uint32_t st = r < 2 ? kst : vst, row = bp + 16u * (2 * hs + (r & 1)) + (uint32_t)g;
            const uint32_t at = __umul24(row, st) + 16u * n;
#pragma unroll
            for (int i = 0; i < 4; ++i)                  // (whole rows: 4i + g)
                ring[unit % kNU][i] =
                    __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r < 2 ? k_rows : v_rows, at + 4u * i * st, 0, 0));
        } else if (r < 2) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) ring[unit % kNU][ks] = fragment(bp, ks * 4 + 2 * hs + r);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                ring[unit % kNU][i] = fragment(bp, kFragsPerOperand + (4 * (r - 2) + i) * 2 + hs);
        }
    };

    // softmax of one tile on 32 keys: pf = P^T in bf16; re-bases the reference when needed.  `member`: this column's
    // token selected the block (always true for one token per tile)
    auto softmax = [&](f32x4 (&s)[2], int u, bool member, bool first, bf16x8 &pf) __attribute__((always_inline)) {
        if (first) {                                      // the tile's one token meets its first block: its reference
            float tmax = fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3]));
#pragma unroll
            for (int j = 0; j < 4; ++j) tmax = fmaxf(tmax, s[1][j]);
            tmax = xgroup_max(tmax) * c;
            if (tmax > -INFINITY) neg_m[u] = -tmax;
        }
        float ps = half_probs(s, c, member ? neg_m[u] : -INFINITY, pf);
        if (__any(!(ps <= kPsumLimit))) {                 // rare: too large, inf, or NaN (no reference yet)
            float tmax = -INFINITY;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) tmax = fmaxf(tmax, s[t][j]);
            tmax = member ? xgroup_max(tmax) * c : -INFINITY;   // per column, same in the four lane groups
            const float old = neg_m[u];                   // NaN = no reference yet
            const float m_new = (old != old) ? tmax : fmaxf(-old, tmax);
            if (m_new > -INFINITY) {
                const float f = (old != old) ? 0.f : fast_exp2(-old - m_new);
                l_run[u] *= f;
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) o[u][dt] *= f;
                neg_m[u] = -m_new;
                ps = half_probs(s, c, member ? -m_new : -INFINITY, pf);
            } else {                                      // every key of this column masked so far
                ps = 0.f;
                pf = zero8();
            }
        }
        l_run[u] += ps;
    };

    // kDirect: the rows of a half (K, then V) in LDS, this wavefront's own piece of the merge area
    char *xt = reinterpret_cast<char *>(attn_smem + C::merge_at(dm.topk)) + wave * (8 * 64 * sizeof(float4));

    // One walk; if a result is not finite (see not_finite), another for each token of a tile.  (A wavefront that works alone
    // has one token per tile.)
    static_assert(!kDirect || (kSplit > 1 && !C::kQLds), "one copy of the tokens, queries in registers");
    static_assert(kSplit > 1 || kTPT == 1, "the flag of the workgroup's waves is exchanged in the merge");
    __shared__ int odd_s[4];
    for (int pass = 0;; ++pass) {
    const uint32_t slot_mask = pass ? 1u << (pass - 1) : (1u << kTPT) - 1u;
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) o[u][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        neg_m[u] = __builtin_nanf("");
        l_run[u] = 0.f;
    }
    // Everything loaded so far (queries, block lists) has to land before the ring starts: the
    // compiler's wait-count bookkeeping otherwise merges those pending loads into the loop and
    // waits for ALL outstanding loads at the top of every iteration, which defeats the ring.
    __builtin_amdgcn_s_waitcnt(0);
    constexpr int kStep = kSplit;                        // the waves of a splitting workgroup take every kSplit-th block
    const int first = kSplit > 1 ? wave : 0;
    uint32_t seen = 0u;                                  // tokens that have met a block
    uint2 e_cur = {0u, 0u}, e_nxt = {0u, 0u};
    if (first < cnt) {
        e_cur = union_entry(first);
        e_nxt = union_entry(first + kStep);
        const auto bp = block_rsrc(e_cur.x);
#pragma unroll
        for (int unit = 0; unit < kNU; ++unit) issue(unit, bp);
    }
    for (int ci = first; ci < cnt; ci += kStep) {
        const int blk = __builtin_amdgcn_readfirstlane(e_cur.x);
        const uint32_t bits = __builtin_amdgcn_readfirstlane(e_cur.y);
        const auto bp = block_rsrc(e_cur.x), bn = block_rsrc(e_nxt.x);
        e_cur = e_nxt;
        e_nxt = union_entry(ci + 2 * kStep);
        const int key0 = blk * kBlock;
        // kDirect: where the lane's piece of row 16t + 4i + g goes (^ (i << 4), + 1024 i), where its piece of the K operand lies
        // (^ (ks << 6)), and where its four V rows for the transposing load begin (keys 16t + 4g .. +3, channels 16dt ..: ^ (dt << 5));
        // formed anew per block: kept, their variants are spilled, and a spill in this loop waits for every load
        uint32_t ln = lane;
        if constexpr (kDirect) asm volatile("" : "+v"(ln));
        const uint32_t xn = ln & 15, xg = ln >> 4, xt_row = 4u * xg + (xn >> 2);
        const uint32_t xt_put = xg * 256u + ((xn ^ (xg << 2)) << 4);
        const uint32_t xt_k = xn * 256u + ((xg ^ (uint32_t)row_swizzle((int)xn)) << 4);
        const uint32_t xt_v = xt_row * 256u + ((((xn & 3) >> 1) ^ (uint32_t)row_swizzle((int)xt_row)) << 4) + 8u * (xn & 1);
        const bool edge = blk == b_own;                  // the last, partial block of a sequence is its last tokens' own
        const uint32_t fresh = bits & ~seen;             // tokens whose first block this is
        seen |= bits;
        uint32_t tb[kTiles];                             // member bits of the tile's tokens
#pragma unroll
        for (int u = 0; u < kTiles; ++u) tb[u] = (bits >> (u * kTPT)) & slot_mask;
#pragma unroll
        for (int hs = 0; hs < 2; ++hs) {
            // ---- S^T = K . Q^T for 32 keys, one key tile per unit ------------------------------
            auto refill = [&](int unit) __attribute__((always_inline)) {
                if (unit + kNU < 8) issue(unit + kNU, bp);
                else issue(unit + kNU - 8, bn);      // (a harmless re-read of this block at the tail)
            };
            auto scores = [&](int r, const bf16x8 (&qu)[4]) __attribute__((always_inline)) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc = mfma16(__builtin_bit_cast(bf16x8, ring[(4 * hs + r) % kNU][ks]), qu[ks], acc);
                return acc;
            };
            f32x4 s[kTiles][2];
            auto keep = [&](int unit) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *reinterpret_cast<u32x4 *>(xt + (xt_put ^ (uint32_t)(i << 4)) + i * 1024 + (unit & 1) * 4096) = ring[unit % kNU][i];
                refill(unit);
            };
            if constexpr (kDirect) {
                keep(4 * hs);
                keep(4 * hs + 1);
#pragma unroll
                for (int u = 0; u < kTiles; ++u) {
                    if (!tb[u]) continue;
                    s[u][0] = s[u][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                        for (int r = 0; r < 2; ++r)
                            s[u][r] = mfma16(__builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(xt + (xt_k ^ (uint32_t)(ks << 6)) + r * 4096)),
                                             qf[u][ks], s[u][r]);
                }
            } else if constexpr (!C::kQLds) {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
#pragma unroll
                    for (int u = 0; u < kTiles; ++u)
                        if (tb[u]) s[u][r] = scores(r, qf[u]);
                    refill(4 * hs + r);
                }
            }
            // ---- probabilities, P^T packed to bf16 in MFMA B layout ---------------------------
            bf16x8 pf[kTiles];
#pragma unroll
            for (int u = 0; u < kTiles; ++u) {
                if (!tb[u]) continue;
                if constexpr (C::kQLds) {                // a tile at a time: its queries come from LDS once per half
                    bf16x8 qu[4];
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) qu[ks] = ql[(u * 4 + ks) * 64];
#pragma unroll
                    for (int r = 0; r < 2; ++r) s[u][r] = scores(r, qu);
                }
                if (edge) {
                    const int tok = t0 + u * kTPT + tn;
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (key0 + 32 * hs + 16 * t + 4 * g + j > tok) s[u][t][j] = -INFINITY;
                }
                softmax(s[u], u, kTPT == 1 || ((tb[u] >> tn) & 1u), kTPT == 1 && hs == 0 && (fresh >> u & 1u), pf[u]);
            }
            if constexpr (C::kQLds) {
#pragma unroll
                for (int r = 0; r < 2; ++r) refill(4 * hs + r);
            }
            // ---- O^T += V^T . P^T, four channel tiles per unit --------------------------------
            if constexpr (kDirect) {
                keep(4 * hs + 2);
                keep(4 * hs + 3);
#pragma unroll
                for (int d4 = 0; d4 < 8; d4 += 4) {
                    bf16x8 vf[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t at = xt_v ^ (uint32_t)((d4 + i) << 5);
                        const s16x4 x0 = lds_read_tr16(xt + at), x1 = lds_read_tr16(xt + at + 4096);
                        vf[i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
                    }
#pragma unroll
                    for (int u = 0; u < kTiles; ++u) {
                        if (!tb[u]) continue;
#pragma unroll
                        for (int i = 0; i < 4; ++i) o[u][d4 + i] = mfma16(vf[i], pf[u], o[u][d4 + i]);
                    }
                }
            } else
#pragma unroll
            for (int r = 2; r < 4; ++r) {
                const int unit = 4 * hs + r, dh = r - 2;
#pragma unroll
                for (int u = 0; u < kTiles; ++u) {
                    if (!tb[u]) continue;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        o[u][4 * dh + i] =
                            mfma16(__builtin_bit_cast(bf16x8, ring[unit % kNU][i]), pf[u], o[u][4 * dh + i]);
                }
                refill(unit);
            }
        }
    }

    if constexpr (kSplit > 1) {
        // ---- merge the four waves, a tile at a time: every wave leaves (o, reference, sum) of its blocks in LDS, then
        // wave w combines channel tiles 2w, 2w+1 of every column --------------------------------------------------
        float4 *po = reinterpret_cast<float4 *>(attn_smem + C::merge_at(dm.topk));   // [wave][dt][lane]
        float2 *pm = reinterpret_cast<float2 *>(po + 4 * 8 * 64);                    // [wave][lane]
        int ln = lane;
        asm volatile("" : "+v"(ln));                      // (what follows is not formed ahead of the walk: no register to spare there)
        const int lane = ln, n = ln & 15, g = ln >> 4, tn = n / kG;
        const bool writes = pass == 0 || tn == pass - 1;
        bool odd = false;
#pragma unroll
        for (int u = 0; u < kTiles; ++u) {
            if (u) __syncthreads();
#pragma unroll
            for (int dt = 0; dt < 8; ++dt)
                po[(wave * 8 + dt) * 64 + lane] = float4{o[u][dt][0], o[u][dt][1], o[u][dt][2], o[u][dt][3]};
            pm[wave * 64 + lane] = float2{(neg_m[u] != neg_m[u]) ? -INFINITY : -neg_m[u], xgroup_sum(l_run[u])};
            __syncthreads();
            const int tok = t0 + u * kTPT + tn;
            float2 m4[4];
            float M = -INFINITY, l_tot = 0.f, f[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                m4[w] = pm[w * 64 + lane];
                M = fmaxf(M, m4[w].x);
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                f[w] = m4[w].x > -INFINITY ? fast_exp2(m4[w].x - M) : 0.f;
                l_tot += f[w] * m4[w].y;
            }
            if (tok < L && writes) {
                const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
                __bf16 *op = out.ptr + b * out.sb + (int64_t)tok * out.st + (int64_t)(h * kG + n % kG) * out.sh + 4 * g;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int dt = 2 * wave + i;
                    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const float4 y = po[(w * 8 + dt) * 64 + lane];
                        x += f32x4{y.x, y.y, y.z, y.w} * f[w];
                    }
                    if (kTPT > 1) odd |= not_finite(x);
                    bf16x4 r;
#pragma unroll
                    for (int j = 0; j < 4; ++j) r[j] = (__bf16)(x[j] * inv);
                    *reinterpret_cast<uint2 *>(op + 16 * dt) = __builtin_bit_cast(uint2, r);
                }
                if (g == 0 && wave == 0)
                    lse[((int64_t)b * dm.max_seqlen + tok) * dm.Hq + h * kG + n % kG] =
                        l_tot > 0.f ? lse_of(M, l_tot) : -INFINITY;
            }
        }
        if (kTPT == 1 || pass == kTPT) return;
        if (pass == 0) {
            const bool again = __any(odd);
            if (lane == 0) odd_s[wave] = again;
        }
        __syncthreads();                                  // (also: everyone is past the merge area)
        if (!(odd_s[0] | odd_s[1] | odd_s[2] | odd_s[3])) return;
        continue;
    }
    // ---- normalise and write: lane holds channels 16*dt + 4*g .. +3 of column n -----------------
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
        const int tok = t0 + u * kTPT + tn;
        if (tok >= L) continue;
        const float l_tot = xgroup_sum(l_run[u]);
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        __bf16 *op = out.ptr + b * out.sb + (int64_t)tok * out.st + (int64_t)(h * kG + n % kG) * out.sh + 4 * g;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
            bf16x4 r;
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = (__bf16)(o[u][dt][j] * inv);
            *reinterpret_cast<uint2 *>(op + 16 * dt) = __builtin_bit_cast(uint2, r);
        }
        if (g == 0)
            lse[((int64_t)b * dm.max_seqlen + tok) * dm.Hq + h * kG + n % kG] =
                l_tot > 0.f ? lse_of(-neg_m[u], l_tot) : -INFINITY;
    }
    return;
    }
}

// ---- attention with one block set per query block (comparison variant) ------------------------------------
// Not the report's method (section 2.1.3: token-level queries); it shows what the same arithmetic
// reaches when the 64 tokens of a query block attend one common block list.  A workgroup takes 8
// consecutive tokens of a query block (a wavefront 2, as above) and walks the shared list in step:
// every packed block is fetched once per workgroup -- each thread carries 1/256 of the next block in
// registers while the current one is consumed -- and all four wavefronts read their operand
// fragments from LDS, which delivers several times what the L2 path does.  Only the query block's
// own key-value block needs the causal mask.
constexpr int kShTok = 2;                                // tokens per wavefront
__global__ __launch_bounds__(256, 2) void attn_prefill_shared_kernel(Dims dm, Tensor q, const uint4 *__restrict__ kvp,
                                                                      int32_t nb_cap, const int32_t *__restrict__ seqlens,
                                                                      const int32_t *__restrict__ block_idx,
                                                                      Tensor out, float *__restrict__ lse,
                                                                      int32_t n_tiles) {
    __shared__ __align__(16) u32x4 stage[2][kPackedBlockU4];
    const uint32_t vid = xcd_contiguous_id(blockIdx.x, gridDim.x);
    const int tile = vid % n_tiles;                      // 8 tokens
    const int h = (vid / n_tiles) % dm.Hkv;
    const int b = vid / (n_tiles * dm.Hkv);
    int32_t L = seqlens[b];
    L = L < 0 ? 0 : (L > dm.max_seqlen ? dm.max_seqlen : L);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tile * 8 >= L) return;                           // uniform over the workgroup
    const int t0 = tile * 8 + wave * kShTok;             // this wavefront's first token (may lie past the end)
    const int I = (tile * 8) / kBlock;                   // the query block, and its own key-value block
    const int n_qb = (dm.max_seqlen + kBlock - 1) / kBlock;
    const int n = lane & 15, g = lane >> 4;
    const int G = dm.G;
    const float c = dm.scale_log2;

    // the shared list, compacted: entries < 0 or above the own block are dropped (each wavefront keeps its own copy)
    __shared__ int blist[4][64];
    int entry = kNone;
    if (lane < dm.topk) {
        const int x = block_idx[(((int64_t)b * dm.Hkv + h) * n_qb + I) * dm.topk + lane];
        if (x >= 0 && x <= I) entry = x;
    }
    const uint64_t have = __ballot(entry != kNone);
    const int cnt = __popcll(have);
    if (entry != kNone) blist[wave][__popcll(have & ((1ull << lane) - 1ull))] = entry;   // same wavefront reads it back
    bf16x8 qf[kShTok][4];
    f32x4 o[kShTok][8];
    float neg_m[kShTok], l_run[kShTok];
#pragma unroll
    for (int u = 0; u < kShTok; ++u) {
        const int tok = min(t0 + u, L - 1);              // rows past the end compute on a copy and are not written
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            qf[u][ks] = load8(q.ptr + b * q.sb + (int64_t)tok * q.st + (int64_t)(h * G + min(n, G - 1)) * q.sh + 32 * ks + 8 * g);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) o[u][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        neg_m[u] = __builtin_nanf("");
        l_run[u] = 0.f;
    }
    auto softmax = [&](f32x4 (&s)[2], int u, bf16x8 &pf) __attribute__((always_inline)) {
        float ps = half_probs(s, c, neg_m[u], pf);
        if (__any(!(ps <= kPsumLimit))) {                 // rare: too large, inf, or NaN (no reference yet)
            float tmax = -INFINITY;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) tmax = fmaxf(tmax, s[t][j]);
            tmax = xgroup_max(tmax) * c;
            const float old = neg_m[u];
            const float m_new = (old != old) ? tmax : fmaxf(-old, tmax);
            if (m_new > -INFINITY) {
                const float f = (old != old) ? 0.f : fast_exp2(-old - m_new);
                l_run[u] *= f;
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) o[u][dt] *= f;
                neg_m[u] = -m_new;
                ps = half_probs(s, c, -m_new, pf);
            } else {
                ps = 0.f;
                pf = zero8();
            }
        }
        l_run[u] += ps;
    };

    const u32x4 *kv_head = reinterpret_cast<const u32x4 *>(kvp) + ((int64_t)b * dm.Hkv + h) * nb_cap * kPackedBlockU4;
    u32x4 r[8];                                          // this thread's 1/256 of a packed block
    auto fetch = [&](int ci) __attribute__((always_inline)) {
        const int blk = blist[wave][min(ci, cnt - 1)];
        const u32x4 *bp = kv_head + (int64_t)blk * kPackedBlockU4 + tid;
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = bp[256 * i];
    };
    auto stash = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) stage[buf][tid + 256 * i] = r[i];
    };
    if (cnt == 0) return;                                // (cannot happen for a live query block: its own block is forced)
    fetch(0);
    stash(0);
    __syncthreads();
    for (int ci = 0; ci < cnt; ++ci) {
        const int cur = ci & 1;
        fetch(ci + 1);                                   // (a copy of the last block at the end, never used)
        const int blk = blist[wave][ci];
        const int key0 = blk * kBlock;
        const bool edge = blk == I;
        const u32x4 *sb = stage[cur] + lane;
#pragma unroll
        for (int hs = 0; hs < 2; ++hs) {
            // four independent accumulation chains (2 key tiles x 2 tokens) interleaved k-step by k-step: a
            // dependent MFMA then issues three MFMAs after the one it waits for, which covers its latency
            f32x4 s[kShTok][2];
#pragma unroll
            for (int u = 0; u < kShTok; ++u) s[u][0] = s[u][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const u32x4 k0 = sb[(ks * 4 + 2 * hs) * 64], k1 = sb[(ks * 4 + 2 * hs + 1) * 64];
#pragma unroll
                for (int u = 0; u < kShTok; ++u) {
                    s[u][0] = mfma16(__builtin_bit_cast(bf16x8, k0), qf[u][ks], s[u][0]);
                    s[u][1] = mfma16(__builtin_bit_cast(bf16x8, k1), qf[u][ks], s[u][1]);
                }
            }
            bf16x8 pf[kShTok];
#pragma unroll
            for (int u = 0; u < kShTok; ++u) {
                if (edge) {
                    const int tok = t0 + u;
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (key0 + 32 * hs + 16 * t + 4 * g + j > tok) s[u][t][j] = -INFINITY;
                }
                softmax(s[u], u, pf[u]);
            }
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) {
                const u32x4 vf = sb[(kFragsPerOperand + dt * 2 + hs) * 64];
#pragma unroll
                for (int u = 0; u < kShTok; ++u) o[u][dt] = mfma16(__builtin_bit_cast(bf16x8, vf), pf[u], o[u][dt]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        stash(cur ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kShTok; ++u) {
        const int tok = t0 + u;
        if (tok >= L || n >= G) continue;
        const float l_tot = xgroup_sum(l_run[u]);
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        __bf16 *op = out.ptr + b * out.sb + (int64_t)tok * out.st + (int64_t)(h * G + n) * out.sh + 4 * g;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
            bf16x4 rr;
#pragma unroll
            for (int j = 0; j < 4; ++j) rr[j] = (__bf16)(o[u][dt][j] * inv);
            *reinterpret_cast<uint2 *>(op + 16 * dt) = __builtin_bit_cast(uint2, rr);
        }
        if (g == 0)
            lse[((int64_t)b * dm.max_seqlen + tok) * dm.Hq + h * G + n] =
                l_tot > 0.f ? (fast_log2(l_tot) - neg_m[u]) * kLn2 : -INFINITY;
    }
}

size_t attn_prefill_ws_bytes(const Dims &dm) {
    const size_t nb_cap = ((size_t)dm.max_seqlen + kBlock - 1) / kBlock;
    return (size_t)dm.batch * dm.Hkv * nb_cap * kPackedBlockU4 * sizeof(uint4);
}

// Workgroups go to the XCDs round-robin by their id.  A sequence's tiles are dealt to the XCDs in runs of kRun, last
// tile first, counted from the sequence's own length: every XCD gets the same share of every sequence (a batch of
// unequal lengths leaves no XCD idle: 12289 + 8693 + 5096 + 1500 tokens 1256 -> 700 us from this alone), neighbours,
// which share blocks, still meet in one L2, and the long rows start first.  (Direct fetches: from the capacity, see the kernel.)

template <int kG, int kTiles, int kSplit, bool kDirect = false>
static int launch_attn_variant(const Dims &dm, Tensor q, Tensor k, Tensor v, const uint4 *kvp, int32_t nb_cap, const int32_t *seqlens,
                               const int32_t *block_idx, Tensor out, float *lse, hipStream_t stream) {
    using C = AttnCfg<kG, kTiles, kSplit>;
    const int32_t n_tiles = (dm.max_seqlen + C::kTokPerWg - 1) / C::kTokPerWg;
    const int32_t slots = (n_tiles + 8 * kRun - 1) / (8 * kRun) * kRun;
    const size_t lds = C::lds_bytes(dm.topk);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)attn_prefill_kernel<kG, kTiles, kSplit, kDirect>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL((attn_prefill_kernel<kG, kTiles, kSplit, kDirect>), dim3(slots * 8, dm.Hkv, dm.batch), dim3(256), lds, stream,
                       dm, q, k, v, kvp, nb_cap, seqlens, block_idx, out, lse);
    return 0;
}

// How many tiles a wavefront takes and whether the waves of a workgroup share their tokens, by how many workgroups the
// call fills (two fit a compute unit, of two tiles at G = 16 three: 512 or 768 fill the chip).  More tiles per wavefront mean fewer bytes per token, since
// a fetched block serves every token that selected it; splitting the blocks over four waves makes four times as many
// waves out of few tokens.  Measured over 150 .. 32768 tokens, 2 key-value heads, top-k 16 (us, start -> now):
//   G = 16: 150 17 -> 9, 1500 56 -> 36, 4096 128 -> 97, 32768 1024 -> 775;  G = 4: 777 31 -> 15, 4096 123 -> 57,
//   32768 1148 -> 755;  G = 1: 777 31 -> 12, 4096 124 -> 38, 32768 1339 -> 534
// The lines: four tiles, split, from 512 workgroups on (at 390 .. 750 it met two tiles for every G; with three workgroups of two tiles
// on a compute unit, G = 16, two heads, two / four tiles: 1040 tokens 27.1 / 27.7, 1280 34.4 / 29.8, 1500 42.4 / 35.5; one head, 2100 31.6 / 30.0); two tiles,
// split, from 192 (at 190 it met one tile, with packed blocks), against direct fetches, which save the packing, from 320 for G >= 8 (one tile direct /
// two tiles packed, both launches, 2 heads: G = 16, 220 tokens 7.6 / 9.3, 300 10.1 / 11.0, 400 13.2 / 12.9; G = 8, 400 10.3 / 11.0, 550
// 12.5 / 12.8, 700 14.5 / 13.9; smaller groups meet at 192: G = 4, 777 13.5 / 13.5); four tiles on every wave by itself (no merge, no idle wave at the end of a list)
// only for G = 16 from 1024 workgroups on (smaller groups have longer unions, where the split's balance wins).
constexpr int kDirectTokens = 896;                       // (see attn_direct; the tiles do not depend on the strides, on which direct fetches do)
static int64_t two_tile_rows(const Dims &dm) { return (int64_t)(dm.max_seqlen <= kDirectTokens && dm.G >= 8 ? 320 : 192) * 2 * (16 / dm.G); }
template <int kG>
static int launch_attn_group(const Dims &dm, Tensor q, Tensor k, Tensor v, bool direct, const uint4 *kvp, int32_t nb_cap, const int32_t *seqlens,
                             const int32_t *block_idx, Tensor out, float *lse, hipStream_t stream) {
    const int64_t rows = (int64_t)dm.batch * dm.max_seqlen * dm.Hkv;
    constexpr int kTPT = 16 / kG;
    if constexpr (kG == 16)
        if (rows >= (int64_t)1024 * 16) return launch_attn_variant<16, 4, 1>(dm, q, k, v, kvp, nb_cap, seqlens, block_idx, out, lse, stream);
    if constexpr (kG > 1)                                // (member bits of at most 32 tokens)
        if (rows >= (int64_t)512 * 4 * kTPT) return launch_attn_variant<kG, 4, 4>(dm, q, k, v, kvp, nb_cap, seqlens, block_idx, out, lse, stream);
    if (rows >= two_tile_rows(dm)) return launch_attn_variant<kG, 2, 4>(dm, q, k, v, kvp, nb_cap, seqlens, block_idx, out, lse, stream);
    return direct ? launch_attn_variant<kG, 1, 4, true>(dm, q, k, v, kvp, nb_cap, seqlens, block_idx, out, lse, stream)
                  : launch_attn_variant<kG, 1, 4>(dm, q, k, v, kvp, nb_cap, seqlens, block_idx, out, lse, stream);
}

// Straight from the cache instead of from a packed copy: where a workgroup has one tile (see launch_attn_group) and the sequences are
// short.  Attention call, packed / direct, us, 2 key-value heads: 100 tokens 7.6 / 5.6 (every G); 256 tokens G = 16 10.3 / 8.0,
// G = 4 8.1 / 6.2; 750 tokens G = 4 13.7 / 12.5, G = 1 11.1 / 10.3; they meet at about 1000 (1 head, G = 4: 11.8 / 12.1; G = 1: 12.6 / 12.2)
// and at 2000 tokens G = 1 takes 18.9 / 20.0.  Offsets are 32-bit and formed by a 24-bit product, and rows must not overlap
// (those past the end are told by their offset).
static bool attn_direct(const Dims &dm, const Tensor &k, const Tensor &v) {
    if (dm.shared_q || dm.max_seqlen > kDirectTokens || (int64_t)dm.batch * dm.max_seqlen * dm.Hkv >= two_tile_rows(dm)) return false;
    const int64_t lo = k.st < v.st ? k.st : v.st, hi = k.st < v.st ? v.st : k.st;
    return lo >= kHeadDim && hi < 1 << 19;
}

int launch_attn_prefill(const Dims &dm, Tensor q, Tensor k, Tensor v, const int32_t *seqlens,
                        const int32_t *block_idx, Tensor out, float *lse, void *ws, hipStream_t stream) {
    const int32_t nb_cap = (dm.max_seqlen + kBlock - 1) / kBlock;
    if (nb_cap <= 0 || dm.batch <= 0) return 0;
    uint4 *kvp = reinterpret_cast<uint4 *>(ws);
    const bool direct = attn_direct(dm, k, v);
    if (!direct) {
        timing_begin("pack_kv_kernel", stream);
        hipLaunchKernelGGL(pack_kv_kernel, dim3(nb_cap, dm.Hkv, dm.batch), dim3(256), 0, stream, dm, k, v,
                           seqlens, kvp, nb_cap, out, lse);
        timing_end(stream);
    }
    if (dm.shared_q) {                                   // one block list per query block (comparison variant)
        const int32_t n_tiles = (dm.max_seqlen + 7) / 8;
        timing_begin("attn_prefill_shared_kernel", stream);
        hipLaunchKernelGGL(attn_prefill_shared_kernel, dim3((uint32_t)((int64_t)n_tiles * dm.Hkv * dm.batch)), dim3(256),
                           0, stream, dm, q, kvp, nb_cap, seqlens, block_idx, out, lse, n_tiles);
        timing_end(stream);
        return (int)hipGetLastError();
    }
    timing_begin("attn_prefill_kernel", stream);
    int err = (int)hipErrorInvalidValue;
    switch (dm.G) {
        case 1: err = launch_attn_group<1>(dm, q, k, v, direct, kvp, nb_cap, seqlens, block_idx, out, lse, stream); break;
        case 2: err = launch_attn_group<2>(dm, q, k, v, direct, kvp, nb_cap, seqlens, block_idx, out, lse, stream); break;
        case 4: err = launch_attn_group<4>(dm, q, k, v, direct, kvp, nb_cap, seqlens, block_idx, out, lse, stream); break;
        case 8: err = launch_attn_group<8>(dm, q, k, v, direct, kvp, nb_cap, seqlens, block_idx, out, lse, stream); break;
        case 16: err = launch_attn_group<16>(dm, q, k, v, direct, kvp, nb_cap, seqlens, block_idx, out, lse, stream); break;
    }
    if (err) return err;
    timing_end(stream);
    return (int)hipGetLastError();
}

}  // namespace infllmv2
