// Backward of the stage-3 attention (section 2.1: the sparse attention is trainable).  The block
// sets are a discrete choice and the mean-pooled semantic kernels have no parameters, so the
// gradient reaches q, k and v through the attention alone.  With p = exp(z - lse) recomputed from
// the forward's log-sum-exp, D = <dout, out> per (token, head):
//     dv_t += p dout_i        dp = <dout_i, v_t>        ds = p (dp - D)
//     dq_i += scale ds k_t    dk_t += scale ds q_i
//
// Per-token block sets make dq a gather (a token walks its blocks, like the forward) and dk/dv a
// scatter (a block collects from every token that selected it).  The scatter is turned around with
// membership words (word of 32 tokens x block) built from the block lists, so both big kernels accumulate
// in registers:
//   pack_bwd_kernel     fragment-major copies of every block (K rows, V rows), its tokens' membership bits, its cleared sums
//   attn_bwd_dq_kernel  first the members of every block, cut into work items, queued per XCD by the tokens they hold (cut_items); then
//                       workgroup = 1 to 4 MFMA tiles of 16 (token, head) columns, walks the union of the tokens' block lists:
//                       D, then S^T = K.Q^T, dP^T = V.dO^T, dQ^T += K^T.dS^T
//   attn_bwd_dkdv_kernel  workgroup = one item of a block after the other, wavefront = 32 keys x 128 channels:
//                       S = Q.K^T, dP = dO.V^T, dV += P^T.dO, dK += dS^T.Q over steps of 32 (token, head) rows
//                       (32x32x16 MFMAs; q and dout rows copied from memory straight into LDS);
//                       fp32 atomics add up the items of a block
//   bwd_finish_kernel   fp32 accumulators -> bf16 dk (times scale), dv
// As in the forward, every second contraction takes an operand straight from the accumulator
// layout of the first, with the contraction index of the other operand permuted to match.
#include "token_union.h"
#include <type_traits>

namespace infllmv2 {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int kBwdBlockU4 = 2 * 16 * 64;              // uint4 per packed block: K rows, V rows (32 KiB)
// The scatter's work items (see cut_items): a block with some of the tokens of a segment of kSegWords words of 32 tokens.  A
// segment has a window per XCD, a window kSlices slices, the XCD's queue a bin per slice (or run of slices).
constexpr int kSegWords = 256;
constexpr int kQueues = 8;                            // one per XCD
constexpr int kWindowWords = kSegWords / kQueues;
constexpr int kSlices = 8;
constexpr int kBins = 256;                            // at most, of a queue
constexpr int kCounterLine = 32;
constexpr uint32_t kBehind = 1u << 31;                // in a queue's place drawn last: there are items behind the queues

// Members of an item, in steps of 32 (token, head) rows: an equal share of the call for each of the chip's kDkdvGroups workgroups,
// within 12 (G = 16: 8) .. 64; a larger share in equal parts of at most 64 (all in items of 64, most workgroups wait for those that have one
// more: 9000 tokens, G = 4, top-k 48, 300 -> 287 us, 6000, G = 16, 250 -> 236).  Below, the fixed part (32 KiB of K and V, 64 KiB of atomic
// sums) is most of an item (8192 tokens, G = 1: 92 / 72 / 80 us with at least 8 / 16 / 32 steps; 1000 tokens, G = 4 would take
// 31 / 43 / 62); above, the last items keep the others waiting (32K tokens, G = 16: 1190 / 1310 us with at most 64 / 256).  An
// item ends with a whole word of 32 tokens, which may exceed its share by G steps: G = 16, 777 tokens 55 us with at least 12, 51.6 with
// 8.  A share of the capacity instead of the call's tokens leaves most of the chip idle: 777 tokens in a buffer of 2000, top-k 8, 65 us, so
// 52; in one of 4096, top-k 16, 112 and 54.  So does one that takes all sequences for as long as the item's own: with the cutting, G = 8,
// 300 + 100 + 900 + 64 tokens 77 us, so 56; G = 16, 1500 + 200 + 800 129 and 100.  From 96 on a share is rounded up to whole words (see
// cut_items): blocks that every token selects are then cut evenly, G = 8, 5000 + 700 tokens, 136 -> 160 members, 129 -> 111 us,
// 4096 + 3333, 236 -> 256, 168 -> 162.  Smaller ones grow too much by it: 1500 + 200 + 800, 80 -> 96, 100 -> 112.
constexpr int kDkdvGroups = 256 * 4;                  // of one pair of wavefronts; of two pairs, half as many
constexpr int kShareRows = 32 * kDkdvGroups;
constexpr int kMaxMembers = 1024;                     // (an item may exceed its share by a word of 32 but one)
constexpr int kMostSteps = 64;
// A short call, of two pairs and at most one item per workgroup, and few enough bins for one look at all of them (8192 tokens and heads together), has no use for
// the queues: a workgroup finds its item by its own number and ends with it.  (Drawn from the queues, every workgroup asked all eight for
// more, one round trip after another.)  Where items are few, two or four workgroups take a part of an item's steps each; more
// parts than that lose to the sums: the chip adds about 270 words per ns, 61 ns per item or part of one (300 tokens, G = 16, 55 items in 1 / 2 / 3 / 4
// parts 20.2 / 18.4 / 21.0 / 23.5 us; 700, G = 4, 28.2 / 19.1 / 21.5 in 1 / 2 / 3).  dk/dv, 2 heads, top-k 16, one pair each, queues / by number, us:
// G = 16, 150 tokens 39 / 14, 500 45 / 31, 1000 65 / 64; G = 8, 500 41 / 20, 1000 47 / 36; G = 1, 500 29 / 13, 1000 34 / 17, 2000 36 / 25.
constexpr int kPartItems = 128;
// What is left of a call of few steps per workgroup are its sums, all at the same time.  Up to a share of kPairSteps steps an item has two pairs of
// wavefronts, half its steps each, whose sums meet in LDS before they are added to the block's: half the workgroups, items of twice the share and
// half the additions.  One pair / two, both by number where that fits: G = 16, 500 tokens 31 / 25 us, 1000 64 / 50, 2000 101 / 81; G = 8, 500 20 / 18, 1000
// 36 / 31, 2500 76 / 64; G = 4, 5000 95 / 79; G = 1, 12000 108 / 87; 2 x 4096, G = 8 (64 steps) 185 / 180.  Short calls of G = 1 lose a little (300
// tokens 11.2 / 12.9, 800 15.7 / 17.0, 2000 24.6 / 26.4, 4000 35.0 / 35.9); they have two all the same, for the one kernel that finds items by number.
// Beyond, two pairs in step wait for each other: 12000, G = 8 261 / 264, 32K, G = 16 1097 / 1180.
constexpr int kPairSteps = 64;
__host__ __device__ constexpr int least_steps(int G, int pairs) { return (G == 16 ? 8 : 12) * pairs; }
__host__ __device__ inline int members_of(int steps, int G, int pairs = 1) {
    const int m = (steps < least_steps(G, pairs) ? least_steps(G, pairs) : steps) * 32 / G;
    return m > kMaxMembers - 32 ? kMaxMembers - 32 : m;
}
__host__ __device__ inline int share_rounds(int share) { return share > kMostSteps ? (share + kMostSteps - 1) / kMostSteps : 1; }
// steps of a workgroup's share of a call with so many rows (beyond 4096 it is cut into items of kMostSteps either way)
__host__ __device__ inline int share_steps(int64_t rows, int pairs = 1) {
    const int64_t s = (rows * pairs + kShareRows - 1) / kShareRows;
    return (int)(s < 4096 ? s : 4096);
}
// rows of (token, head) per block of 64 tokens
static inline int64_t rows_per_block(const Dims &dm) { return (int64_t)kBlock * dm.Hkv * dm.topk * dm.G; }

// Where items lie and what an item says.  A queue has n bins of `cap` places, the last bin of a window `tail` more; what finds its bin
// full goes to one list behind the queues, taken when they are empty, which has room for every item of the call.  Counters, of a
// queue and then of that list: the bins' lengths, then, on a line of its own, the place drawn last; on the list's also the call's
// blocks, in four words to be added.  (That the list has items is told with the places: every workgroup's look at its length is one
// address for the chip, 3.5 of 35 us for 500 tokens.)
struct BwdBins {
    int32_t n, shift;                                 // bins of a queue; slices of a bin (log2)
    int32_t cap, tail, window;                        // a window's bins (log2)
    int32_t size, stride;                             // places, counters of a queue
    int32_t block_bits;
    __host__ __device__ int64_t begin(int queue, int bin) const {
        return (int64_t)queue * size + (int64_t)bin * cap + (int64_t)(bin >> window) * tail;
    }
    __device__ uint32_t places(int bin) const { return (uint32_t)(cap + ((bin + 1) & ((1 << window) - 1) ? 0 : tail)); }
    // {sequence and head, block, first word, words - 1}.  It fits: the membership words, two per block and block, are in memory.
    __device__ uint64_t item(int64_t bh, int j, int w, int n_words) const {
        return ((((uint64_t)bh << block_bits | (uint32_t)j) << (block_bits + 1) | (uint32_t)w) << 8) | (uint32_t)(n_words - 1);
    }                                                 // (a segment's first word is a multiple of 256: the words' bits are the low 16)
    __device__ uint4 unpack(uint64_t x) const {
        const uint64_t w = x >> 8, j = w >> (block_bits + 1);
        return uint4{(uint32_t)(j >> block_bits), (uint32_t)j & ((1u << block_bits) - 1u), (uint32_t)w & ((2u << block_bits) - 1u),
                     (uint32_t)(x & 255u) + 1u};
    }
};
struct BwdLayout {
    int32_t nb_cap, words, n_seg;                     // per sequence: blocks, words of 32 tokens, segments of kSegWords words
    int32_t members;                                  // of an item, about: what the bins are laid out for
    int32_t pairs;                                    // of wavefronts to an item of dk and dv
    BwdBins bins;
    size_t kvb, rowc, bits, acc_dk, acc_dv, counters, items, total; // byte offsets into the workspace
};
static inline size_t al256(size_t x) { return (x + 255) / 256 * 256; }
static BwdLayout bwd_layout(const Dims &dm) {
    BwdLayout l;
    const size_t T = (size_t)dm.max_seqlen, BH = (size_t)dm.batch * dm.Hkv;
    l.nb_cap = (dm.max_seqlen + kBlock - 1) / kBlock;
    l.words = 2 * l.nb_cap;
    l.n_seg = (l.words + kSegWords - 1) / kSegWords;
    const int64_t rows = dm.batch * (int64_t)l.nb_cap * rows_per_block(dm);
    l.pairs = rows <= (int64_t)kPairSteps * kShareRows ? 2 : 1;
    l.members = members_of((int)(rows / kShareRows < kMostSteps ? rows / kShareRows : kMostSteps), dm.G);
    const size_t nb = (size_t)l.nb_cap, words = (size_t)l.words, windows = BH * ((words + kWindowWords - 1) / kWindowWords);
    const size_t slots = windows ? (windows + kQueues - 1) / kQueues : 1;       // windows of a queue
    BwdBins &t = l.bins;
    t.shift = 0;
    while ((slots * kSlices + ((size_t)1 << t.shift) - 1) >> t.shift > (size_t)kBins) ++t.shift;
    t.n = (int32_t)((slots * kSlices + ((size_t)1 << t.shift) - 1) >> t.shift);
    t.stride = (t.n + kCounterLine - 1) / kCounterLine * kCounterLine + kCounterLine;
    t.block_bits = 1;
    while (nb >> t.block_bits) ++t.block_bits;
    // Items that end in a slice: at most one per `members` list entries (a smaller call has smaller items, not more of them), one more per block with an entry (begun before) and the
    // own tokens' of its blocks.  That every block's ends there is provided for in the list behind; a bin has room for twice the mean
    // and, blocks that are equally popular being cut at about the same tokens, a sixteenth of the blocks.  (Bins for the worst case
    // took 4.9 MB for 32K tokens x 2 heads, top-k 16, and 76 MB for 128K; these 0.4 and 3.0.)  A bin of several
    // slices has several slices' places, so that a call of fewer or shorter sequences never asks for more than a larger one.
    const size_t slice_words = kWindowWords / kSlices, rw = slice_words < words ? slice_words : words;
    const size_t topk = (size_t)dm.topk < nb ? (size_t)dm.topk : nb;            // (a block that a row lists twice counts once)
    const size_t ent = rw * 32 * topk, most = (ent < nb ? ent : nb) + ent / l.members + rw / 2;
    const size_t sparse = 64 * topk < nb ? 64 * topk : nb;
    size_t cap = 2 * ent / l.members + rw / 2 + sparse / 16;
    cap = cap < most ? cap : most;
    // what is left of the blocks at the segments' ends: to the last slices of all windows alike
    const size_t seg_ent = (words < (size_t)kSegWords ? words : (size_t)kSegWords) * 32 * topk;
    const size_t tails = BH * l.n_seg * (seg_ent < nb ? seg_ent : nb), tail = (tails + slots * kQueues - 1) / (slots * kQueues);
    // The most items that a call of up to so many rows has where `members` are full, all sequences together (one of them may have more than its
    // part): a share's parts make kDkdvGroups x rounds, but no item is smaller than the least and, of the largest, each is full.
    const size_t entries = BH * words * 32 * topk;
    const size_t parts = (size_t)kDkdvGroups * share_rounds(share_steps(rows)), by_least = entries / members_of(0, dm.G);
    const size_t by_most = entries / members_of(kMostSteps, dm.G), some = parts < by_least ? parts : by_least;
    const size_t full = some > by_most ? some : by_most;
    const size_t spill = full + BH * nb + tails;
    // Never more than a list per queue took when segments had 2048 tokens, an item 16 bytes and at least 12 steps: buffers of that size stay
    // large enough.
    const int64_t steps0 = dm.batch * (int64_t)T * (rows_per_block(dm) / kBlock) / kShareRows;
    const size_t members0 = (size_t)(steps0 < 12 ? 12 : steps0 > 64 ? 64 : steps0) * 32 / dm.G;
    const size_t ent0 = (size_t)64 * 32 * dm.topk, seg0 = (ent0 < nb ? ent0 : nb) + 2 * ent0 / (members0 < 1024 ? members0 : 1024) + 33;
    const size_t lists0 = 2 * ((BH * ((words + 63) / 64) + kQueues - 1) / kQueues) * seg0;            // places per queue
    const size_t rest = spill / kQueues + slots * tail + (size_t)9 * t.stride / 16 + 64;
    const size_t room = (lists0 > rest ? lists0 - rest : 0) / (slots * kSlices);
    cap = cap < room ? cap : room;
    t.window = t.shift < 3 ? 3 - t.shift : 0;
    t.cap = (int32_t)(cap << t.shift);
    t.tail = (int32_t)(t.shift < 3 ? tail : tail << (t.shift - 3));
    t.size = (int32_t)t.begin(0, t.n);
    size_t o = 0;
    l.kvb = o;      o += al256(BH * l.nb_cap * kBwdBlockU4 * sizeof(uint4));
    l.rowc = o;     o += al256(((size_t)dm.batch * T * dm.Hq * 2 + 32) * sizeof(float));
    l.bits = o;     o += al256(BH * l.words * l.nb_cap * sizeof(uint32_t));
    l.acc_dk = o;   o += al256(BH * T * kHeadDim * sizeof(float));
    l.acc_dv = o;   o += al256(BH * T * kHeadDim * sizeof(float));
    l.counters = o; o += al256((size_t)(kQueues + 1) * t.stride * sizeof(uint32_t));
    l.items = o;    o += al256(((size_t)kQueues * t.size + spill) * sizeof(uint64_t));
    l.total = o;
    return l;
}

size_t attn_bwd_ws_bytes(const Dims &dm) { return bwd_layout(dm).total; }

__device__ inline int seq_len(const Dims &dm, const int32_t *__restrict__ seqlens, int b) {
    const int32_t L = seqlens[b];
    return L < 0 ? 0 : (L > dm.max_seqlen ? dm.max_seqlen : L);
}

// ---- everything per 64-token block, one workgroup each: its fragments, the membership bits of its tokens, its cleared
// accumulators (the memory is touched anyway and a launch is saved) --------------------------------------------------
// section 0, K rows:  fragment (ks, mt), lane (g, m):  K[64j + 16mt + m][32ks + 8g .. +7]
// section 1, V rows:  the same of V
__global__ __launch_bounds__(256) void pack_bwd_kernel(Dims dm, Tensor k, Tensor v,
                                                        const int32_t *__restrict__ seqlens,
                                                        uint4 *__restrict__ kvb, int32_t nb_cap,
                                                        const int32_t *__restrict__ block_idx, uint32_t *__restrict__ bits,
                                                        float *__restrict__ acc_dk, float *__restrict__ acc_dv,
                                                        uint32_t *__restrict__ counters, int32_t n_counters, float *__restrict__ null_row) {
    __shared__ __align__(16) __bf16 Ks[kBlock * 136];
    __shared__ __align__(16) __bf16 Vs[kBlock * 136];
    arguments_arrive(dm.Hkv, dm.topk, dm.max_seqlen, seqlens, k.ptr, k.sb, k.sh, k.st, kvb, nb_cap, block_idx, bits);
    arguments_arrive(v.ptr, v.sb, v.sh, v.st, acc_dk, acc_dv);
    const int j = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x;
    if (j == nb_cap) {                                    // behind the blocks, a workgroup for the whole call
        if ((h | b) != 0) return;
        int blocks = 0;                                   // of the call, a word per wavefront
        for (int i = tid; i < dm.batch; i += 256) blocks += (seq_len(dm, seqlens, i) + kBlock - 1) / kBlock;
        blocks = wave_inclusive_sum(blocks);
        for (int i = tid; i < n_counters; i += 256)
            if (i < n_counters - kCounterLine + 4 || i >= n_counters - kCounterLine + 8) counters[i] = 0u;
        if ((tid & 63) == 63) counters[n_counters - kCounterLine + 4 + (tid >> 6)] = (uint32_t)blocks;
        if (tid < 32) null_row[tid] = tid < 16 ? -INFINITY : 0.f;       // the constants of a row that is not there: p = 0
        return;
    }
    int32_t L = uniform_load(seqlens + b);
    const int sc = tid & 15, sr = tid >> 4;
    const int64_t bh = (int64_t)b * dm.Hkv + h;
    const __bf16 *kb = k.ptr + (b * k.sb + h * k.sh + (int64_t)j * kBlock * k.st), *vb = v.ptr + (b * v.sb + h * v.sh + (int64_t)j * kBlock * v.st);
    const int32_t *rows = block_idx + (bh * dm.max_seqlen + (int64_t)j * kBlock) * dm.topk;
    L = L < 0 ? 0 : (L > dm.max_seqlen ? dm.max_seqlen : L);
    const int n_tok = min(kBlock, (int)L - j * kBlock), n_ent = n_tok * dm.topk;
    if (n_tok <= 0) return;
    // Everything is asked for at once: the lists, which the membership words are made of while the rows are on their way (500 tokens 5.3 -> 4.4 us,
    // 2 x 4096 13.2 -> 11.0, 32K x 2 heads 27.8 -> 23.7: 105 MB).
    constexpr int kEnt = 4;                               // entries of a thread kept in registers: top-k 16; more are read where they are used
    int ent[kEnt];
    uint4 xk[4], xv[4];
#pragma unroll
    for (int i = 0; i < kEnt; ++i) ent[i] = rows[min(tid + 256 * i, n_ent - 1)];
#pragma unroll
    for (int i = 0; i < 4; ++i) {                         // (rows past the end repeat the last one and are stored as zeros)
        xk[i] = *reinterpret_cast<const uint4 *>(kb + min(sr + 16 * i, n_tok - 1) * k.st + 8 * sc);
        xv[i] = *reinterpret_cast<const uint4 *>(vb + min(sr + 16 * i, n_tok - 1) * v.st + 8 * sc);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int64_t a0 = (bh * dm.max_seqlen + (int64_t)j * kBlock) * kHeadDim;
    for (int i = tid; i < n_tok * (kHeadDim / 4); i += 256) {
        *reinterpret_cast<float4 *>(acc_dk + a0 + 4 * i) = float4{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<float4 *>(acc_dv + a0 + 4 * i) = float4{0.f, 0.f, 0.f, 0.f};
    }
    // membership: bit t % 32 of word [t / 32][block] = token t selected the block (blocks 0 .. j, 2048 at a time)
    uint32_t *w = reinterpret_cast<uint32_t *>(Ks);
    static_assert(2 * 2048 * sizeof(uint32_t) <= sizeof(Ks), "two words of 2048 blocks");
    const uint32_t inv = (1u << 20) / (uint32_t)dm.topk + 1u;   // entry e belongs to token e / topk (exact: e < 64 topk <= 4096)
    for (int base = 0; base <= j; base += 2048) {
        const int n = min(2048, j + 1 - base);
        for (int i = tid; i < n; i += 256) w[i] = w[2048 + i] = 0u;
        __syncthreads();
        auto mark = [&](int x, int e) __attribute__((always_inline)) {
            const uint32_t r = (uint32_t)(x - base), tok = ((uint32_t)e * inv) >> 20;
            if (r < (uint32_t)n) atomicOr(&w[2048 * (tok >> 5) + r], 1u << (tok & 31));
        };
#pragma unroll
        for (int i = 0; i < kEnt; ++i)
            if (tid + 256 * i < n_ent) mark(ent[i], tid + 256 * i);
        for (int e = tid + 256 * kEnt; e < n_ent; e += 256) mark(rows[e], e);
        __syncthreads();
        uint32_t *o = bits + (bh * 2 * nb_cap + 2 * j) * nb_cap + base;
        for (int i = tid; i < n; i += 256) {
            o[i] = w[i];
            o[nb_cap + i] = w[2048 + i];
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = sr + 16 * i;
        if (r >= n_tok) xk[i] = xv[i] = uint4{0u, 0u, 0u, 0u};
        *reinterpret_cast<uint4 *>(&Ks[r * 136 + 8 * sc]) = xk[i];
        *reinterpret_cast<uint4 *>(&Vs[r * 136 + 8 * sc]) = xv[i];
    }
    __syncthreads();
    uint4 *dst = kvb + (bh * nb_cap + j) * kBwdBlockU4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = tid + 256 * i;                     // fragment f = c/64, lane = c%64
        const int f = c >> 6, lane = c & 63, m = lane & 15, g = lane >> 4;
        const int ks = f >> 2, mt = f & 3;
        dst[c] = *reinterpret_cast<const uint4 *>(&Ks[(16 * mt + m) * 136 + 32 * ks + 8 * g]);
        dst[1024 + c] = *reinterpret_cast<const uint4 *>(&Vs[(16 * mt + m) * 136 + 32 * ks + 8 * g]);
    }
}

// ---- the scatter's work items --------------------------------------------------------------------------------------
// A wavefront per (segment, kItemBlocks blocks), a lane per four words: the block's members in the segment, cut behind the word that holds
// every `members`-th of them (and behind those inside the block itself, which alone meet the causal edge); item = {sequence and head,
// block, first word, words}.  An item goes to the slice of 128 tokens that it ends in, in the queue of that slice's window, what is
// left at the segment's end to the last slice of one by the block's number.  So workgroups that run together on an XCD read the same
// tokens' q and dout rows, and a block that few tokens
// select is cut once per 8192 of them: every item costs 32 KiB of K and V and 64 KiB of atomic sums (four times the items: 1190 -> 2210 us
// for 32K tokens).  Against segments of 2048 tokens, queued as their wavefronts finished: dk/dv 1220 -> 1120 us at 32K tokens, G = 16
// (segments of 4096: 1100 with the windows' order, 1150 with 2048); the cutting 11.5 -> 9.6 us there and 11.4 -> 6.5 us for
// 2 x 4096 tokens (a thread per block walked its words twice, one after the other).  The slices' order instead of the order in which the
// wavefronts finished inside a window (1024 tokens are 8 MiB of rows, an XCD's L2 holds 4): misses 64 -> 54 million lines, dk/dv by
// itself the same, the backward call 2410 -> 2350 us at 32K tokens, 10950 -> 10850 at 128K (fewer lines from the far cache: the clock
// stays higher in dq too).  Workgroups in front of dq's, which does not need them: as a launch of its own, of 5 to 10 us, 500 tokens, G = 8,
// the whole backward 46.8 -> 41.8 us, training step of 2 x 4096 453.5 -> 449.6.  With windows dealt by their place in the segment, four sequences of 4096 tokens kept half the
// queues empty: 1125 -> 1110.
constexpr int kItemBlocks = 4;
struct BwdItems {                                         // where they come from and go
    const uint32_t *bits;
    uint32_t *counters;
    uint64_t *items;
    int64_t rows_per_block;
    int32_t n_seg, groups;                                // workgroups per sequence and head, a multiple of 8
    int32_t pairs;                                        // of wavefronts to an item
    BwdBins bins;
};
__device__ __forceinline__ void cut_items(const Dims &dm, const int32_t *__restrict__ seqlens, int32_t nb_cap, const BwdItems &to_cut) {
    const uint32_t *__restrict__ bits = to_cut.bits;
    uint32_t *__restrict__ counters = to_cut.counters;
    uint64_t *__restrict__ items = to_cut.items;
    int64_t rows_per_block = to_cut.rows_per_block;
    const int32_t n_seg = to_cut.n_seg;
    BwdBins bins = to_cut.bins;
    static_assert(kSegWords == 4 * 64 && kWindowWords == 4 * 8 && kSlices == 8, "four words a lane, eight lanes a window, one a slice");
    // (the arguments arrive together, not one round trip after another where each is first used)
    asm volatile("" : "+s"(bins.shift), "+s"(bins.cap), "+s"(bins.tail), "+s"(bins.window), "+s"(bins.size), "+s"(bins.stride),
                 "+s"(bins.block_bits), "+s"(rows_per_block), "+s"(counters), "+s"(items));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int seg = (int)(blockIdx.x % (uint32_t)n_seg), j0 = (int)(blockIdx.x / (uint32_t)n_seg * 4 + wave) * kItemBlocks;
    const int h = blockIdx.y, b = blockIdx.z;
    const int64_t bh = (int64_t)b * dm.Hkv + h;
    const int L = seq_len(dm, seqlens, b);
    const uint4 blocks = *reinterpret_cast<const uint4 *>(counters + (kQueues + 1) * bins.stride - kCounterLine + 4);
    const int w0 = seg * kSegWords, w1 = min(w0 + kSegWords, (L + 31) / 32);   // block j's tokens start at word 2j
    if (w0 >= w1 || 2 * j0 >= w1) return;
    const int at = w0 + 4 * lane;                         // this lane's words
    const uint32_t *src = bits + bh * 2 * nb_cap * nb_cap;
    uint32_t x[kItemBlocks][4];
#pragma unroll
    for (int i = 0; i < kItemBlocks; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[i][e] = src[(int64_t)min(at + e, w1 - 1) * nb_cap + min(j0 + i, nb_cap - 1)];
    const int64_t rows = (int64_t)__builtin_amdgcn_readfirstlane(blocks.x + blocks.y + blocks.z + blocks.w) * rows_per_block;
    const int share = share_steps(rows, to_cut.pairs), rounds = share_rounds(share), m = members_of((share + rounds - 1) / rounds, dm.G, to_cut.pairs);
    const float inv = 1.f / (float)(m >= 96 ? min((m + 31) / 32 * 32, kMaxMembers - 32) : m);
    // Windows are numbered through all sequences and heads of the capacity, eight to the queues' next slices; a sequence's are dealt to the
    // queues round robin by its own length (by the capacity's, short sequences in long buffers meet in one queue: 1000 tokens of 8000,
    // 2 heads, G = 16, top-k 8: dk/dv 121 us, so 115; one of 16384 and three short ones 677, so 667).
    const int windows = (2 * nb_cap + kWindowWords - 1) / kWindowWords;
    const int slot = min((int)(bh * windows + seg * kQueues + (lane >> 3)) / kQueues, ((int)(dm.batch * dm.Hkv * windows) + kQueues - 1) / kQueues - 1);
    const int bin = (slot * kSlices + (lane & 7)) >> bins.shift;
    const int queue = (int)((lane >> 3) + bh * ((L + 32 * kWindowWords - 1) / (32 * kWindowWords))) & (kQueues - 1);
    const int run = (1 << min(bins.shift, 3)) - 1;        // lanes of a window that share a bin: run + 1
    const uint32_t places = bins.places(bin);
    const uint32_t begin = (uint32_t)bins.begin(queue, bin);          // (all of it is under a hundredth of a workspace that fits the card)
    uint32_t ends[kItemBlocks];                           // bits 0 .. 3: an item ends with the lane's word; bit 4: the block's last one
    int place[kItemBlocks];                               // (the first lane of a run: where the run's items go)
#pragma unroll
    for (int i = 0; i < kItemBlocks; ++i) {
        const int j = j0 + i;
        int n[4], sum = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            n[e] = at + e < w1 && at + e >= 2 * j ? __popc(x[i][e]) : 0;
            sum += n[e];
        }
        const int incl = wave_inclusive_sum(sum);
        int before = incl - sum, left = 0;                // members so far; those behind the lane's last end (or all, if it has none)
        uint32_t m = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // quotients of integers below 2^13 + 32: half a unit away from the next one, more than the product's error
            const bool full = (int)(((float)(before + n[e]) + 0.5f) * inv) > (int)(((float)before + 0.5f) * inv);
            left += n[e];
            if (full || (at + e == 2 * j + 1 && left > 0)) {
                m |= 1u << e;
                left = 0;
            }
            before += n[e];
        }
        // what is left at the end: behind the last lane that has an end
        const uint64_t have = __ballot(m != 0u);
        const int lane_end = have ? 63 - __builtin_clzll(have) : -1;
        const int total = __builtin_amdgcn_readlane(incl, 63);
        const int tail = have ? total - __builtin_amdgcn_readlane(incl, max(lane_end, 0)) + __builtin_amdgcn_readlane(left, max(lane_end, 0)) : total;
        if (tail > 0 && lane == 8 * (j & 7) + 7) m |= 16u;
        ends[i] = m;
        const int mine = __popc(m), sums = wave_inclusive_sum(mine);
        const int start = __builtin_amdgcn_ds_bpermute(4 * ((lane & ~run) - 1), sums);     // lanes before the run
        const int own = sums - ((lane & ~run) ? start : 0);                                // of the run's, up to this lane
        const int all = __builtin_amdgcn_ds_bpermute(4 * (lane | run), own);
        int to = 0;
        if ((lane & run) == 0 && all > 0) to = (int)atomicAdd(&counters[queue * bins.stride + bin], (uint32_t)all);
        place[i] = to;
        n[0] = own - mine;
        ends[i] |= (uint32_t)n[0] << 8;
    }
    int over = 0;                                         // this lane's items that find their bin full
#pragma unroll
    for (int i = 0; i < kItemBlocks; ++i) {
        const int mine = __popc(ends[i] & 31u);
        place[i] = __builtin_amdgcn_ds_bpermute(4 * (lane & ~run), place[i]) + (int)(ends[i] >> 8);
        over += max(0, min(mine, place[i] + mine - (int)places));
    }
    uint32_t behind = 0;
    if (__any(over > 0)) {
        const int incl = wave_inclusive_sum(over);
        if (lane == 63) behind = atomicAdd(&counters[kQueues * bins.stride], (uint32_t)incl);
        behind = (uint32_t)bins.begin(kQueues, 0) + (uint32_t)__builtin_amdgcn_readlane((int)behind, 63) + (uint32_t)(incl - over);
        // (a length never falls below `places` again: in the end it is what the bin holds)
        if (over > 0) atomicSub(&counters[queue * bins.stride + bin], (uint32_t)over);
        if (lane < kQueues) atomicOr(&counters[lane * bins.stride + bins.stride - kCounterLine], kBehind);
    }
#pragma unroll
    for (int i = 0; i < kItemBlocks; ++i) {
        const uint32_t m = ends[i] & 31u;
        const uint64_t have = __ballot((m & 15u) != 0u);
        const int lane_end = have ? 63 - __builtin_clzll(have) : 0;
        // first word behind the last end of the lanes before this one, and of all
        const uint64_t below = have & ((1ull << lane) - 1ull);
        const int mine_end = 4 * lane + 32 - __clz(m & 15u);                               // (behind the lane's own last end)
        const int prev = __builtin_amdgcn_ds_bpermute(4 * (below ? 63 - __builtin_clzll(below) : 0), mine_end);
        const int last = __builtin_amdgcn_readlane(mine_end, lane_end);
        const int own = max(2 * (j0 + i) - w0, 0);        // (the words before the block's own tokens hold nothing: not even zeros)
        int first = below ? prev : own;
        uint32_t to = begin + (uint32_t)place[i];
        const uint64_t head = bins.item(bh, j0 + i, w0, 1);
        auto put = [&](int f, int e) __attribute__((always_inline)) {
            const uint32_t at = to < begin + places ? to : behind;
            behind += to >= begin + places ? 1u : 0u;
            ++to;
            items[at] = head | (uint64_t)(uint32_t)(f << 8 | (e - f - 1));
        };
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (m & (1u << e)) {
                put(first, 4 * lane + e + 1);
                first = 4 * lane + e + 1;
            }
        if (m & 16u) put(have ? last : own, w1 - w0);
    }
}

// ---- dq: a workgroup owns the tokens of kTiles MFMA tiles of one key-value head ---------------------------
// As in the forward: the 16 columns of a tile are the G query heads of 16 / G tokens, the union of the tokens' block
// lists is walked once, every fragment serves every tile with a token that selected the block; the four wavefronts take
// every fourth block of the union and their sums are added at the end.
// A block is processed as two halves of 32 keys; per half four units of 4 fragments (4 KiB each) rotate through a ring
// of register buffers (8 units per block):
//   K rows of key tile 2hs, of key tile 2hs+1      -> S^T  = K . Q^T
//   V rows of key tile 2hs, of key tile 2hs+1      -> dP^T = V . dO^T
// and the K rows also go to 8 KiB of LDS, from which the transposing load makes the A fragments of dQ^T += K^T . dS^T.
// No single bound at 32K tokens, G = 16: matrix cores 33 % of the time, vector arithmetic 33 %, waits 35 % of the wavefronts'
// time (all four ring units are asked for again only after the last tile's dP).  With several tiles the queries and upstream
// gradients sit in LDS and a tile's scores and dP are formed together; with one tile they sit in registers and the units are
// used one at a time.
// Against two whole tokens per wavefront: 2 x 4096 tokens, G = 8 332 -> 171; 8192 tokens, G = 1 (16 tokens a tile) ~480 -> 96; 32K
// tokens, G = 16 1590 -> 1280 (1415 with a third, transposed copy of K read from memory in place of the LDS turn), D included.
constexpr int kDqUnits = 8, kDqRing = 4;
template <int kG, int kTiles>
struct DqCfg {
    static constexpr bool kLds = kTiles > 1;
    static constexpr int kTPT = 16 / kG, kTok = kTiles * kTPT;
    // LDS: each wave's 32 K rows, [q | dout][tile][ks][lane] (kLds), per column {exponent offset, D}, union list; the merge area
    // lies over the front
    static constexpr int kRowBytes = 4 * 32 * kHeadDim * 2;
    static constexpr int kQueryBytes = kLds ? 2 * kTiles * 4 * 64 * (int)sizeof(uint4) : 0;
    static constexpr int kColumnBytes = kTiles * 16 * (int)sizeof(float2);
    static constexpr int kUnionAt = kRowBytes + kQueryBytes + kColumnBytes;
    static_assert(4 * 8 * 64 * sizeof(float4) <= kRowBytes, "the merge area");
    static size_t lds_bytes(int topk) { return kUnionAt + UnionLds::bytes(kTok, topk) + 16; }
};

template <int kG, int kTiles>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_kernel(Dims dm, Tensor q, Tensor out, Tensor dout,
                                                              const uint4 *__restrict__ kvb,
                                                              int32_t nb_cap, const int32_t *__restrict__ seqlens,
                                                              const int32_t *__restrict__ block_idx,
                                                              const float *__restrict__ lse,
                                                              float *__restrict__ rowc, Tensor dq, BwdItems to_cut) {
    using C = DqCfg<kG, kTiles>;
    constexpr int kRing = kDqRing, kTPT = C::kTPT, kTok = C::kTok;
    static_assert(64 % kTok == 0 && kTok <= 32, "one own block per workgroup; member bits in one word");
    extern __shared__ __align__(16) unsigned char dq_smem[];
    float2 *row_s = reinterpret_cast<float2 *>(dq_smem + C::kRowBytes + C::kQueryBytes);   // [tile][column]: -lse log2(e), D
    int &cnt_s = *reinterpret_cast<int *>(dq_smem + C::kUnionAt + UnionLds::bytes(kTok, dm.topk));
    if ((int)blockIdx.x < to_cut.groups) return cut_items(dm, seqlens, nb_cap, to_cut);
    arguments_arrive(dm.Hkv, dm.Hq, dm.topk, dm.max_seqlen, dm.fill, seqlens, block_idx, q.ptr, q.sb, q.st, q.sh, lse);
    arguments_arrive(out.ptr, out.sb, out.st, out.sh, dout.ptr, dout.sb, dout.st, dout.sh, dm.scale_log2, kvb, nb_cap, rowc);
    const int xcd = blockIdx.x & 7, sl = (int)(blockIdx.x - to_cut.groups) >> 3, h = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t L = uniform_load(seqlens + b);
    L = L < 0 ? 0 : (L > dm.max_seqlen ? dm.max_seqlen : L);
    const int n_tiles = (L + kTok - 1) / kTok, tile = n_tiles - 1 - (((sl / kRun) * 8 + xcd) * kRun + sl % kRun);   // (see the forward's launch)
    const int t0 = tile * kTok;
    if (dm.fill) {                                        // rows past the end: this tile's, or those of a tile behind the last
        const int f0 = tile >= 0 ? t0 : (n_tiles - 1 - tile) * kTok;
        for (int i = threadIdx.x; i < kTok * kG * 16; i += 256) {
            const int tok = f0 + i / (kG * 16);
            if (tok >= L && tok < dm.max_seqlen)
                *reinterpret_cast<uint4 *>(dq.ptr + b * dq.sb + (int64_t)tok * dq.st +
                                           (int64_t)(h * kG + i / 16 % kG) * dq.sh + 8 * (i & 15)) = uint4{0u, 0u, 0u, 0u};
        }
    }
    if (tile < 0) return;                                 // uniform over the workgroup
    // Lists and rows are asked for before anything waits; the union is built meanwhile, by a wavefront that has no rows of its own to turn where
    // there is one (2 x 500 tokens: one tile, G = 1, 10.9 -> 7.5 us; two tiles, G = 16, 15.8 -> 14.7).  With several tiles a wavefront brings one to
    // LDS, with one each keeps it and the first forms D.
    const int union_wave = C::kLds && kTiles == 4 ? 0 : 3;
    const int32_t *idx_rows = block_idx + (((int64_t)b * dm.Hkv + h) * dm.max_seqlen + t0) * dm.topk;
    const UnionRows<kTok> idx_head(idx_rows, wave == union_wave ? min(kTok, L - t0) * dm.topk : 0, lane);
    const int b_own = t0 / kBlock;
    const int n = lane & 15, g = lane >> 4;               // MFMA column (token, query head) and 16-lane group
    const int tn = n / kG;
    const float c = dm.scale_log2;

    static_assert(C::kLds || kTiles == 1, "a tile a wavefront, or one for all");
    bf16x8 qf[1][4], gf[1][4];
    bf16x8 *ql = reinterpret_cast<bf16x8 *>(dq_smem + C::kRowBytes) + lane;   // [q | dout][tile][ks][lane]
    f32x4 acc[kTiles][8];
    const int own = C::kLds ? wave : 0;                   // tile
    const bool forms_d = C::kLds ? wave < kTiles : wave == 0;
    const int tok_d = t0 + own * kTPT + tn, tk = min(tok_d, L - 1);
    const int row_d = h * kG + n % kG;
    bf16x8 xo[4];
    float ls = 0.f;
    if (!C::kLds || wave < kTiles) {
        const __bf16 *qr = q.ptr + b * q.sb + (tk * q.st + row_d * q.sh + 8 * g);
        const __bf16 *gr = dout.ptr + b * dout.sb + (tk * dout.st + row_d * dout.sh + 8 * g);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            qf[0][ks] = load8(qr + 32 * ks);
            gf[0][ks] = load8(gr + 32 * ks);
        }
    }
    if (forms_d) {
        const __bf16 *orow = out.ptr + b * out.sb + (tk * out.st + row_d * out.sh + 8 * g);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) xo[ks] = load8(orow + 32 * ks);
        ls = lse[((int64_t)b * dm.max_seqlen + tk) * dm.Hq + row_d];
    }
    __builtin_amdgcn_sched_barrier(0);
    const UnionLds ul(dq_smem + C::kUnionAt);
    if (wave == union_wave) {
        const int x = build_union<kTok>(idx_head, idx_rows, dm.topk, min(kTok, L - t0), b_own, ul, lane);
        if (lane == 0) cnt_s = x;
    }
    if (forms_d) {
        float d = 0.f;                                    // D = <dout, out> of the row
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) d = __builtin_fmaf((float)xo[ks][e], (float)gf[0][ks][e], d);
        if constexpr (C::kLds)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                ql[(own * 4 + ks) * 64] = qf[0][ks];
                ql[((kTiles + own) * 4 + ks) * 64] = gf[0][ks];
            }
        d = xgroup_sum(d);
        // p = 2^(s*c - lse*log2e); a dead column (no such token, or a row that attended nothing) gets p = 0
        const float ne = (ls > -INFINITY && ls < INFINITY) ? -ls * kLog2e : -INFINITY;
        if (g == 0) {
            row_s[own * 16 + n] = float2{tok_d < L ? ne : -INFINITY, d};
            // the same for dk and dv, per (token, key-value head): G exponent offsets, then G times D
            float *rec = rowc + (((int64_t)b * dm.max_seqlen + tk) * dm.Hkv + h) * (2 * kG) + n % kG;
            if (tok_d < L) {
                rec[0] = ne;
                rec[kG] = d;
            }
        }
    }
    __syncthreads();
    const int cnt = __builtin_amdgcn_readfirstlane(cnt_s);
    // the tokens' own block, the one with the causal edge, comes last; the others from `start` on
    const int own_at = __builtin_amdgcn_readfirstlane(cnt > 0 && ul.list[max(cnt - 1, 0)].x == (uint32_t)b_own ? cnt - 1 : cnt);
    const int start = walk_start(own_at, tile, 64, b_own);
    auto union_entry = [&](int i) __attribute__((always_inline)) {
        const int at = i + start;
        return ul.list[i >= own_at ? min(i, cnt - 1) : at >= own_at ? at - own_at : at];
    };

    // block addresses are uniform: buffer loads, no vector address arithmetic
    const char *kv_head = reinterpret_cast<const char *>(kvb) + ((int64_t)b * dm.Hkv + h) * nb_cap * (kBwdBlockU4 * 16);
    const uint32_t lane16 = 16u * lane;
    u32x4 ring[kRing][4];
    auto block_rsrc = [&](uint32_t blk) __attribute__((always_inline)) {
        const int64_t at = (int64_t)(int)__builtin_amdgcn_readfirstlane(blk) * (kBwdBlockU4 * 16);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(kv_head) + at, 0, kBwdBlockU4 * 16, 0x00027000);
    };
    auto fragment = [&](__amdgpu_buffer_rsrc_t bp, int f) __attribute__((always_inline)) {
        return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(bp, lane16, f * 1024, 0));
    };
    auto issue = [&](int unit, __amdgpu_buffer_rsrc_t bp) __attribute__((always_inline)) {
        const int hs = unit / 4, sec = (unit >> 1) & 1, mt = 2 * hs + (unit & 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) ring[unit % kRing][ks] = fragment(bp, sec * 16 + ks * 4 + mt);
    };
    // this wave's K rows of the half in LDS
    char *kt = reinterpret_cast<char *>(dq_smem) + wave * (C::kRowBytes / 4);

    // One walk; if a result is not finite (see not_finite), another for each token of a tile.
    __shared__ int odd_s[4];
    for (int pass = 0;; ++pass) {
    const uint32_t slot_mask = pass ? 1u << (pass - 1) : (1u << kTPT) - 1u;
#pragma unroll
    for (int u = 0; u < kTiles; ++u)
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) acc[u][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    __builtin_amdgcn_s_waitcnt(0);                        // nothing of the prologue may still be pending inside the ring loop
    uint32_t blk = 0u, bits = 0u;                         // the block at hand and its member bits
    if (wave < cnt) {
        const uint2 e = union_entry(wave);
        blk = __builtin_amdgcn_readfirstlane(e.x);
        bits = __builtin_amdgcn_readfirstlane(e.y);
        const __amdgpu_buffer_rsrc_t bp = block_rsrc(blk);
#pragma unroll
        for (int unit = 0; unit < kRing; ++unit) issue(unit, bp);
    }
    // `edge`: the tokens' own block, the last of the union: the only one with the causal edge
    auto block = [&](auto edge, int ci) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t bp = block_rsrc(blk);
        __amdgpu_buffer_rsrc_t bn = bp;                   // the next block's, known from the second half on
        const int key0 = (int)blk * kBlock;
        // where the lane's piece of key 16t + n goes, and where its four rows for the transposing load begin (keys 16t + 4g .. +3,
        // channels 16dt ..: ^ (dt << 5)); formed anew per block: kept, their variants are spilled
        uint32_t ln = lane;
        asm volatile("" : "+v"(ln));
        const uint32_t kn = ln & 15, kg = ln >> 4, kt_row = 4u * kg + (kn >> 2);
        const uint32_t kt_put = kn * 256u + ((kg ^ (uint32_t)row_swizzle((int)kn)) << 4);            // ^ (ks << 6)
        const uint32_t kt_get = kt_row * 256u + ((((kn & 3) >> 1) ^ (uint32_t)row_swizzle((int)kt_row)) << 4) + 8u * (kn & 1);
        uint32_t tb[kTiles];                              // member bits of the tile's tokens
#pragma unroll
        for (int u = 0; u < kTiles; ++u) {
            tb[u] = (bits >> (u * kTPT)) & slot_mask;
            asm volatile("" : "+s"(tb[u]));               // (its tests stay scalar)
        }
        auto refill = [&](int unit) __attribute__((always_inline)) {
            if (unit + kRing < kDqUnits) issue(unit + kRing, bp);
            else issue(unit + kRing - kDqUnits, bn);      // (a harmless re-read of this block at the tail)
        };
        auto product = [&](int unit, const bf16x8 (&x)[4]) __attribute__((always_inline)) {
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a = mfma16(__builtin_bit_cast(bf16x8, ring[unit % kRing][ks]), x[ks], a);
            return a;
        };
        auto grad = [&](int u, int hs, const f32x4 (&s)[2], const f32x4 (&dp)[2], bf16x8 &dsf) __attribute__((always_inline)) {
            const float2 r = row_s[u * 16 + n];
            const float ne = (kTPT == 1 || ((tb[u] >> tn) & 1u)) ? r.x : -INFINITY;
            const int tok = t0 + u * kTPT + tn;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float p = fast_exp2(__builtin_fmaf(s[t][j], c, ne));
                    if (decltype(edge)::value && key0 + 32 * hs + 16 * t + 4 * g + j > tok) p = 0.f;
                    dsf[4 * t + j] = (__bf16)(p * (dp[t][j] - r.y));
                }
        };
#pragma unroll
        for (int hs = 0; hs < 2; ++hs) {
            if (hs == 1) {
                const uint2 e = union_entry(ci + 4);
                blk = __builtin_amdgcn_readfirstlane(e.x);
                bits = __builtin_amdgcn_readfirstlane(e.y);
                bn = block_rsrc(blk);
            }
            bf16x8 dsf[kTiles];
            auto keep = [&](int r) __attribute__((always_inline)) {
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    *reinterpret_cast<u32x4 *>(kt + (kt_put ^ (uint32_t)(ks << 6)) + r * 4096) = ring[(4 * hs + r) % kRing][ks];
            };
            if constexpr (C::kLds) {
                keep(0);
                keep(1);
#pragma unroll
                for (int u = 0; u < kTiles; ++u) {
                    if (!tb[u]) continue;
                    f32x4 s[2], dp[2];
                    bf16x8 x[4];
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) x[ks] = ql[(u * 4 + ks) * 64];
#pragma unroll
                    for (int r = 0; r < 2; ++r) s[r] = product(4 * hs + r, x);
                    if constexpr (kTiles > 2) __builtin_amdgcn_sched_barrier(0);   // (the next loads reuse x: no register to spare)
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) x[ks] = ql[((kTiles + u) * 4 + ks) * 64];
#pragma unroll
                    for (int r = 0; r < 2; ++r) dp[r] = product(4 * hs + 2 + r, x);
                    grad(u, hs, s, dp, dsf[u]);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) refill(4 * hs + r);
            } else {
                f32x4 s[kTiles][2], dp[kTiles][2];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (r < 2) keep(r);
#pragma unroll
                    for (int u = 0; u < kTiles; ++u) {
                        if (!tb[u]) continue;
                        if (r < 2) s[u][r] = product(4 * hs + r, qf[u]);
                        else dp[u][r - 2] = product(4 * hs + r, gf[u]);
                    }
                    refill(4 * hs + r);
                }
#pragma unroll
                for (int u = 0; u < kTiles; ++u)
                    if (tb[u]) grad(u, hs, s[u], dp[u], dsf[u]);
            }
#pragma unroll
            for (int d4 = 0; d4 < 8; d4 += 4) {
                bf16x8 kf[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t at = kt_get ^ (uint32_t)((d4 + i) << 5);
                    const s16x4 x0 = lds_read_tr16(kt + at), x1 = lds_read_tr16(kt + at + 4096);
                    kf[i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
                }
#pragma unroll
                for (int u = 0; u < kTiles; ++u) {
                    if (!tb[u]) continue;
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[u][d4 + i] = mfma16(kf[i], dsf[u], acc[u][d4 + i]);
                }
            }
        }
    };
    for (int ci = wave; ci < own_at; ci += 4) block(std::false_type{}, ci);
    if (own_at < cnt && (own_at & 3) == wave) block(std::true_type{}, own_at);
    // ---- add the four wavefronts' sums, a tile at a time, and write: lane holds channels 16*dt + 4*g .. +3 of column n ----
    int ln = lane;
    asm volatile("" : "+v"(ln));                          // (what follows is not formed ahead of the walk: no register to spare there)
    {
    const int lane = ln, n = ln & 15, g = ln >> 4, tn = n / kG;
    const float scale = c * kLn2;
    float4 *po = reinterpret_cast<float4 *>(dq_smem);     // [wave][dt][lane]
    const bool writes = pass == 0 || tn == pass - 1;
    bool odd = false;
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
        __syncthreads();
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
            po[(wave * 8 + dt) * 64 + lane] = float4{acc[u][dt][0], acc[u][dt][1], acc[u][dt][2], acc[u][dt][3]};
        __syncthreads();
        const int tok = t0 + u * kTPT + tn;
        if (tok < L && writes) {
            __bf16 *op = dq.ptr + b * dq.sb + (int64_t)tok * dq.st + (int64_t)(h * kG + n % kG) * dq.sh + 4 * g;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int dt = 2 * wave + i;
                f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float4 y = po[(w * 8 + dt) * 64 + lane];
                    x += f32x4{y.x, y.y, y.z, y.w};
                }
                if (kTPT > 1) odd |= not_finite(x);
                bf16x4 r;
#pragma unroll
                for (int j = 0; j < 4; ++j) r[j] = (__bf16)(x[j] * scale);
                *reinterpret_cast<uint2 *>(op + 16 * dt) = __builtin_bit_cast(uint2, r);
            }
        }
    }
    if (kTPT > 1 && pass == 0) {
        const bool again = __any(odd);
        if (lane == 0) odd_s[wave] = again;
    }
    }
    if (kTPT == 1 || pass == kTPT) return;
    __syncthreads();                                      // (also: everyone is past the merge area)
    if (!(odd_s[0] | odd_s[1] | odd_s[2] | odd_s[3])) return;
    }
}

template <int kG, int kTiles>
static int launch_dq_variant(const Dims &dm, Tensor q, Tensor out, Tensor dout, const uint4 *kvb, int32_t nb_cap, const int32_t *seqlens,
                             const int32_t *block_idx, const float *lse, float *rowc, Tensor dq, const BwdItems &to_cut, hipStream_t stream) {
    using C = DqCfg<kG, kTiles>;
    const int32_t n_tiles = (dm.max_seqlen + C::kTok - 1) / C::kTok;
    const int32_t slots = (n_tiles + 8 * kRun - 1) / (8 * kRun) * kRun;
    const size_t lds = C::lds_bytes(dm.topk);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)attn_bwd_dq_kernel<kG, kTiles>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL((attn_bwd_dq_kernel<kG, kTiles>), dim3(to_cut.groups + slots * 8, dm.Hkv, dm.batch), dim3(256), lds,
                       stream, dm, q, out, dout, kvb, nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut);
    return 0;
}

// Tiles per workgroup, by (token, key-value head) rows: four as soon as that still gives every CU its two workgroups
// (the more tokens share a walk, the fewer bytes per token), two while that gives at least three workgroups to four CUs, else
// one.  Past those lines the fewer, longer workgroups lose more to an idle chip than the walk saves (1000 tokens, G = 4:
// 13 / 16 / 27 us with 1 / 2 / 4; 8192 x 2, G = 1: 123 / 107 with 1 / 2; 4096 x 2 x 2, G = 8: 258 / 189 / 173).  A tile of
// G = 1 is 16 tokens and four would not fit the 32 member bits.
template <int kG>
static int launch_dq_group(const Dims &dm, Tensor q, Tensor out, Tensor dout, const uint4 *kvb, int32_t nb_cap, const int32_t *seqlens,
                           const int32_t *block_idx, const float *lse, float *rowc, Tensor dq, const BwdItems &to_cut, hipStream_t stream) {
    const int64_t rows = (int64_t)dm.batch * dm.max_seqlen * dm.Hkv;
    constexpr int kTPT = 16 / kG;
    if constexpr (kG > 1)
        if (rows >= (int64_t)512 * 4 * kTPT) return launch_dq_variant<kG, 4>(dm, q, out, dout, kvb, nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut, stream);
    if (rows >= (int64_t)192 * 2 * kTPT) return launch_dq_variant<kG, 2>(dm, q, out, dout, kvb, nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut, stream);
    return launch_dq_variant<kG, 1>(dm, q, out, dout, kvb, nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut, stream);
}

// ---- dk, dv of one block from the tokens that selected it ------------------------------------------------------
// 128 threads, or 256 in two pairs (kPairs), persistent: a workgroup takes items from its XCD's queue, then from the others', until all are empty.  An item's
// member tokens are expanded from the membership words into a list and walked in steps of 32 rows = (token, head), 32 / G
// tokens; wave = 32 keys of the block through the whole step, in registers from the scores to the sums (32x32x16 MFMAs):
//   S[row, key] = Q.K^T and dP = dO.V^T       A = rows from LDS, B = the keys' K and V rows, held in registers
//   P = exp(S - lse), dS = P (dP - D)         lane = key, 16 rows: as bf16 they are the next products' A operands
//   dV[key, c] += P^T.dO, dK += dS^T.Q        B = the same rows through the transposing LDS load, contraction index permuted to match
// Nothing passes between the two waves but the staged rows: one barrier per step.
// Bound by the matrix cores (busy 54 % of the time at 32K tokens, G = 16) and by the rows' way from the memory-side cache (5.3 GB
// past L2, whose hit rate is 36 %; at 128K 35 GB at 7.1 TB/s).  Leaving parts out, of 1120 us: without the copies 910, without the products 980,
// without the atomic sums 1060.  Operands are read one product ahead; two ahead spill (1120 -> 1690 us).  The 32 keys are what lets 128 accumulator registers and the 64 of K and V fit a wavefront of two per SIMD; with 16
// keys the LDS reads double.  Against a workgroup per (block, 2048-token segment) with P and dS exchanged through LDS, rows
// of two whole tokens a step, and blocks dealt to the XCDs by their number (the first block, which every token selects, kept
// one XCD busy while the others waited: CUs 55 % busy): 32K tokens, G = 16 3440 -> 1190 us; 2 x 4096 tokens, G = 8
// 690 -> 160; 8192 tokens, G = 1 770 -> 75; 777 tokens, G = 16, top-k 8 204 -> 47.
// Staging: the 16 KiB of q and dout rows of a step (and its 64 scalars) go from memory straight into LDS one step ahead.
// The two slots are two objects and the loop is unrolled by two, so that the compiler's wait counts let reads of one slot run
// under the copies into the other.  A row is 256 bytes; its sixteen 16-byte pieces are stored XOR-swizzled with the
// row's two bit pairs exchanged: an operand load takes one piece from each of 32 rows, a transposing load 32 bytes
// from each of 4 consecutive rows, and both then touch every bank once.
typedef float f32x16 __attribute__((ext_vector_type(16)));
struct __align__(16) BwdSlot {
    uint16_t rows[2][32][kHeadDim];                       // [q | dout][(token, head)][channel]: 16 KiB
    float ld[64];                                         // [exponent offset | D][(token, head)]
};
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
template <int kG, int kPairs>
__global__ __launch_bounds__(128 * kPairs, 2) void attn_bwd_dkdv_kernel(Dims dm, Tensor q, Tensor dout, const uint4 *__restrict__ kvb,
                                                                int32_t nb_cap, const int32_t *__restrict__ seqlens,
                                                                const float *__restrict__ rowc, const float *__restrict__ null_row,
                                                                const uint32_t *__restrict__ bits, uint32_t *__restrict__ counters,
                                                                const uint64_t *__restrict__ items, BwdBins bins,
                                                                float *__restrict__ acc_dk, float *__restrict__ acc_dv) {
    constexpr int kTPS = 32 / kG;                         // tokens per step
    __shared__ uint16_t list[kMaxMembers];                // the item's member tokens as offsets from its first word's first token
    __shared__ BwdSlot slot0s[kPairs], slot1s[kPairs];
    __shared__ uint4 item_s;
    __shared__ int tries_s, total_s;
    __shared__ int part_s, parts_s;                       // a short call's workgroup: its part of an item, of how many (0: items from the queues)
    __shared__ __align__(16) uint32_t bins_s[kBins];                  // items in the queue's bins up to this one
    __shared__ BwdBins geo;                               // `bins`, which would hold scalar registers through the walk
    const int tid = threadIdx.x, lane = tid & 63;
    int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    asm volatile("" : "+s"(wave));                        // (a scalar, also after the compiler's own rewriting)
    const int c32 = lane & 31, hf = lane >> 5;
    const int kh = kPairs == 2 ? wave & 1 : wave, pair = kPairs == 2 ? wave >> 1 : 0;     // key half; the pair's part of the steps
    BwdSlot &slot0 = slot0s[pair], &slot1 = slot1s[pair];
    const float c = dm.scale_log2;
    const __bf16 *const s_ptr = kh == 0 ? q.ptr : dout.ptr;
    const int64_t s_sb = kh == 0 ? q.sb : dout.sb, s_sh = kh == 0 ? q.sh : dout.sh, s_st = kh == 0 ? q.st : dout.st;
    const uint32_t s_head = (uint32_t)(s_sh * 2);         // bytes from head to head
    auto queue_of = [&](int x) __attribute__((always_inline)) { return x < kQueues ? (int)((blockIdx.x + x) % kQueues) : kQueues; };
    auto draw = [&](int x) __attribute__((always_inline)) {
        return atomicAdd(&counters[queue_of(x) * geo.stride + geo.stride - kCounterLine], 1u);
    };
    uint32_t ticket = 0;                                  // thread 0: place in queue `tries` behind the own one
    auto look_at = [&](int x) __attribute__((always_inline)) {       // wave 0: a queue's lengths and a place in it, one round trip
        static_assert(kBins == 4 * 64 && kCounterLine % 4 == 0, "four bins a lane");
        uint4 n = {0u, 0u, 0u, 0u};
        if (4 * lane < geo.stride - kCounterLine) n = reinterpret_cast<const uint4 *>(counters + queue_of(x) * geo.stride)[lane];   // (0 past geo.n)
        if (lane == 0) {
            tries_s = x;
            ticket = draw(x);
        }
        n.y += n.x;
        n.z += n.y;
        n.w += n.z;
        const uint32_t before = (uint32_t)wave_inclusive_sum((int)n.w) - n.w;
        reinterpret_cast<uint4 *>(bins_s)[lane] = uint4{n.x + before, n.y + before, n.z + before, n.w + before};
    };
    if (wave == 0) {
        geo = bins;                                       // by every lane: each reads what it has written itself
        uint4 it = {0u, 0u, 0u, 0u};
        int parts = 0, part = 0;
        if (kPairs == 2 && bins.n <= kSlices) {                          // every bin of every queue in one look
            const uint32_t n = counters[(lane >> 3) * bins.stride + (lane & 7)], behind = counters[kQueues * bins.stride];
            const uint32_t incl = (uint32_t)wave_inclusive_sum((int)n), queued = __builtin_amdgcn_readlane(incl, 63);
            const uint32_t all = queued + __builtin_amdgcn_readfirstlane(behind);
            if (all <= (uint32_t)(kDkdvGroups / kPairs)) {
                parts = all <= kPartItems / 4 ? 4 : all <= kPartItems ? 2 : 1;
                // neighbours in the queues' order, which share rows, to one XCD
                const uint32_t ids = all * (uint32_t)parts, per = ids >> 3, rem = ids & 7u, xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;
                if (slot < per + (xcd < rem ? 1u : 0u)) {
                    const uint32_t id = xcd * per + (xcd < rem ? xcd : rem) + slot, t = id / (uint32_t)parts;
                    part = (int)(id - t * (uint32_t)parts);
                    int64_t at = geo.begin(kQueues, 0) + (int64_t)(t - queued);
                    if (t < queued) {
                        const int bin = __popcll(__ballot(incl <= t));
                        at = geo.begin(bin >> 3, bin & 7) + (int64_t)(t - (bin ? __builtin_amdgcn_readlane(incl, bin - 1) : 0u));
                    }
                    it = geo.unpack(items[at]);
                }
            }
        }
        if (parts == 0) look_at(0);
        if (kPairs == 2 && lane == 0) {
            item_s = it;
            parts_s = parts;
            part_s = part;
        }
    }
    for (;;) {
        // ---- next item ----------------------------------------------------------------------------------------------
        if (wave == 0 && (kPairs == 1 || parts_s == 0)) {
            uint4 it = {0u, 0u, 0u, 0u};
            for (int x = __builtin_amdgcn_readfirstlane(tries_s);;) {   // ends: a queue that is found empty stays empty
                const uint32_t drawn = __builtin_amdgcn_readfirstlane(ticket), t = drawn & ~kBehind;
                const int four = __popcll(__ballot(bins_s[4 * lane + 3] <= t));
                const int bin = 4 * four + __popcll(__ballot(bins_s[min(4 * four + (lane & 3), kBins - 1)] <= t) & 15ull);
                if (four < 64) {
                    const uint32_t before = bin ? __builtin_amdgcn_readfirstlane(bins_s[bin - 1]) : 0u;
                    it = geo.unpack(items[geo.begin(queue_of(x), bin) + (t - before)]);
                    break;
                }
                if (++x >= kQueues + (int)(drawn / kBehind)) break;
                look_at(x);
            }
            if (lane == 0) item_s = it;
        }
        __syncthreads();                                  // (also: everyone is past the last item's reads of the list and the slots)
        const int bh = (int)__builtin_amdgcn_readfirstlane(item_s.x), j = (int)__builtin_amdgcn_readfirstlane(item_s.y);
        const int tok0 = 32 * (int)__builtin_amdgcn_readfirstlane(item_s.z);
        const int nw = (int)__builtin_amdgcn_readfirstlane(item_s.w);
        if (nw == 0) return;                              // uniform: every queue is empty
        const int b = bh / dm.Hkv, h = bh - b * dm.Hkv;
        const int L = seq_len(dm, seqlens, b);
        // ---- B operands: K and V rows of keys 32kh + c32, channels 16ks + 8hf .. +7 -------------------------------------
        const u32x4 *blk = reinterpret_cast<const u32x4 *>(kvb) + ((int64_t)bh * nb_cap + j) * kBwdBlockU4 +
                           (2 * kh + ((lane >> 4) & 1)) * 64 + hf * 16 + (lane & 15);
        bf16x8 kB[8], vB[8];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const int at = (ks >> 1) * 4 * 64 + (ks & 1) * 32;
            kB[ks] = __builtin_bit_cast(bf16x8, blk[at]);
            vB[ks] = __builtin_bit_cast(bf16x8, blk[16 * 64 + at]);
        }
        // ---- member tokens, ascending -----------------------------------------------------------------------------------
        if (wave == 0) {
            int n = 0;
            for (int w0 = 0; w0 < nw; w0 += 64) {
                uint32_t w = 0u;
                if (w0 + lane < nw) w = bits[((int64_t)bh * 2 * nb_cap + (tok0 >> 5) + w0 + lane) * nb_cap + j];
                const int mine = __popc(w), incl = wave_inclusive_sum(mine);
                int at = n + incl - mine;
                n += __builtin_amdgcn_readlane(incl, 63);
                while (w) {
                    const int bit = __ffs(w) - 1;
                    w &= w - 1;
                    list[at++] = (uint16_t)((w0 + lane) * 32 + bit);
                }
            }
            if (lane == 0) total_s = n;
        }
        __syncthreads();
        int total = __builtin_amdgcn_readfirstlane(total_s), first = 0, last = (total + kTPS - 1) / kTPS;     // members; this pair's steps
        if constexpr (kPairs == 2) {
            const int parts = __builtin_amdgcn_readfirstlane(parts_s), part = __builtin_amdgcn_readfirstlane(part_s), steps = last;
            if (parts) {
                first = steps * part / parts;
                last = steps * (part + 1) / parts;
                if (first >= last) return;                // (more parts than steps)
            }
            total = min(total, last * kTPS);              // (the second pair may go a step past them: rows that are not there)
            const int each = (last - first + 1) / 2;
            first += pair * each;
            last = first + each;
        }

        const __bf16 *s_base = s_ptr + b * s_sb + (int64_t)(h * kG) * s_sh + (int64_t)tok0 * s_st;
        asm volatile("" : "+s"(s_base));
        const char *s_rec = reinterpret_cast<const char *>(rowc + (((int64_t)b * dm.max_seqlen + tok0) * dm.Hkv + h) * (2 * kG));
        auto stage = [&](BwdSlot &dst, int p) __attribute__((always_inline)) {
            // wave 0 copies q, wave 1 dout: 1 KiB copies of rows 4i + lane/16 (what depends on the lane only is formed anew each
            // time: registers are what this kernel has least of)
            uint32_t ln = lane;
            asm volatile("" : "+v"(ln));
            const uint32_t s_row = ((ln >> 4) % kG) * s_head, s_piece = ((ln & 15) ^ ((ln >> 4) << 2)) << 4;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                auto to = (__attribute__((address_space(3))) void *)&dst.rows[kh][4 * i][0];
                if constexpr (kG >= 4) {
                    const int tok = __builtin_amdgcn_readfirstlane((int)list[min(p * kTPS + 4 * i / kG, total - 1)]);
                    const __amdgpu_buffer_rsrc_t src =
                        __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(s_base + (int64_t)tok * s_st), 0, 0xffffffffu, 0x00027000);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, to, 16, (int)((s_piece ^ ((i & 3) << 4)) + s_row), (int)(4 * i % kG * s_head), 0, 0);
                } else {
                    const int tok = list[min(p * kTPS + (int)(4 * i + (ln >> 4)) / kG, total - 1)];
                    const char *src = reinterpret_cast<const char *>(s_base + (int64_t)tok * s_st) + (s_piece ^ ((i & 3) << 4)) + s_row;
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, to, 16, 0, 0);
                }
            }
            if (kh == 1) {
                const int at = p * kTPS + (int)(ln & 31) / kG;
                const uint32_t off = list[min(at, total - 1)] * (uint32_t)(dm.Hkv * 2 * kG * 4) + 4u * ((ln >> 5) * kG + ln % kG);
                const char *src = at < total ? s_rec + off : reinterpret_cast<const char *>(null_row) + 4u * (16 * (ln >> 5));
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                                 (__attribute__((address_space(3))) void *)&dst.ld[0], 4, 0, 0);
            }
        };
        // an item's walk; `edge`: the members lie inside the block itself (apart: the others have no registers for it)
        auto walk = [&](auto edge) __attribute__((always_inline)) {
        f32x16 dk[4], dv[4];                              // [channel tile]: keys 8(v/4) + 4hf + v%4 of the half, channel 32ct + c32
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) dk[i][v] = dv[i][v] = 0.f;
        auto step = [&](const BwdSlot &cur, BwdSlot &next, int p) __attribute__((always_inline)) {
            __builtin_amdgcn_s_waitcnt(0);                // this wavefront's copies for step p have landed
            __syncthreads();                              // everyone's have, and everyone is past step p - 1
            stage(next, p + 1);                           // (past the end: copies of the last token, never used)
            const char *xq = reinterpret_cast<const char *>(&cur.rows[0][0][0]);
            const char *xg = reinterpret_cast<const char *>(&cur.rows[1][0][0]);
            uint32_t ln = lane;
            asm volatile("" : "+v"(ln));
            const uint32_t hf = ln >> 5;
            // operand loads: piece 2ks + hf of row lane % 32; transposed: rows 16s + 8rd + 4hf + 0..3 at channel tile ct, whose pieces
            // start at 4ct and have swizzle 2rd ^ that of row 4hf + 0..3
            const uint32_t ar = (ln & 31) * 256u + ((hf ^ (uint32_t)row_swizzle((int)(ln & 15))) << 4);
            const uint32_t t_r = 4u * hf + ((ln & 15) >> 2), t_c = 2u * ((ln >> 4) & 1) + ((ln & 3) >> 1);
            const uint32_t at = t_r * 256u + ((t_c ^ (uint32_t)row_swizzle((int)t_r)) << 4) + 8u * (ln & 1);
            auto rows_of = [&](const char *x, int ks) __attribute__((always_inline)) {
                return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(x + (ar ^ (uint32_t)(ks << 5))));
            };
            auto columns_of = [&](const char *x, int i) __attribute__((always_inline)) {       // i = 4 s2 + ct
                const uint32_t s2 = i >> 2, ct = i & 3;
                const s16x4 x0 = lds_read_tr16(x + ((at ^ (ct << 6)) + 16 * s2 * 256u));
                const s16x4 x1 = lds_read_tr16(x + ((at ^ ((ct << 6) | (2 << 4))) + (16 * s2 + 8) * 256u));
                return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
            };
            f32x16 s, dp;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = dp[v] = 0.f;
            bf16x8 xa[2], xb[2];                          // the next operands are under way while the matrix cores work
            xa[0] = rows_of(xq, 0);
            xb[0] = rows_of(xg, 0);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                if (ks < 7) {
                    xa[(ks + 1) & 1] = rows_of(xq, ks + 1);
                    xb[(ks + 1) & 1] = rows_of(xg, ks + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                s = mfma32(xa[ks & 1], kB[ks], s);
                dp = mfma32(xb[ks & 1], vB[ks], dp);
            }
            // entry v: row 8(v/4) + 4hf + v%4, key 32kh + lane % 32
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                if (v4 & 1) __builtin_amdgcn_sched_barrier(0);
                const float4 n4 = *reinterpret_cast<const float4 *>(&cur.ld[8 * v4 + 4 * hf]);
                const float ne[4] = {n4.x, n4.y, n4.z, n4.w};
#pragma unroll
                for (int r = 0; r < 4; ++r) s[4 * v4 + r] = fast_exp2(__builtin_fmaf(s[4 * v4 + r], c, ne[r]));
            }
            if constexpr (decltype(edge)::value) {
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int m = p * kTPS + (int)(8 * v4 + 4 * hf + (kG < 4 ? r : 0)) / kG;
                        const int tok = tok0 + list[min(m, total - 1)];
                        s[4 * v4 + r] = j * kBlock + 32 * kh + (int)(ln & 31) > tok ? 0.f : s[4 * v4 + r];
                    }
            }
            bf16x8 pf[2], sf[2];
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                if (v4 & 1) __builtin_amdgcn_sched_barrier(0);
                const float4 d4 = *reinterpret_cast<const float4 *>(&cur.ld[32 + 8 * v4 + 4 * hf]);
                const float dl[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pf[v4 >> 1][4 * (v4 & 1) + r] = (__bf16)s[4 * v4 + r];
                    sf[v4 >> 1][4 * (v4 & 1) + r] = (__bf16)(s[4 * v4 + r] * (dp[4 * v4 + r] - dl[r]));
                }
            }
            xa[0] = columns_of(xg, 0);
            xb[0] = columns_of(xq, 0);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (i < 7) {
                    xa[(i + 1) & 1] = columns_of(xg, i + 1);
                    xb[(i + 1) & 1] = columns_of(xq, i + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                dv[i & 3] = mfma32(pf[i >> 2], xa[i & 1], dv[i & 3]);
                dk[i & 3] = mfma32(sf[i >> 2], xb[i & 1], dk[i & 3]);
            }
        };
        stage(slot0, first);
        for (int p = first;;) {
            step(slot0, slot1, p);
            if (++p >= last) break;
            step(slot1, slot0, p);
            if (++p >= last) break;
        }
        // ---- add to the block's sums: an instruction covers 32 channels of two keys, two cache lines ------------------------
        if (tid == 0 && (kPairs == 1 || parts_s == 0)) ticket = draw(tries_s);       // the next item's place, under way meanwhile
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int64_t o = ((int64_t)bh * dm.max_seqlen + (int64_t)j * kBlock + 32 * kh + 4 * (ln >> 5)) * kHeadDim + (ln & 31);
        const int left = L - (j * kBlock + 32 * kh + 4 * (ln >> 5));
        if constexpr (kPairs == 2) {                      // the first pair adds up dk, the second dv
            float4 *hand0 = reinterpret_cast<float4 *>(&slot0s[0]), *hand1 = reinterpret_cast<float4 *>(&slot1s[0]);
            static_assert(sizeof(slot0s) >= 2 * 16 * 64 * sizeof(float4), "a pair's sums of one kind");
            __builtin_amdgcn_s_waitcnt(0);                // (the copies past the end have landed)
            __syncthreads();
            float4 *put = (pair ? hand1 : hand0) + kh * 1024 + ln;
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const f32x16 &x = pair ? dk[ct] : dv[ct];
                    put[(ct * 4 + v4) * 64] = float4{x[4 * v4], x[4 * v4 + 1], x[4 * v4 + 2], x[4 * v4 + 3]};
                }
            __syncthreads();
            const float4 *get = (pair ? hand0 : hand1) + kh * 1024 + ln;
            float *to = (pair ? acc_dv : acc_dk) + o;
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                float4 y[4];
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) y[ct] = get[(ct * 4 + v4) * 64];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (8 * v4 + r < left) {
#pragma unroll
                        for (int ct = 0; ct < 4; ++ct) {
                            const float z = r == 0 ? y[ct].x : r == 1 ? y[ct].y : r == 2 ? y[ct].z : y[ct].w;
                            unsafeAtomicAdd(to + (8 * v4 + r) * kHeadDim + 32 * ct, (pair ? dv[ct][4 * v4 + r] : dk[ct][4 * v4 + r]) + z);
                        }
                    }
            }
        } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = 8 * (v >> 2) + (v & 3);
            if (key < left) {
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) {
                    unsafeAtomicAdd(acc_dk + o + key * kHeadDim + 32 * ct, dk[ct][v]);
                    unsafeAtomicAdd(acc_dv + o + key * kHeadDim + 32 * ct, dv[ct][v]);
                }
            }
        }
        }
        };
        if (tok0 >= (j + 1) * kBlock) walk(std::false_type{});
        else walk(std::true_type{});
        __builtin_amdgcn_s_waitcnt(0);                    // the copies past the end have landed: the slots may be filled anew
        if (kPairs == 2 && parts_s != 0) return;          // uniform
        __syncthreads();
    }
}

template <int kG, int kPairs>
static void launch_dkdv_pairs(const Dims &dm, Tensor q, Tensor dout, const uint4 *kvb, const BwdLayout &l, const int32_t *seqlens,
                        const float *rowc, const float *null_row, const uint32_t *bits, uint32_t *counters, const uint64_t *items,
                        float *acc_dk, float *acc_dv, hipStream_t stream) {
    hipLaunchKernelGGL((attn_bwd_dkdv_kernel<kG, kPairs>), dim3(kDkdvGroups / kPairs), dim3(128 * kPairs), 0, stream, dm, q, dout, kvb, l.nb_cap, seqlens, rowc,
                       null_row, bits, counters, items, l.bins, acc_dk, acc_dv);
}

template <int kG>
static void launch_dkdv(const Dims &dm, Tensor q, Tensor dout, const uint4 *kvb, const BwdLayout &l, const int32_t *seqlens,
                        const float *rowc, const float *null_row, const uint32_t *bits, uint32_t *counters, const uint64_t *items,
                        float *acc_dk, float *acc_dv, hipStream_t stream) {
    if (l.pairs == 2) launch_dkdv_pairs<kG, 2>(dm, q, dout, kvb, l, seqlens, rowc, null_row, bits, counters, items, acc_dk, acc_dv, stream);
    else launch_dkdv_pairs<kG, 1>(dm, q, dout, kvb, l, seqlens, rowc, null_row, bits, counters, items, acc_dk, acc_dv, stream);
}

// ---- fp32 accumulators -> bf16 gradients ------------------------------------------------------------------
__global__ __launch_bounds__(256) void bwd_finish_kernel(Dims dm, const int32_t *__restrict__ seqlens,
                                                          const float *__restrict__ acc_dk,
                                                          const float *__restrict__ acc_dv, Tensor dk, Tensor dv) {
    const int b = blockIdx.z, h = blockIdx.y;
    const int L = seq_len(dm, seqlens, b);
    const int t = blockIdx.x * 16 + (threadIdx.x >> 4), c8 = (threadIdx.x & 15) * 8;
    if (t >= L) {
        if (dm.fill && t < dm.max_seqlen) {
            *reinterpret_cast<uint4 *>(dk.ptr + b * dk.sb + h * dk.sh + (int64_t)t * dk.st + c8) = uint4{0u, 0u, 0u, 0u};
            *reinterpret_cast<uint4 *>(dv.ptr + b * dv.sb + h * dv.sh + (int64_t)t * dv.st + c8) = uint4{0u, 0u, 0u, 0u};
        }
        return;
    }
    const float scale = dm.scale_log2 * kLn2;
    const int64_t src = (((int64_t)b * dm.Hkv + h) * dm.max_seqlen + t) * kHeadDim + c8;
    const float4 k0 = *reinterpret_cast<const float4 *>(acc_dk + src), k1 = *reinterpret_cast<const float4 *>(acc_dk + src + 4);
    const float4 v0 = *reinterpret_cast<const float4 *>(acc_dv + src), v1 = *reinterpret_cast<const float4 *>(acc_dv + src + 4);
    const float kf[8] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w};
    const float vf[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
    bf16x8 ko, vo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        ko[e] = (__bf16)(kf[e] * scale);
        vo[e] = (__bf16)vf[e];
    }
    *reinterpret_cast<uint4 *>(dk.ptr + b * dk.sb + h * dk.sh + (int64_t)t * dk.st + c8) = __builtin_bit_cast(uint4, ko);
    *reinterpret_cast<uint4 *>(dv.ptr + b * dv.sb + h * dv.sh + (int64_t)t * dv.st + c8) = __builtin_bit_cast(uint4, vo);
}

int launch_attn_bwd(const Dims &dm, Tensor q, Tensor k, Tensor v, Tensor out, Tensor dout, const float *lse,
                    const int32_t *seqlens, const int32_t *block_idx, Tensor dq, Tensor dk, Tensor dv, void *ws,
                    hipStream_t stream) {
    if (dm.batch <= 0 || dm.max_seqlen <= 0) return 0;
    const BwdLayout l = bwd_layout(dm);
    char *base = reinterpret_cast<char *>(ws);
    uint4 *kvb = reinterpret_cast<uint4 *>(base + l.kvb);
    float *rowc = reinterpret_cast<float *>(base + l.rowc);
    float *null_row = rowc + (size_t)dm.batch * dm.max_seqlen * dm.Hq * 2;
    uint32_t *bits = reinterpret_cast<uint32_t *>(base + l.bits), *counters = reinterpret_cast<uint32_t *>(base + l.counters);
    uint64_t *items = reinterpret_cast<uint64_t *>(base + l.items);
    float *acc_dk = reinterpret_cast<float *>(base + l.acc_dk), *acc_dv = reinterpret_cast<float *>(base + l.acc_dv);
    const int T = dm.max_seqlen;
    timing_begin("pack_bwd_kernel", stream);
    hipLaunchKernelGGL(pack_bwd_kernel, dim3(l.nb_cap + 1, dm.Hkv, dm.batch), dim3(256), 0, stream, dm, k, v, seqlens, kvb,
                       l.nb_cap, block_idx, bits, acc_dk, acc_dv, counters, (kQueues + 1) * l.bins.stride, null_row);
    timing_end(stream);
    const int32_t groups = l.n_seg * ((l.nb_cap + 4 * kItemBlocks - 1) / (4 * kItemBlocks));
    const BwdItems to_cut = {bits, counters, items, rows_per_block(dm), l.n_seg, (groups + 7) & ~7, l.pairs, l.bins};
    timing_begin("attn_bwd_dq_kernel", stream);
    int err = (int)hipErrorInvalidValue;
    switch (dm.G) {
        case 1: err = launch_dq_group<1>(dm, q, out, dout, kvb, l.nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut, stream); break;
        case 2: err = launch_dq_group<2>(dm, q, out, dout, kvb, l.nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut, stream); break;
        case 4: err = launch_dq_group<4>(dm, q, out, dout, kvb, l.nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut, stream); break;
        case 8: err = launch_dq_group<8>(dm, q, out, dout, kvb, l.nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut, stream); break;
        case 16: err = launch_dq_group<16>(dm, q, out, dout, kvb, l.nb_cap, seqlens, block_idx, lse, rowc, dq, to_cut, stream); break;
    }
    if (err) return err;
    timing_end(stream);
    timing_begin("attn_bwd_dkdv_kernel", stream);
    switch (dm.G) {
        case 1: launch_dkdv<1>(dm, q, dout, kvb, l, seqlens, rowc, null_row, bits, counters, items, acc_dk, acc_dv, stream); break;
        case 2: launch_dkdv<2>(dm, q, dout, kvb, l, seqlens, rowc, null_row, bits, counters, items, acc_dk, acc_dv, stream); break;
        case 4: launch_dkdv<4>(dm, q, dout, kvb, l, seqlens, rowc, null_row, bits, counters, items, acc_dk, acc_dv, stream); break;
        case 8: launch_dkdv<8>(dm, q, dout, kvb, l, seqlens, rowc, null_row, bits, counters, items, acc_dk, acc_dv, stream); break;
        case 16: launch_dkdv<16>(dm, q, dout, kvb, l, seqlens, rowc, null_row, bits, counters, items, acc_dk, acc_dv, stream); break;
    }
    timing_end(stream);
    timing_begin("bwd_finish_kernel", stream);
    hipLaunchKernelGGL(bwd_finish_kernel, dim3((T + 15) / 16, dm.Hkv, dm.batch), dim3(256), 0, stream, dm, seqlens,
                       acc_dk, acc_dv, dk, dv);
    timing_end(stream);
    return (int)hipGetLastError();
}

}  // namespace infllmv2
