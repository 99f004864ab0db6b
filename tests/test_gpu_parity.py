"""GPU parity: the HIP path, called through the C ABI, against the fp64 oracle element by
element on the same seeded inputs.  Sizes span several tiles and ragged tails; the largest
stated workloads are checked on sampled rows."""
import os

import numpy as np
import pytest
import torch

from oracle import ref
from paper_2506_07900_amd import binding, synth
from util import grad_err, logit_mag, out_err, OUT_TOL, compare_selection, lse_err, oracle_params, to_bits, to_dev

pytestmark = pytest.mark.gpu


def dev_i32(a):
    return torch.tensor(np.asarray(a, np.int32), dtype=torch.int32, device="cuda")


def make_batch(seed, seqlens, Hq, Hkv, n_planted=0, heavy=()):
    """Padded batch of independent sequences -> numpy bits q [B,T,Hq,d], k/v [B,Hkv,T,d]."""
    T = max(int(max(seqlens)), 1)
    B = len(seqlens)
    q = np.zeros((B, T, Hq, 128), np.uint16)
    k = np.zeros((B, Hkv, T, 128), np.uint16)
    v = np.zeros((B, Hkv, T, 128), np.uint16)
    for b, l in enumerate(seqlens):
        if l == 0:
            continue
        s = synth.make_sequence(seed * 100 + b, l, Hq, Hkv, n_planted=n_planted, heavy_tail=b in heavy)
        q[b, :l], k[b, :, :l], v[b, :, :l] = s.q, s.k, s.v
    return q, k, v, T


# ------------------------------------------------------------------ the boundary from plain C

def test_c_client_of_the_abi():
    # a C99 program (no Python, no torch: HIP runtime + include/infllmv2.h) runs the three stages on a
    # small dense-degrade case and checks them against loops of its own; exit status 0 = all checks passed
    import subprocess
    here = os.path.join(os.path.dirname(os.path.abspath(__file__)), "c_client")
    exe = os.path.join(here, "abi_client")
    if not os.path.exists(exe):                           # normally built by __graft_entry__.build()
        import importlib.util
        spec = importlib.util.spec_from_file_location("c_client_build", os.path.join(here, "build.py"))
        mod = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(mod)
        mod.build()
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout, r.stderr, flush=True)
    assert r.returncode == 0 and "abi_client ok" in r.stdout


# ------------------------------------------------------------------ stage 1

@pytest.mark.parametrize("seqlens,Hkv", [([2048], 1), ([1077, 31, 32, 0, 47, 48], 2), ([5000, 4999], 2)])
def test_compress_keys_bit_exact(seqlens, Hkv):
    print("case compress", seqlens, Hkv, flush=True)
    prm = binding.Params(Hkv * 4, Hkv)
    q, k, v, T = make_batch(11, seqlens, Hkv * 4, Hkv, heavy=(1,))
    kd = to_dev(k)
    n_cap = binding.num_kernels(T, prm) + 3
    ck = torch.full((len(seqlens), Hkv, n_cap, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    binding.compress_keys(prm, kd, dev_i32(seqlens), T, ck=ck)
    torch.cuda.synchronize()
    got = to_bits(ck)
    sentinel = to_bits(torch.full((1,), 7.0, dtype=torch.bfloat16))[0]
    for b, l in enumerate(seqlens):
        _, want = ref.compress_keys(k[b, :, :l], oracle_params(prm))
        n_c = want.shape[1]
        assert np.array_equal(got[b, :, :n_c], want), (b, l)
        assert np.all(got[b, :, n_c:] == sentinel)          # rows past n_c(l) are never written


def test_compress_keys_incremental_equals_from_scratch():
    print("case compress incremental", flush=True)
    Hkv, L0, steps = 2, 1000, 70
    prm = binding.Params(32, Hkv)
    q, k, v, T = make_batch(12, [L0 + steps, L0 + steps - 13], 32, Hkv)
    kd = to_dev(k)
    lens = np.array([L0, L0 - 13], np.int32)
    ck = binding.compress_keys(prm, kd, dev_i32(lens), T)
    for _ in range(steps):
        lens = lens + 1
        binding.compress_keys(prm, kd, dev_i32(lens), T, ck=ck, n_new_tokens=1)
    full = binding.compress_keys(prm, kd, dev_i32(lens), T)
    torch.cuda.synchronize()
    assert torch.equal(ck.view(torch.int16), full.view(torch.int16))
    for b in range(2):
        _, want = ref.compress_keys(k[b, :, :lens[b]], oracle_params(prm))
        assert np.array_equal(to_bits(ck)[b, :, :want.shape[1]], want)


# ------------------------------------------------------------------ stages 2 + 3, prefill

PREFILL_CASES = [
    # seqlens, Hq, Hkv, topk, planted
    ([2048], 4, 1, 8, 4),            # the smallest stated workload (G = 4)
    ([1077, 333], 32, 2, 16, 6),     # G = 16, ragged tails, two sequences
    ([700], 16, 2, 6, 3),            # G = 8
    ([300, 64, 63, 1], 4, 2, 4, 0),  # G = 2, tiny sequences
    ([450], 2, 2, 5, 2),             # G = 1
    ([1500], 16, 1, 32, 5),          # everything selected up to 2048 tokens: dense degrade
    ([5200], 32, 2, 48, 6),          # wide top-k: two neighbouring tokens list more than 64 distinct blocks
]


def run_prefill(seqlens, Hq, Hkv, topk, planted, seed=21, forced=(1, 2)):
    prm = binding.Params(Hq, Hkv, topk=topk, n_init_blocks=forced[0], n_local_blocks=forced[1])
    q, k, v, T = make_batch(seed, seqlens, Hq, Hkv, n_planted=planted)
    qd, kd, vd, sl = to_dev(q), to_dev(k), to_dev(v), dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, sl, T)
    torch.cuda.synchronize()
    return prm, (q, k, v, T), (qd, kd, vd, sl), ck, idx


@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,planted", PREFILL_CASES)
def test_select_blocks_prefill(seqlens, Hq, Hkv, topk, planted):
    print("case select prefill", seqlens, Hq, Hkv, topk, flush=True)
    prm, (q, k, v, T), dev, ck, idx = run_prefill(seqlens, Hq, Hkv, topk, planted)
    oprm = oracle_params(prm)
    idx = idx.cpu().numpy()
    ckb = to_bits(ck)
    tot = exact = near = 0
    for b, l in enumerate(seqlens):
        if l == 0:
            continue
        n_c = ref.num_kernels(l, 32, 16)
        pos = np.arange(l, dtype=np.int32)
        want, margins, R = ref.select_blocks(q[b, :l], ckb[b, :, :n_c], pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx[b, :, :l], want, margins, R)
        assert not hard, hard[:3]
        tot, exact, near = tot + n, exact + e, near + nt
    print("rows %d exact %d near-tie %d" % (tot, exact, near), flush=True)
    assert near <= max(2, tot // 200)


# Up to 4096 tokens the selection is one pass in one kernel: both sides of each of its sizes (32, 64 blocks) for every
# group size, forced counts including none, batches, tokens that need no scores, few tiles (wavefronts share a tile) and
# many (wavefronts take several), and short lengths of the two-pass kernels.
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,forced", [
    ([2047, 31], 32, 2, 16, (1, 2)), ([2048], 16, 2, 8, (0, 0)), ([2049, 2048, 1], 4, 1, 16, (1, 2)), ([1100], 2, 2, 6, (0, 1)),
    ([4096], 2, 1, 16, (2, 1)), ([4097, 100], 32, 2, 8, (0, 0)), ([4095, 3000], 4, 2, 64, (1, 2)), ([3001], 1, 1, 3, (1, 2)),
    ([8192, 8177, 33], 16, 1, 16, (1, 2)), ([8191], 32, 2, 24, (1, 2)), ([8192], 4, 4, 16, (0, 3)), ([8190, 5000], 2, 2, 16, (1, 0)),
    ([8193, 64], 32, 2, 16, (1, 2)), ([8193], 4, 1, 8, (0, 0))])
def test_select_blocks_prefill_short(seqlens, Hq, Hkv, topk, forced):
    print("case short select", seqlens, Hq, Hkv, topk, forced, flush=True)
    prm, (q, k, v, T), dev, ck, idx = run_prefill(seqlens, Hq, Hkv, topk, 5, seed=33, forced=forced)
    oprm = oracle_params(prm)
    ckb = to_bits(ck)
    tot = near = 0
    rng = np.random.default_rng(8)
    for b, l in enumerate(seqlens):
        pos = np.array(sorted(set(rng.integers(0, l, 150).tolist()) | set(range(max(0, l - 70), l)) | set(range(min(l, 40)))), np.int32)
        want, margins, R = ref.select_blocks(q[b, pos], ckb[b, :, :ref.num_kernels(l, 32, 16)], pos, oprm, want_scores=True)
        got = idx[b][:, torch.from_numpy(pos).long().cuda()].cpu().numpy()
        n, e, nt, hard = compare_selection(got, want, margins, R)
        assert not hard, hard[:3]
        tot, near = tot + n, near + nt
        assert bool((idx[b, :, l:] == -1).all())
    print("rows %d near-tie %d" % (tot, near), flush=True)
    assert near <= max(2, tot // 200)


@pytest.mark.parametrize("T", [5000, 4090])
def test_select_blocks_prefill_ties_go_to_the_lower_block(T):
    # keys of all zeros: every visible kernel of a row scores the same, the tie rule alone decides (more than 64 candidate
    # blocks in the two-pass kernels, fewer in the one-pass kernel)
    Hq, Hkv, topk = 32, 2, 8
    prm = binding.Params(Hq, Hkv, topk=topk)
    q = torch.randn((1, T, Hq, 128), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)).bfloat16()
    ck = torch.zeros((1, Hkv, binding.num_kernels(T, prm), 128), dtype=torch.bfloat16, device="cuda")
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, ck, dev_i32([T]), T)[0].cpu()
    own = torch.arange(T) // 64
    for t in list(range(0, T, 37)) + [T - 1]:
        o = int(own[t])
        want = list(range(min(o + 1, topk - 2))) + [j for j in (o - 1, o) if j >= min(o + 1, topk - 2)]
        assert idx[0, t].tolist() == (want + [-1] * topk)[:topk], t


@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([1077, 333], 32, 2, 16), ([700, 65], 4, 1, 6), ([450], 2, 2, 5)])
def test_block_scores_against_the_oracle(seqlens, Hq, Hkv, topk):
    # the scores the selection ranks (Eq. 1 after the group mean and the max over intersecting kernels),
    # value by value: fp32 with hardware exp2 / log2 on one side, fp64 on the other
    print("case block scores", seqlens, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(23, seqlens, Hq, Hkv, n_planted=4)
    qd, kd, sl = to_dev(q), to_dev(k), dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, T)
    got = binding.block_scores(prm, qd, ck, sl, T).cpu().numpy().astype(np.float64)
    torch.cuda.synchronize()
    ckb = to_bits(ck)
    worst = 0.0
    for b, l in enumerate(seqlens):
        pos = np.arange(l, dtype=np.int32)
        _, _, R = ref.select_blocks(q[b, :l], ckb[b, :, :ref.num_kernels(l, 32, 16)], pos, oprm, want_scores=True)
        for t in range(l):
            lo, hi = min(prm.n_init_blocks, t // 64 + 1), t // 64 - prm.n_local_blocks       # candidate blocks lo..hi
            if hi < lo:
                continue
            w, g = R[:, t, lo:hi + 1], got[b, :, t, lo:hi + 1]
            assert np.array_equal(np.isneginf(w), np.isneginf(g)), (b, t)
            fin = np.isfinite(w)
            assert np.all(np.isfinite(g[fin]))
            if fin.any():
                worst = max(worst, float(np.max(np.abs(g[fin] - w[fin]) / w[fin])))
    print("largest relative error of a block score %.3e" % worst, flush=True)
    assert worst <= 2e-5


# The block scores are those the selection ranks, bit for bit: ranking them gives its lists exactly, on inputs so small that
# scores differ in their last bits only (an independent computation of them ranks about one row in a hundred otherwise).
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,forced", [
    ([1500, 20, 65], 32, 2, 8, (1, 2)), ([3000], 32, 2, 16, (0, 0)), ([4096, 4000], 16, 2, 8, (1, 2)), ([4097, 31], 16, 1, 8, (1, 1)),
    ([2000, 1], 4, 1, 8, (0, 1)), ([4097], 16, 2, 6, (2, 0)), ([2049, 2048], 4, 2, 12, (1, 2)), ([1000], 2, 2, 64, (0, 0)), ([5000], 1, 1, 8, (1, 2)),
    ([5000], 16, 1, 3, (1, 2)), ([5000, 700], 4, 1, 3, (1, 2)), ([1500], 32, 2, 2, (0, 2))])         # (every selected block is forced)
def test_block_scores_rank_as_the_selection_does(seqlens, Hq, Hkv, topk, forced):
    print("case scores ranked", seqlens, Hq, Hkv, topk, forced, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk, n_init_blocks=forced[0], n_local_blocks=forced[1])
    B, T = len(seqlens), max(seqlens)
    gen = torch.Generator(device="cuda").manual_seed(T)
    q = (0.02 * torch.randn((B, T, Hq, 128), device="cuda", generator=gen)).bfloat16()
    k = (0.02 * torch.randn((B, Hkv, T, 128), device="cuda", generator=gen)).bfloat16()
    sl = dev_i32(seqlens)
    ck = binding.compress_keys(prm, k, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, ck, sl, T)
    R = binding.block_scores(prm, q, ck, sl, T)
    own = torch.arange(T, device="cuda")[:, None] // 64
    j = torch.arange(R.shape[-1], device="cuda")[None]
    candidate = (j >= forced[0]) & (j <= own - forced[1])
    for b, l in enumerate(seqlens):
        r = R[b, :, :l]
        assert not bool(torch.isnan(r[:, candidate[:l]]).any())             # every candidate's score is written
        r = torch.where(candidate[:l], r, torch.where(j <= own[:l], float("inf"), -float("inf")))
        best = torch.sort(r, dim=-1, descending=True, stable=True)[1][..., :topk]      # (ties: the lower block)
        best = torch.where(torch.arange(best.shape[-1], device="cuda") <= own[:l], best, 1 << 20)
        best = torch.sort(best, dim=-1)[0]
        best = torch.nn.functional.pad(torch.where(best == 1 << 20, -1, best), (0, topk - best.shape[-1]), value=-1)
        assert bool((best == idx[b, :, :l]).all()), (b, int((best != idx[b, :, :l]).any(-1).sum()))


# The ranking of the two-pass selection, row by row of sixteen lanes and chunk by chunk, where its threshold and its limits lie: 1, 13 | 14,
# 15 .. 32 | 33 picks beside the forced blocks; scores that rise along the row (every chunk replaces all picks), that are high in
# one lane's blocks only (more could enter than are kept) and that tie.
@pytest.mark.parametrize("T,Hq,Hkv,topk", [
    (4500, 16, 1, 4), (4500, 16, 1, 17), (4500, 8, 1, 18), (4500, 4, 1, 35), (4500, 1, 1, 36), (4500, 2, 1, 16),
    (18000, 4, 1, 16), (18000, 8, 1, 35), (36000, 16, 1, 16), (36000, 16, 1, 35), (70000, 16, 1, 17)])
@pytest.mark.parametrize("shape", ["rising", "lane", "ties"])
def test_block_scores_rank_as_the_selection_does_at_its_limits(T, Hq, Hkv, topk, shape):
    print("case ranking", T, Hq, Hkv, topk, shape, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    gen = torch.Generator(device="cuda").manual_seed(topk)
    n_c = binding.num_kernels(T, prm)
    u = torch.randn((128,), device="cuda", generator=gen)
    block = torch.arange(n_c, device="cuda") // 4
    a = {"rising": torch.arange(n_c, device="cuda") / n_c,
         "lane": torch.rand((n_c,), device="cuda", generator=gen) * 0.3 + ((block // 4) % 16 == 3),
         "ties": torch.randint(0, 3, (n_c,), device="cuda", generator=gen) * 0.25}[shape]
    ck = (a[:, None] * u[None])[None, None].bfloat16().contiguous()
    q = (0.1 * u + 0.01 * torch.randn((1, T, Hq, 128), device="cuda", generator=gen)).bfloat16()
    sl = dev_i32([T])
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, ck, sl, T)[0, 0]
    R = binding.block_scores(prm, q, ck, sl, T)[0, 0]
    for t in [x for x in range(0, T, 1531)] + [63, 64, 1023, T // 2, T - 65, T - 1]:
        own = t // 64
        r = R[t, 1:max(1, own - 1)].double()                                # the candidates
        order = torch.argsort(r, descending=True, stable=True)[:max(0, topk - 3)] + 1       # (ties: the lower block)
        want = sorted(set([0] + order.tolist() + [x for x in (own - 1, own) if x >= 0]))
        assert idx[t].tolist() == want + [-1] * (topk - len(want)), t


@pytest.mark.parametrize("forced", [(0, 0), (0, 1), (3, 0), (2, 4)])
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([1100, 333, 70], 32, 2, 8), ([700, 65], 4, 1, 6)])
def test_select_blocks_prefill_other_forced_counts(seqlens, Hq, Hkv, topk, forced):
    # with no local block forced, the query's own block competes on its score, also while it is too
    # short to hold a visible kernel (score -inf)
    print("case select prefill forced", seqlens, Hq, Hkv, topk, forced, flush=True)
    prm, (q, k, v, T), dev, ck, idx = run_prefill(seqlens, Hq, Hkv, topk, 3, forced=forced)
    oprm = oracle_params(prm)
    idx = idx.cpu().numpy()
    ckb = to_bits(ck)
    tot = near = 0
    for b, l in enumerate(seqlens):
        n_c = ref.num_kernels(l, 32, 16)
        pos = np.arange(l, dtype=np.int32)
        want, margins, R = ref.select_blocks(q[b, :l], ckb[b, :, :n_c], pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx[b, :, :l], want, margins, R)
        assert not hard, hard[:3]
        tot, near = tot + n, near + nt
    assert near <= max(2, tot // 200)


@pytest.mark.parametrize("fill", [0, 255])
@pytest.mark.parametrize("topk", [6, 30])
@pytest.mark.parametrize("Hq,Hkv", [(32, 2), (8, 1), (2, 2)])
def test_select_blocks_prefill_own_block_is_a_candidate(Hq, Hkv, topk, fill):
    # no forced local blocks: a token's own block is ranked like any other, on the one kernel that
    # reaches into it from the left (if the token sees it yet).  Lengths just past a multiple of 256
    # put that block one 16-kernel tile (one 64-kernel chunk) past the last kernel of the sequence.
    # The workspace starts as all zeros / all ones: a score the kernels leave unwritten shows up.
    seqlens = [542, 282, 2072, 40, 257]
    prm = binding.Params(Hq, Hkv, topk=topk, n_init_blocks=1, n_local_blocks=0)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(71, seqlens, Hq, Hkv, n_planted=3)
    qd, kd, sl = to_dev(q), to_dev(k), dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, T)
    ws = torch.full((binding.workspace_bytes(binding.OP_SELECT_PREFILL, prm, len(seqlens), T),), fill, dtype=torch.uint8,
                    device="cuda")
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, sl, T, workspace=ws)
    torch.cuda.synchronize()
    ckb, idx_np = to_bits(ck), idx.cpu().numpy()
    near = 0
    for b, l in enumerate(seqlens):
        want, margins, R = ref.select_blocks(q[b, :l], ckb[b, :, :ref.num_kernels(l, 32, 16)], np.arange(l, dtype=np.int32),
                                             oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx_np[b, :, :l], want, margins, R)
        assert not hard, (b, hard[:3])
        near += nt
    assert near <= 2


@pytest.mark.parametrize("cap", [20000, 40000, 70000, 132000])
@pytest.mark.parametrize("Hq,Hkv,n_local,topk", [(16, 1, 2, 16), (16, 1, 0, 16), (4, 1, 1, 16), (16, 1, 1, 48), (16, 1, 1, 64)])
def test_select_blocks_prefill_long_capacity(Hq, Hkv, n_local, topk, cap):
    # the chunk of blocks pass 2 ranks at a time is chosen by the capacity of the buffers and by top-k (128,
    # 256 or 512 blocks; fewer when a wide top-k needs the on-chip memory); short sequences in long buffers
    # reach every variant
    seqlens = [5000, 257]
    prm = binding.Params(Hq, Hkv, topk=topk, n_init_blocks=1, n_local_blocks=n_local)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(83, seqlens, Hq, Hkv, n_planted=5)
    B = len(seqlens)
    qd = torch.zeros((B, cap, Hq, 128), dtype=torch.bfloat16, device="cuda")
    kd = torch.zeros((B, Hkv, cap, 128), dtype=torch.bfloat16, device="cuda")
    qd[:, :T].copy_(to_dev(q))
    kd[:, :, :T].copy_(to_dev(k))
    sl = dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, cap)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, sl, cap)
    torch.cuda.synchronize()
    ckb = to_bits(ck)
    near = 0
    for b, l in enumerate(seqlens):
        idx_b = idx[b, :, :l].cpu().numpy()
        assert bool((idx[b, :, l:] == -1).all())
        want, margins, R = ref.select_blocks(q[b, :l], ckb[b, :, :ref.num_kernels(l, 32, 16)], np.arange(l, dtype=np.int32),
                                             oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx_b, want, margins, R)
        assert not hard, (b, hard[:3])
        near += nt
    assert near <= 2


@pytest.mark.parametrize("l,Hq,Hkv,topk,n_local", [(40000, 16, 1, 16, 2),    # G = 16: chunks of 512 blocks, 2 chunks
                                                   (20000, 16, 1, 64, 1),    # wide top-k: chunks of 256 blocks
                                                   (36000, 4, 1, 16, 0),     # other group sizes: chunks of 256, 3 chunks
                                                   (17000, 2, 2, 8, 1),      # G = 1
                                                   (5000, 2, 2, 64, 1),      # G = 1, widest top-k: the most LDS a launch asks for
                                                   (5000, 4, 2, 64, 0)])     # G = 2, widest top-k
def test_select_blocks_prefill_rows_longer_than_one_chunk(l, Hq, Hkv, topk, n_local):
    # pass 2 ranks the block scores chunk by chunk inside the kernel and carries the running picks from
    # chunk to chunk: sequences long enough for several chunks, checked on sampled query rows (the rows
    # around the positions where a new chunk starts, the last rows, and random ones)
    print("case select prefill chunks", l, Hq, Hkv, topk, n_local, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk, n_init_blocks=1, n_local_blocks=n_local)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(91, [l], Hq, Hkv, n_planted=40)
    qd, kd, sl = to_dev(q), to_dev(k), dev_i32([l])
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, sl, T)
    torch.cuda.synchronize()
    rng = np.random.default_rng(5)
    pos = set(rng.integers(0, l, 150).tolist()) | set(range(l - 40, l))
    for edge in (256 * 64, 512 * 64):
        pos |= {p_ for p_ in range(edge - 70, edge + 200) if 0 <= p_ < l}
    pos = np.array(sorted(pos), np.int32)
    ckb = to_bits(ck)
    idx_np = idx[0].cpu().numpy()
    want, margins, R = ref.select_blocks(q[0, pos], ckb[0, :, :ref.num_kernels(l, 32, 16)], pos, oprm, want_scores=True)
    n, e, nt, hard = compare_selection(idx_np[:, pos], want, margins, R)
    print("rows %d exact %d near-tie %d" % (n, e, nt), flush=True)
    assert not hard, hard[:3]
    assert nt <= max(2, n // 200)


@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,planted", PREFILL_CASES)
def test_sparse_attn_prefill(seqlens, Hq, Hkv, topk, planted):
    print("case attn prefill", seqlens, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(21, seqlens, Hq, Hkv, n_planted=planted)
    # attention is checked in isolation: both sides consume the oracle's block sets
    idx_ref = np.full((len(seqlens), Hkv, T, topk), -1, np.int32)
    outs = []
    for b, l in enumerate(seqlens):
        if l == 0:
            outs.append(None)
            continue
        _, ckb = ref.compress_keys(k[b, :, :l], oprm)
        pos = np.arange(l, dtype=np.int32)
        idx_b, _ = ref.select_blocks(q[b, :l], ckb, pos, oprm)
        idx_ref[b, :, :l] = idx_b
        outs.append(ref.sparse_attn(q[b, :l], k[b, :, :l], v[b, :, :l], pos, idx_b, oprm))
    qd, kd, vd, sl = to_dev(q), to_dev(k), to_dev(v), dev_i32(seqlens)
    out = torch.full_like(qd, 3.0)
    lse = torch.full((len(seqlens), T, Hq), 5.0, dtype=torch.float32, device="cuda")
    binding.sparse_attn_prefill(prm, qd, kd, vd, sl, T, torch.from_numpy(idx_ref).cuda(), out=out, lse=lse)
    torch.cuda.synchronize()
    o = out.float().cpu().numpy().astype(np.float64)
    ls = lse.cpu().numpy().astype(np.float64)
    for b, l in enumerate(seqlens):
        if l:
            want_o, want_l = outs[b]
            eo = np.abs(o[b, :l] - want_o).max()
            el = lse_err(ls[b, :l], want_l)
            print("seq %d len %d: max|dO| %.3e LSE err/tol %.3f" % (b, l, eo, el), flush=True)
            assert eo <= OUT_TOL and el <= 1.0
        assert np.all(o[b, l:] == 3.0) and np.all(ls[b, l:] == 5.0)     # padding rows untouched


# One case on each side of every line of the attention's dispatch (tiles per wavefront, split over the waves or not,
# by tokens x key-value heads), per group size; ragged batches, odd lengths, a sequence shorter than a tile, and more
# than 2048 blocks (the union's bitmap takes two rounds there).
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [
    ([383], 16, 1, 16), ([385], 16, 1, 16), ([1023], 32, 2, 5), ([1025, 3], 32, 2, 16), ([8191], 32, 2, 8), ([8193, 700], 32, 2, 24),
    ([300], 16, 2, 16), ([771, 1], 16, 2, 16), ([2049], 16, 2, 64), ([700, 40], 8, 2, 16), ([1600], 8, 2, 33), ([4101, 65], 8, 2, 16),
    ([1500], 4, 2, 16), ([1601], 4, 2, 48), ([8201, 15], 4, 2, 16), ([3000], 2, 2, 16), ([3090, 31], 2, 2, 16), ([6500], 1, 1, 64),
    ([139333], 16, 1, 16), ([132001], 4, 1, 16)])
def test_sparse_attn_prefill_dispatch(seqlens, Hq, Hkv, topk):
    print("case attn prefill dispatch", seqlens, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    gen = torch.Generator(device="cuda").manual_seed(77)
    B, T = len(seqlens), max(seqlens)
    q = torch.randn((B, T, Hq, 128), device="cuda", generator=gen).bfloat16()
    k = torch.randn((B, Hkv, T, 128), device="cuda", generator=gen).bfloat16()
    v = torch.randn((B, Hkv, T, 128), device="cuda", generator=gen).bfloat16()
    # lists in no particular order: neighbours share most of their blocks, a few entries are their own, some are empty
    own = (torch.arange(T, device="cuda") // 64)[None, None, :, None]
    i = torch.arange(topk, device="cuda")[None, None, None, :]
    shift = torch.randint(0, 3, (B, Hkv, T, 1), device="cuda", generator=gen) * 3
    idx = (own + 1 - 7 * i - torch.where(i % 4 == 3, shift, torch.zeros_like(shift)))
    idx = torch.where((i % 5 == 4) | (idx < 0), torch.full_like(idx, -1), torch.where(i == 0, own.expand_as(idx), idx))
    idx = idx.flip(-1).to(torch.int32).contiguous()
    out, lse = torch.full_like(q, 3.0), torch.full((B, T, Hq), 5.0, dtype=torch.float32, device="cuda")
    binding.sparse_attn_prefill(prm, q, k, v, dev_i32(seqlens), T, idx, out=out, lse=lse)
    torch.cuda.synchronize()
    rng = np.random.default_rng(3)
    for b, l in enumerate(seqlens):
        pos = np.array(sorted(set(rng.integers(0, l, 60).tolist()) | set(range(max(0, l - 35), l)) | set(range(min(l, 5)))), np.int32)
        at = torch.from_numpy(pos).long().cuda()
        want_o, want_l = ref.sparse_attn(to_bits(q[b, at]), to_bits(k[b, :, :l]), to_bits(v[b, :, :l]), pos,
                                         idx[b, :, at].cpu().numpy(), oprm)
        eo = np.abs(out[b, at].double().cpu().numpy() - want_o).max()
        el = lse_err(lse[b, at].double().cpu().numpy(), want_l)
        print("len %d: max|dO| %.3e LSE err/tol %.3f" % (l, eo, el), flush=True)
        assert eo <= OUT_TOL and el <= 1.0
        assert bool((out[b, l:] == 3.0).all()) and bool((lse[b, l:] == 5.0).all())


@pytest.mark.parametrize("seqlens,T,Hq,Hkv", [([130, 0, 31, 77], 130, 32, 2), ([65, 200], 257, 4, 1), ([20, 3], 31, 8, 2)])
def test_results_made_by_the_call_are_clear_past_the_end(seqlens, T, Hq, Hkv):
    # tensors the binding allocates: rows of shorter sequences read 0 (block lists -1), whatever the memory held before
    print("case padding", seqlens, T, Hq, Hkv, flush=True)
    prm = binding.Params(Hq, Hkv, topk=8)
    B = len(seqlens)
    gen = torch.Generator(device="cuda").manual_seed(4)
    q = torch.randn((B, T, Hq, 128), device="cuda", generator=gen).bfloat16()
    k, v = (torch.randn((B, Hkv, T, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    dout = torch.randn((B, T, Hq, 128), device="cuda", generator=gen).bfloat16()
    sl = dev_i32(seqlens)

    def poison():                                        # the allocator hands these bytes out again
        junk = [torch.full((n,), 0x41, dtype=torch.uint8, device="cuda") for n in (1 << 14, 1 << 17, 1 << 20, 1 << 22, 1 << 24) for _ in range(4)]
        torch.cuda.synchronize()
        del junk

    poison()
    ck = binding.compress_keys(prm, k, sl, T)
    poison()
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, ck, sl, T)
    poison()
    out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx)
    poison()
    dq, dk, dv = binding.sparse_attn_bwd(prm, q, k, v, out, dout, lse, sl, T, idx)
    torch.cuda.synchronize()
    assert ck.shape == (B, Hkv, max(1, binding.num_kernels(T, prm)), 128) and idx.shape == (B, Hkv, T, 8)
    for b, l in enumerate(seqlens):
        assert bool((ck[b, :, binding.num_kernels(l, prm):] == 0).all())
        assert bool((idx[b, :, l:] == -1).all()) and bool((idx[b, :, :l, 0] >= 0).all())
        for t in (out[b, l:], lse[b, l:], dq[b, l:], dk[b, :, l:], dv[b, :, l:]):
            assert bool((t == 0).all())
    # and the same values as in the caller's own buffers
    out2, lse2 = torch.zeros_like(q), torch.zeros_like(lse)
    binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx, out=out2, lse=lse2)
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16)) and torch.equal(lse, lse2)
    with pytest.raises(binding.InfLLMv2Error, match="bf16"):
        binding.compress_keys(prm, k.float(), sl, T)
    with pytest.raises(binding.InfLLMv2Error, match="workspace"):
        binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx, workspace=torch.empty(8, dtype=torch.uint8, device="cuda"))


# Tensors with fewer rows than max_seqlen (a prompt's own queries beside caches of a larger capacity): the results, made like
# them by the binding, hold just those rows.  Nothing behind a sequence's last row is written: not the next sequence's rows,
# not the memory after the tensor.  Both forms of the attention (straight from the cache, packed), both tile counts of dq.
@pytest.mark.parametrize("rows,lens,T,Hq,Hkv", [(100, [100, 65], 300, 16, 1), (200, [1, 200], 257, 4, 2), (1000, [1000, 999], 2100, 16, 1)])
def test_results_made_by_the_call_end_with_the_tensor(rows, lens, T, Hq, Hkv):
    print("case short tensors", rows, lens, T, Hq, Hkv, flush=True)
    prm = binding.Params(Hq, Hkv, topk=8)
    B = len(lens)
    gen = torch.Generator(device="cuda").manual_seed(rows)
    q, do = (torch.randn((B, rows, Hq, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn((B, Hkv, rows, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    sl = dev_i32(lens)

    def padded(x, dim):                                  # the same rows in a tensor of max_seqlen
        y = torch.zeros(tuple(T if i == dim else n for i, n in enumerate(x.shape)), dtype=x.dtype, device="cuda")
        y.narrow(dim, 0, rows).copy_(x)
        return y

    ck = binding.compress_keys(prm, k, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, ck, sl, T)
    ws_f = torch.empty(binding.workspace_bytes(binding.OP_ATTN_PREFILL, prm, B, T), dtype=torch.uint8, device="cuda")
    ws_b = torch.empty(binding.workspace_bytes(binding.OP_ATTN_BWD, prm, B, T), dtype=torch.uint8, device="cuda")
    q2, do2, k2, v2 = padded(q, 1), padded(do, 1), padded(k, 2), padded(v, 2)
    want_out, want_lse = binding.sparse_attn_prefill(prm, q2, k2, v2, sl, T, idx, workspace=ws_f)
    want_dq, want_dk, want_dv = binding.sparse_attn_bwd(prm, q2, k2, v2, want_out, do2, want_lse, sl, T, idx, workspace=ws_b)
    assert torch.equal(idx, binding.select_blocks(prm, binding.MODE_PREFILL, q2, ck, sl, T))

    def holes(*sizes):                                   # gaps for the results, each with a known pattern right behind it
        guards, gaps = [], []
        for n in sizes:
            gaps.append(torch.empty((n,), dtype=torch.uint8, device="cuda"))
            guards.append(torch.full((1536 << 10 if n > 1 << 20 else 64 << 10,), 0x5a, dtype=torch.uint8, device="cuda"))
            assert guards[-1].data_ptr() - gaps[-1].data_ptr() == (n + 511) // 512 * 512
        torch.cuda.synchronize()
        return guards, [x.data_ptr() for x in gaps]

    pools = torch.cuda.MemPool(), torch.cuda.MemPool()
    with torch.cuda.use_mem_pool(pools[0]):
        guards, at = holes(q.numel() * 2, B * T * Hq * 4)
        out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx, workspace=ws_f)
        assert [x.data_ptr() for x in (out, lse)] == at
    with torch.cuda.use_mem_pool(pools[1]):
        more, at = holes(q.numel() * 2, k.numel() * 2, v.numel() * 2)
        dq, dk, dv = binding.sparse_attn_bwd(prm, q, k, v, out, do, lse, sl, T, idx, workspace=ws_b)
        assert [x.data_ptr() for x in (dq, dk, dv)] in (at, [at[0], at[2], at[1]])
    torch.cuda.synchronize()
    for x in guards + more:
        assert bool((x == 0x5a).all())
    for x, y, dim in ((out, want_out, 1), (dq, want_dq, 1), (dk, want_dk, 2), (dv, want_dv, 2)):
        assert x.shape == (q if dim == 1 else k).shape
        for b, l in enumerate(lens):
            a, w = x[b].narrow(dim - 1, 0, l), y[b].narrow(dim - 1, 0, l)
            if x is out or x is dq:
                assert torch.equal(a, w)
            else:                                        # summed with atomics: fp32 order, one bf16 rounding of the sum
                assert bool(((a.double() - w.double()).abs() <= 2.0 ** -7 * w.double().abs() + 1e-5).all())
            assert bool((x[b].narrow(dim - 1, l, rows - l) == 0).all())
    assert torch.equal(lse, want_lse)


def test_numbers_the_library_refuses_raise():
    # what the binding works out itself (result shapes) must not trip over them first: a stride of zero, more tokens than 32 bits hold
    k = torch.zeros((1, 1, 64, 128), dtype=torch.bfloat16, device="cuda")
    q = torch.zeros((1, 64, 4, 128), dtype=torch.bfloat16, device="cuda")
    sl = dev_i32([64])
    for bad in (dict(kernel_stride=0), dict(kernel_stride=-16), dict(kernel_size=0), dict(kernel_size=-(1 << 31)), dict(topk=0)):
        with pytest.raises(binding.InfLLMv2Error, match="invalid argument"):
            binding.compress_keys(binding.Params(4, 1, **bad), k, sl, 64)
    prm = binding.Params(4, 1, topk=4)
    ck = binding.compress_keys(prm, k, sl, 64)
    for T in ((1 << 32) + 64, 1 << 31, -(1 << 32) + 64):
        with pytest.raises(binding.InfLLMv2Error, match="32 bits"):
            binding.compress_keys(prm, k, sl, T)
        with pytest.raises(binding.InfLLMv2Error, match="32 bits"):
            binding.select_blocks(prm, binding.MODE_PREFILL, q, ck, sl, T)


def test_sparse_attn_prefill_row_that_repeats_a_block():
    # the contract asks for duplicate-free rows; a row that repeats a block all the same must stay inside
    # the caches and attend that block once: same output as the clean row, bit for bit
    print("case attn prefill duplicate entries", flush=True)
    l, Hq, Hkv, topk = 700, 32, 2, 16
    prm = binding.Params(Hq, Hkv, topk=topk)
    q, k, v, T = make_batch(29, [l], Hq, Hkv, n_planted=3)
    qd, kd, vd, sl = to_dev(q), to_dev(k), to_dev(v), dev_i32([l])
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, sl, T)
    out0, lse0 = binding.sparse_attn_prefill(prm, qd, kd, vd, sl, T, idx)
    dup = idx.clone()
    n_valid = (dup >= 0).sum(-1)                           # at most 11 blocks exist: every row has padding
    rows = n_valid < topk
    first = dup[..., 0]
    last_real = torch.gather(dup, -1, (n_valid - 1).clamp(min=0)[..., None].long())[..., 0]
    dup[..., topk - 1] = torch.where(rows, first, dup[..., topk - 1])          # repeat the lowest block at the end
    dup[..., topk - 2] = torch.where(rows & (n_valid < topk - 1), last_real, dup[..., topk - 2])   # and the highest
    out1, lse1 = binding.sparse_attn_prefill(prm, qd, kd, vd, sl, T, dup)
    torch.cuda.synchronize()
    assert torch.equal(out0.view(torch.int16), out1.view(torch.int16)) and torch.equal(lse0, lse1)


@pytest.mark.parametrize("rho", [2, 4])
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,planted,heavy", [([1077, 333], 32, 2, 16, 6, ()),
                                                               ([2500], 16, 1, 8, 5, ()),
                                                               ([1900, 130, 127, 64], 32, 2, 6, 3, (0,))])
def test_select_blocks_prefill_approximate_lse(seqlens, Hq, Hkv, topk, planted, heavy, rho):
    # the approximate log-sum-exp from coarse semantic kernels: same parity bar against the
    # oracle's definition of it; the recall against the exact selection is printed
    print("case approximate lse", seqlens, Hq, Hkv, topk, "rho", rho, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk, lse_coarse_ratio=rho)
    oprm = oracle_params(prm)
    exact = binding.Params(Hq, Hkv, topk=topk)
    q, k, v, T = make_batch(51, seqlens, Hq, Hkv, n_planted=planted, heavy=heavy)
    qd, kd, sl = to_dev(q), to_dev(k), dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, sl, T).cpu().numpy()
    idx_exact = binding.select_blocks(exact, binding.MODE_PREFILL, qd, ck, sl, T).cpu().numpy()
    ckb = to_bits(ck)
    tot = ex = near = 0
    same = picks = 0
    for b, l in enumerate(seqlens):
        n_c = ref.num_kernels(l, 32, 16)
        pos = np.arange(l, dtype=np.int32)
        want, margins, R = ref.select_blocks(q[b, :l], ckb[b, :, :n_c], pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx[b, :, :l], want, margins, R)
        assert not hard, hard[:3]
        tot, ex, near = tot + n, ex + e, near + nt
        for h in range(Hkv):
            for t in range(l):
                a = set(idx[b, h, t].tolist()) - {-1}
                same += len(a & (set(idx_exact[b, h, t].tolist()) - {-1}))
                picks += len(a)
    print("rows %d exact %d near-tie %d; blocks shared with the exact selection: %.4f" %
          (tot, ex, near, same / max(1, picks)), flush=True)
    assert near <= max(2, tot // 100)
    assert same / max(1, picks) > 0.9
    # decode with the same approximation: the row of the last token, bit for bit
    last = [max(l - 1, 0) for l in seqlens]
    q1 = np.stack([q[b, last[b]] for b in range(len(seqlens))])[:, None]
    idx_dec = binding.select_blocks(prm, binding.MODE_DECODE, to_dev(q1), ck, sl, T).cpu().numpy()
    for b, l in enumerate(seqlens):
        assert np.array_equal(idx_dec[b, :, 0], idx[b, :, l - 1]), b


def test_exact_ties_go_to_the_lower_block_index():
    # zero queries: every visible kernel gets the same probability, so every block score of a
    # row is the same number on both sides; the selection is decided by the tie rule alone
    print("case ties", flush=True)
    seqlens, Hq, Hkv, topk = [1300, 700], 32, 2, 8
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(41, seqlens, Hq, Hkv)
    q[:] = 0
    qd, kd, sl = to_dev(q), to_dev(k), dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, sl, T).cpu().numpy()
    last = [l - 1 for l in seqlens]
    q1 = np.stack([q[b, last[b]] for b in range(len(seqlens))])[:, None]
    idx_dec = binding.select_blocks(prm, binding.MODE_DECODE, to_dev(q1), ck, sl, T).cpu().numpy()
    ckb = to_bits(ck)
    for b, l in enumerate(seqlens):
        n_c = ref.num_kernels(l, 32, 16)
        want, _ = ref.select_blocks(q[b, :l], ckb[b, :, :n_c], np.arange(l, dtype=np.int32), oprm)
        assert np.array_equal(idx[b, :, :l], want)
        assert np.array_equal(idx_dec[b, :, 0], want[:, l - 1])
        # the rule itself: the scored picks are the lowest-numbered candidates with a visible kernel
        row = want[0, l - 1]
        assert row.tolist() == sorted(set(row.tolist())) and row[1] == 1 and row[topk - 4] == topk - 4


def test_sparse_attn_prefill_accepts_unsorted_block_lists():
    # the block list of a token is a set: any order, padding anywhere
    print("case unsorted lists", flush=True)
    l, Hq, Hkv, topk = 1100, 32, 2, 16
    prm, (q, k, v, T), (qd, kd, vd, sl), ck, idx = run_prefill([l], Hq, Hkv, topk, 4)
    out0, lse0 = binding.sparse_attn_prefill(prm, qd, kd, vd, sl, T, idx)
    rng = np.random.default_rng(5)
    shuffled = idx.cpu().numpy().copy()
    for h in range(Hkv):
        for t in range(l):
            rng.shuffle(shuffled[0, h, t])
    out1, lse1 = binding.sparse_attn_prefill(prm, qd, kd, vd, sl, T, torch.from_numpy(shuffled).cuda())
    torch.cuda.synchronize()
    # same set, same ascending processing order inside the kernel: identical results
    assert torch.equal(out0.view(torch.int16), out1.view(torch.int16)) and torch.equal(lse0, lse1)


def test_prefill_end_to_end_dense_degrade():
    # top-k covering every block: the whole path equals dense causal attention
    print("case dense degrade", flush=True)
    l, Hq, Hkv = 900, 32, 2
    prm, (q, k, v, T), (qd, kd, vd, sl), ck, idx = run_prefill([l], Hq, Hkv, 16, 0)
    out, lse = binding.sparse_attn_prefill(prm, qd, kd, vd, sl, T, idx)
    torch.cuda.synchronize()
    G = Hq // Hkv
    qt = torch.from_numpy(synth.bf16_bits_to_f32(q[0]).astype(np.float64)).permute(1, 0, 2)
    kt = torch.from_numpy(synth.bf16_bits_to_f32(k[0]).astype(np.float64)).repeat_interleave(G, 0)
    vt = torch.from_numpy(synth.bf16_bits_to_f32(v[0]).astype(np.float64)).repeat_interleave(G, 0)
    want = torch.nn.functional.scaled_dot_product_attention(qt, kt, vt, is_causal=True).permute(1, 0, 2)
    assert (out[0].double().cpu() - want).abs().max().item() <= OUT_TOL


# ------------------------------------------------------------------ decode

@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,forced", [
    ([3000, 1077, 64, 33, 31, 1], 32, 2, 16, (1, 2)),
    ([2048, 129], 4, 1, 8, (1, 2)), ([777], 16, 2, 6, (1, 2)),
    ([9000, 4500, 200], 32, 2, 64, (1, 2)),
    ([4100, 4097, 20], 32, 2, 16, (1, 2)),                  # 65 blocks, 255 kernels
    ([4100, 4097, 4128, 20, 70], 32, 2, 16, (0, 0)),        # nothing forced: the query's own (short) block competes
])
def test_decode_select_and_attn(seqlens, Hq, Hkv, topk, forced):
    print("case decode", seqlens, Hq, Hkv, topk, forced, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk, n_init_blocks=forced[0], n_local_blocks=forced[1])
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(31, seqlens, Hq, Hkv, n_planted=4, heavy=(1,))
    B = len(seqlens)
    last = np.array([l - 1 for l in seqlens])
    q1 = np.stack([q[b, last[b]] for b in range(B)])[:, None]            # [B,1,Hq,d]
    qd, kd, vd, sl = to_dev(q1), to_dev(k), to_dev(v), dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_DECODE, qd, ck, sl, T)
    torch.cuda.synchronize()
    idx_np = idx.cpu().numpy()
    ckb = to_bits(ck)
    idx_ref = np.full((B, Hkv, 1, topk), -1, np.int32)
    want = []
    for b, l in enumerate(seqlens):
        pos = np.array([l - 1], np.int32)
        n_c = ref.num_kernels(l, 32, 16)
        ib, margins, R = ref.select_blocks(q1[b], ckb[b, :, :n_c], pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx_np[b], ib, margins, R)
        assert not hard, (b, hard)
        idx_ref[b] = ib
        want.append(ref.sparse_attn(q1[b], k[b, :, :l], v[b, :, :l], pos, ib, oprm))
    out, lse = binding.sparse_attn_decode(prm, qd, kd, vd, sl, T, torch.from_numpy(idx_ref).cuda())
    torch.cuda.synchronize()
    for b in range(B):
        eo = np.abs(out[b].double().cpu().numpy() - want[b][0]).max()
        el = lse_err(lse[b].double().cpu().numpy(), want[b][1][0])
        print("seq %d len %d: max|dO| %.3e LSE err/tol %.3f" % (b, seqlens[b], eo, el), flush=True)
        assert eo <= OUT_TOL and el <= 1.0


@pytest.mark.parametrize("fused", [False, True, "one call"])
def test_decode_steps_with_append_and_incremental_compress(fused):
    # a short run of real decode steps: append, incremental compression (its own launch, or
    # inside the append), select, attend; every step equals the oracle on the cache as it stands
    print("case decode steps, fused append+compress:", fused, flush=True)
    cfg = synth.CONFIGS[3]
    steps, L0 = 40, 1500
    x = synth.make_decode(cfg, steps=steps, seqlen=L0)
    prm = binding.Params(cfg.n_q_heads, cfg.n_kv_heads, topk=cfg.topk)
    oprm = oracle_params(prm)
    cap = x.capacity
    kd, vd = to_dev(x.k_cache), to_dev(x.v_cache)
    lens = x.seqlens0.copy()
    sl = dev_i32(lens)
    ck = binding.compress_keys(prm, kd, sl, cap)
    k_np, v_np = x.k_cache.copy(), x.v_cache.copy()
    for s in range(steps):
        lens = lens + 1
        sl = dev_i32(lens)
        kn = to_dev(x.k_steps[s][:, :, None])
        vn = to_dev(x.v_steps[s][:, :, None])
        qd = to_dev(x.q_steps[s][:, None])
        if fused == "one call":                               # the whole step behind one entry point, five launches
            idx, out, lse = binding.decode_step(prm, qd, kn, vn, kd, vd, ck, sl, cap)
        else:
            if fused:
                binding.append_kv(prm, kn, vn, kd, vd, sl, cap, ck=ck)
            else:
                binding.append_kv(prm, kn, vn, kd, vd, sl, cap)
                binding.compress_keys(prm, kd, sl, cap, ck=ck, n_new_tokens=1)
            idx = binding.select_blocks(prm, binding.MODE_DECODE, qd, ck, sl, cap)
            out, lse = binding.sparse_attn_decode(prm, qd, kd, vd, sl, cap, idx)
        torch.cuda.synchronize()
        l = int(lens[0])
        k_np[0, :, l - 1] = x.k_steps[s][0]
        v_np[0, :, l - 1] = x.v_steps[s][0]
        if s % 8 == 0 or s == steps - 1 or (l - 32) % 16 == 0:
            pos = np.array([l - 1], np.int32)
            _, ckb = ref.compress_keys(k_np[0, :, :l], oprm)
            assert np.array_equal(to_bits(ck)[0, :, :ckb.shape[1]], ckb)
            ib, margins, R = ref.select_blocks(x.q_steps[s][0][None], ckb, pos, oprm, want_scores=True)
            n, e, nt, hard = compare_selection(idx.cpu().numpy()[0], ib, margins, R)
            assert not hard, (s, hard)
            if nt == 0:
                wo, wl = ref.sparse_attn(x.q_steps[s][0][None], k_np[0, :, :l], v_np[0, :, :l], pos, ib, oprm)
                assert np.abs(out[0].double().cpu().numpy() - wo).max() <= OUT_TOL
                assert lse_err(lse[0].double().cpu().numpy(), wl[0]) <= 1.0
    assert torch.equal(kd.view(torch.int16).cpu(), torch.from_numpy(k_np.view(np.int16)))


# ------------------------------------------------------------------ draft verification (section 4.1)

def tree_masks(rng, n, kind):
    """uint64 mask words of n drafted tokens: 'chain', a random 'tree' (node 0 the root, each word
    the node's ancestors and itself) or 'holes' (a tree with some words emptied or cut down)."""
    if kind == "chain":
        return np.array([(1 << (t + 1)) - 1 for t in range(n)], np.uint64)
    parent = [-1] + [int(rng.integers(0, t)) for t in range(1, n)]
    words = []
    for t in range(n):
        w, a = 0, t
        while a >= 0:
            w |= 1 << a
            a = parent[a]
        words.append(w)
    if kind == "holes":
        for t in range(0, n, 3):
            words[t] = 0 if t % 2 else words[t] & ~(1 << t)          # nothing / no self bit
        words[n - 1] |= 1 << (n - 1)
        if n > 2:
            words[1] |= 1 << (n - 1)                                  # a later draft token: allowed inside selected blocks
    return np.array(words, np.uint64)


def dev_masks(m):
    return torch.from_numpy(np.ascontiguousarray(m).view(np.int64)).cuda()


@pytest.mark.parametrize("seqlens,n,Hq,Hkv,topk,kind", [
    ([1500, 700, 69, 8, 3, 0], 8, 32, 2, 16, "chain"),
    ([2100, 16, 130, 1029], 16, 32, 2, 16, "tree"),
    ([900, 64, 100, 4160], 64, 16, 2, 8, "tree"),
    ([333, 1], 1, 8, 2, 4, "tree"),
    ([1300, 40, 24, 200], 24, 32, 2, 16, "holes"),
    ([520, 513], 5, 4, 1, 6, "holes"),
    ([4096, 2049, 1025], 7, 2, 2, 8, "tree"),
])
def test_verify_select_and_attn(seqlens, n, Hq, Hkv, topk, kind):
    print("case verify", seqlens, n, Hq, Hkv, topk, kind, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(41, seqlens, Hq, Hkv, n_planted=4, heavy=(1,))
    B = len(seqlens)
    rng = np.random.default_rng(5)
    qn = np.zeros((B, n, Hq, 128), np.uint16)
    masks = np.zeros((B, n), np.uint64)
    for b, l in enumerate(seqlens):
        masks[b] = tree_masks(rng, n, kind)
        if l >= n:
            qn[b] = q[b, l - n:l]
    qd, kd, vd, sl = to_dev(qn), to_dev(k), to_dev(v), dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks_verify(prm, qd, ck, sl, T)
    torch.cuda.synchronize()
    idx_np = idx.cpu().numpy()
    assert idx_np.shape == (B, Hkv, n, topk)
    ckb = to_bits(ck)
    idx_ref = np.full((B, Hkv, n, topk), -1, np.int32)
    want = [None] * B
    for b, l in enumerate(seqlens):
        if l < n:                                                     # skipped as a whole
            assert np.all(idx_np[b] == -1)
            continue
        pos = np.arange(l - n, l, dtype=np.int32)
        n_c = ref.num_kernels(l, 32, 16)
        ib, margins, R = ref.select_blocks(qn[b], ckb[b, :, :n_c], pos, oprm, want_scores=True)
        rows, e, nt, hard = compare_selection(idx_np[b], ib, margins, R)
        assert not hard, (b, hard)
        idx_ref[b] = ib
        want[b] = ref.sparse_attn_tree(qn[b], k[b, :, :l], v[b, :, :l], ib, masks[b], l - n, oprm)
        if kind == "chain":                                           # the chain is the causal prefill rows
            wc = ref.sparse_attn(qn[b], k[b, :, :l], v[b, :, :l], pos, ib, oprm)
            assert np.array_equal(want[b][0], wc[0]) and np.array_equal(want[b][1], wc[1])
    idx_d = torch.from_numpy(idx_ref).cuda()
    out, lse = binding.sparse_attn_verify(prm, qd, kd, vd, sl, T, idx_d, tree_mask=dev_masks(masks))
    torch.cuda.synchronize()
    if kind == "chain":                                               # no mask = the chain, bit for bit
        out2, lse2 = binding.sparse_attn_verify(prm, qd, kd, vd, sl, T, idx_d)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), out2.view(torch.int16)) and torch.equal(lse, lse2)
    for b, l in enumerate(seqlens):
        o, ls = out[b].double().cpu().numpy(), lse[b].double().cpu().numpy()
        if l < n:
            assert np.all(o == 0) and np.all(np.isneginf(ls))
            continue
        wo, wl = want[b]
        empty = np.isneginf(wl)
        assert np.array_equal(np.isneginf(ls), empty)                 # rows whose mask hides every key
        assert np.all(o[empty] == 0)
        eo = np.abs(o - wo).max()
        el = lse_err(ls[~empty], wl[~empty])
        print("seq %d len %d: max|dO| %.3e LSE err/tol %.3f, %d empty rows" % (b, l, eo, el, int(empty.sum())),
              flush=True)
        assert eo <= OUT_TOL and el <= 1.0


# The two forms in which the scoring workgroups hand on what they found, on either side of their line (lists that fit the scratch of the rows'
# scores and the second partials, or those scores): 26 | 27 picks beside the forced blocks for lists of 32, 40 | 41 for the lists of 64
# that a larger call has; G = 16, whose lists always fit; either side of 65536 tokens, beyond which half as many workgroups do for the larger lists.
@pytest.mark.parametrize("seqlens,n,Hq,Hkv,topk", [
    ([4500, 2100], 5, 4, 1, 29), ([4500, 2100], 5, 4, 1, 30), ([4500, 4160], 64, 16, 4, 43), ([4500, 4160], 64, 16, 4, 44),
    ([8300, 4100], 3, 4, 1, 64), ([8300, 4100], 6, 32, 2, 64), ([65537], 29, 2, 1, 8), ([65536], 30, 2, 1, 8)])
def test_verify_selection_lists_and_rows(seqlens, n, Hq, Hkv, topk):
    test_verify_select_and_attn(seqlens, n, Hq, Hkv, topk, "tree")


def test_verify_append_writes_rows_and_completed_kernels():
    print("case verify append", flush=True)
    Hkv, n = 2, 12
    prm = binding.Params(32, Hkv)
    seqlens = [1000, 44, 32, 12, 7, 0]                                # 7 and 0: shorter than n, untouched
    q, k, v, T = make_batch(43, seqlens, 32, Hkv)
    B = len(seqlens)
    k0, v0 = k.copy(), v.copy()
    kn = np.zeros((B, Hkv, n, 128), np.uint16)
    vn = np.zeros((B, Hkv, n, 128), np.uint16)
    for b, l in enumerate(seqlens):
        if l >= n:
            kn[b], vn[b] = k[b, :, l - n:l], v[b, :, l - n:l]
            k0[b, :, l - n:l] = 0
            v0[b, :, l - n:l] = 0
    kd, vd = to_dev(k0), to_dev(v0)
    before = dev_i32([max(l - n, 0) if l >= n else l for l in seqlens])
    n_cap = binding.num_kernels(T, prm) + 2
    ck = torch.full((B, Hkv, n_cap, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    binding.compress_keys(prm, kd, before, T, ck=ck)
    binding.append_kv_verify(prm, to_dev(kn), to_dev(vn), kd, vd, dev_i32(seqlens), T, ck=ck)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(kd), k) and np.array_equal(to_bits(vd), v)
    got = to_bits(ck)
    for b, l in enumerate(seqlens):
        _, w = ref.compress_keys(k[b, :, :l], oracle_params(prm))
        assert np.array_equal(got[b, :, :w.shape[1]], w), (b, l)


# One call against its parts, bit for bit: new kernels on either side of a workgroup's 128, caches no longer than the draft, a length
# beyond the cache, both widths of the scoring workgroups; buffers (three longer than the longest) of up to 4096 tokens, whose rows one kernel
# scores, on either side of the workgroups up to which it attends as well; longer ones on either side of those up to which every workgroup ranks, fewer
# beyond 131072 tokens, whose lists are more than are merged; chunks of kernels in columns of their number and of a multiple of eight, up to 16 tiles of
# four drafted tokens and beyond, and up to 768 workgroups.
@pytest.mark.parametrize("seqlens,n,Hq,Hkv,topk,rho", [
    ([2080, 2079, 2096, 4128, 31], 33, 32, 2, 16, 1), ([2081, 2, 33, 1], 2, 4, 1, 6, 1), ([4200, 64, 95, 63, 9999], 64, 16, 2, 64, 1),
    ([3000, 2090], 16, 16, 1, 24, 2), ([1021], 32, 32, 2, 16, 1), ([1021], 33, 8, 2, 16, 1), ([4093], 16, 32, 2, 16, 1),
    ([4093, 20], 17, 2, 1, 32, 1), ([4094], 16, 32, 2, 16, 1), ([5000], 64, 8, 2, 16, 1), ([5000], 64, 8, 2, 17, 1), ([5000], 42, 4, 1, 24, 1),
    ([5000], 43, 4, 1, 24, 1), ([131069], 64, 4, 1, 17, 1), ([131070], 64, 4, 1, 16, 1), ([131070], 64, 4, 1, 17, 1),
    ([20000], 32, 4, 2, 8, 1), ([20000, 19990], 20, 4, 2, 8, 1), ([98000], 32, 2, 2, 8, 1), ([100000], 32, 2, 2, 8, 1)])
def test_verify_step_equals_its_parts(seqlens, n, Hq, Hkv, topk, rho):
    print("case verify step", seqlens, n, Hq, Hkv, topk, rho, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk, lse_coarse_ratio=rho)
    gen = torch.Generator(device="cuda").manual_seed(12)
    B, T = len(seqlens), max(x for x in seqlens if x != 9999) + 3
    q = torch.randn((B, n, Hq, 128), device="cuda", generator=gen).bfloat16()
    kn, vn = (torch.randn((B, Hkv, n, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn((B, Hkv, T, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    sl = dev_i32(seqlens)
    ck = torch.full((B, Hkv, binding.num_kernels(T, prm), 128), 5.0, dtype=torch.bfloat16, device="cuda")
    binding.compress_keys(prm, k, dev_i32([x - n if n <= x <= T else min(x, T) for x in seqlens]), T, ck=ck)
    masks = dev_masks(np.stack([tree_masks(np.random.default_rng(3 + b), n, "tree") for b in range(B)]))
    parts, step = [x.clone() for x in (k, v, ck)], [x.clone() for x in (k, v, ck)]
    binding.append_kv_verify(prm, kn, vn, parts[0], parts[1], sl, T, ck=parts[2])
    idx = binding.select_blocks_verify(prm, q, parts[2], sl, T)
    out, lse = binding.sparse_attn_verify(prm, q, parts[0], parts[1], sl, T, idx, tree_mask=masks)
    got = binding.verify_step(prm, q, kn, vn, *step, sl, T, tree_mask=masks)
    torch.cuda.synchronize()
    for a, b in zip(parts + [idx, out, lse], step + list(got)):
        assert torch.equal(a.view(torch.int16) if a.dtype == torch.bfloat16 else a, b.view(torch.int16) if b.dtype == torch.bfloat16 else b)


# ------------------------------------------------------------------ backward of the sparse attention

@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,planted", [
    ([1077, 333], 32, 2, 16, 6),     # G = 16, ragged tails, two sequences
    ([700], 16, 2, 6, 3),            # G = 8
    ([300, 64, 63, 1, 0], 4, 2, 4, 0),  # G = 2, tiny and empty sequences
    ([450], 2, 2, 5, 2),             # G = 1
    ([1500], 16, 1, 32, 5),          # everything selected: dense causal attention
    ([2500], 32, 2, 8, 4),           # blocks whose members make many work items
])
def test_sparse_attn_backward(seqlens, Hq, Hkv, topk, planted):
    print("case attn backward", seqlens, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(51, seqlens, Hq, Hkv, n_planted=planted)
    B = len(seqlens)
    rng = np.random.default_rng(9)
    do = synth.f32_to_bf16_bits(rng.standard_normal((B, T, Hq, 128), dtype=np.float32))
    idx_ref = np.full((B, Hkv, T, topk), -1, np.int32)
    want = [None] * B
    for b, l in enumerate(seqlens):
        if l == 0:
            continue
        _, ckb = ref.compress_keys(k[b, :, :l], oprm)
        pos = np.arange(l, dtype=np.int32)
        ib, _ = ref.select_blocks(q[b, :l], ckb, pos, oprm)
        idx_ref[b, :, :l] = ib
        want[b] = ref.sparse_attn_bwd(q[b, :l], k[b, :, :l], v[b, :, :l], do[b, :l], pos, ib, oprm, want_mag=True)
    qd, kd, vd, dod, sl = to_dev(q), to_dev(k), to_dev(v), to_dev(do), dev_i32(seqlens)
    idx_d = torch.from_numpy(idx_ref).cuda()
    out, lse = binding.sparse_attn_prefill(prm, qd, kd, vd, sl, T, idx_d)
    sentinel = 3.0
    dq = torch.full_like(qd, sentinel)
    dk = torch.full_like(kd, sentinel)
    dv = torch.full_like(vd, sentinel)
    binding.sparse_attn_bwd(prm, qd, kd, vd, out, dod, lse, sl, T, idx_d, dq=dq, dk=dk, dv=dv)
    torch.cuda.synchronize()
    dq, dk, dv = dq.double().cpu().numpy(), dk.double().cpu().numpy(), dv.double().cpu().numpy()
    for b, l in enumerate(seqlens):
        assert np.all(dq[b, l:] == sentinel) and np.all(dk[b, :, l:] == sentinel) and np.all(dv[b, :, l:] == sentinel)
        if l == 0:
            continue
        wq, wk, wv, mq, mk, mv = want[b]
        eq, ek, ev = grad_err(dq[b, :l], wq, mq), grad_err(dk[b, :, :l], wk, mk), grad_err(dv[b, :, :l], wv, mv)
        print("seq %d len %d: err/tol dq %.3f dk %.3f dv %.3f   (max|dq| %.2e max|dk| %.2e max|dv| %.2e)"
              % (b, l, eq, ek, ev, np.abs(wq).max(), np.abs(wk).max(), np.abs(wv).max()), flush=True)
        assert eq <= 1.0 and ek <= 1.0 and ev <= 1.0


def test_results_made_by_the_call_are_clear_beyond_the_heads():
    # tensors with more heads than the parameters say: what no kernel visits reads 0 in the results the binding allocates
    Hq, Hkv, T = 4, 2, 300
    prm = binding.Params(Hq, Hkv, topk=8)
    gen = torch.Generator(device="cuda").manual_seed(6)
    q, do = (torch.randn((1, T, Hq + 2, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn((2, Hkv + 1, T, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    sl = dev_i32([T])
    junk = [torch.full((n,), 0x41, dtype=torch.uint8, device="cuda") for n in (1 << 17, 1 << 20, 1 << 22, 1 << 24) for _ in range(8)]
    torch.cuda.synchronize()
    del junk                                             # the allocator hands these bytes out again
    ck = binding.compress_keys(prm, k[:1], sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, ck, sl, T)
    out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx)
    dq, dk, dv = binding.sparse_attn_bwd(prm, q, k, v, out, do, lse, sl, T, idx)
    o1 = binding.sparse_attn_decode(prm, q[:, -1:], k, v, sl, T, idx[:, :, -1:].contiguous())[0]
    o2 = binding.sparse_attn_verify(prm, q[:, -2:], k, v, sl, T, idx[:, :, -2:].contiguous())[0]
    torch.cuda.synchronize()
    for t in (ck[:, Hkv:], out[:, :, Hq:], dq[:, :, Hq:], dk[:, Hkv:], dv[:, Hkv:], dk[1:], dv[1:], o1[:, :, Hq:], o2[:, :, Hq:]):
        assert bool((t == 0).all())


# Lists in no particular order with holes, most with the first block: each side of the lines of the backward's dispatch (tiles per workgroup by
# tokens x key-value heads), per group size; more than 2048 blocks (the membership words are built in rounds).
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [
    ([383], 16, 1, 16), ([385], 16, 1, 8), ([1025, 3], 32, 2, 16), ([770, 65], 8, 1, 16), ([2050], 16, 2, 24), ([1537], 4, 1, 64),
    ([4100], 8, 2, 8), ([3080, 31], 2, 1, 16), ([8200], 4, 2, 5), ([3080, 1], 2, 2, 33), ([132001], 1, 1, 3)])
def test_sparse_attn_backward_dispatch(seqlens, Hq, Hkv, topk):
    print("case attn backward dispatch", seqlens, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    gen = torch.Generator(device="cuda").manual_seed(78)
    B, T = len(seqlens), max(seqlens)
    q, do = (torch.randn((B, T, Hq, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn((B, Hkv, T, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    own = (torch.arange(T, device="cuda") // 64)[None, None, :, None]
    i = torch.arange(topk, device="cuda")[None, None, None, :]
    shift = torch.randint(0, 3, (B, Hkv, T, 1), device="cuda", generator=gen) * 3
    idx = (own + 1 - 7 * i - torch.where(i % 4 == 3, shift, torch.zeros_like(shift)))
    idx = torch.where((i % 5 == 4) | (idx < 0), torch.full_like(idx, -1), torch.where(i == 0, own.expand_as(idx), idx))
    idx = torch.where((own > 0) & (idx <= 0), torch.where((i == topk - 1).expand_as(idx), torch.zeros_like(idx), torch.full_like(idx, -1)), idx)
    idx = idx.flip(-1).to(torch.int32).contiguous()
    sl = dev_i32(seqlens)
    out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx)
    dq, dk, dv = torch.full_like(q, 3.0), torch.full_like(k, 3.0), torch.full_like(v, 3.0)
    binding.sparse_attn_bwd(prm, q, k, v, out, do, lse, sl, T, idx, dq=dq, dk=dk, dv=dv)
    torch.cuda.synchronize()
    for b, l in enumerate(seqlens):
        pos = np.arange(l, dtype=np.int32)
        wq, wk, wv, mq, mk, mv = ref.sparse_attn_bwd(to_bits(q[b, :l]), to_bits(k[b, :, :l]), to_bits(v[b, :, :l]), to_bits(do[b, :l]),
                                                     pos, idx[b, :, :l].cpu().numpy(), oprm, want_mag=True)
        eq = grad_err(dq[b, :l].double().cpu().numpy(), wq, mq)
        ek = grad_err(dk[b, :, :l].double().cpu().numpy(), wk, mk)
        ev = grad_err(dv[b, :, :l].double().cpu().numpy(), wv, mv)
        print("seq %d len %d: err/tol dq %.3f dk %.3f dv %.3f" % (b, l, eq, ek, ev), flush=True)
        assert eq <= 1.0 and ek <= 1.0 and ev <= 1.0
        assert bool((dq[b, l:] == 3.0).all()) and bool((dk[b, :, l:] == 3.0).all()) and bool((dv[b, :, l:] == 3.0).all())


# The scatter's work items: more slices than a queue has bins (a bin is part of a window, or several), and the first word of a second
# segment of 8192 tokens.
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([200 - 6 * i for i in range(33)], 2, 2, 4), ([8193, 8192, 8161], 16, 1, 3),
                                                 ([65 - i % 61 for i in range(130)], 2, 2, 3)])
def test_sparse_attn_backward_items(seqlens, Hq, Hkv, topk):
    test_sparse_attn_backward_dispatch(seqlens, Hq, Hkv, topk)


# Items sized by the tokens of the whole call: more sequences than the workgroup that counts them has threads, and one long one among
# short and empty ones, which then has more than its part of the items (whole words of 32 tokens, and less than that).
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([90 - i % 90 for i in range(300)], 4, 1, 3), ([3000] + [40, 0] * 6, 16, 1, 12),
                                                 ([2100, 70, 0, 500, 1], 16, 2, 16)])
def test_sparse_attn_backward_items_of_ragged_batches(seqlens, Hq, Hkv, topk):
    test_sparse_attn_backward_dispatch(seqlens, Hq, Hkv, topk)


# Items of an equal part of a share beyond 64 steps: 2 x 35 of 69 (70 members, less than whole words), 2 x 40 of 80 (ten whole words).
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([2100], 32, 2, 33), ([5000], 8, 2, 64)])
def test_sparse_attn_backward_items_of_large_shares(seqlens, Hq, Hkv, topk):
    test_sparse_attn_backward_dispatch(seqlens, Hq, Hkv, topk)


# Short calls, whose workgroups find their item by number: four parts of an item (more than it has steps: 2), two and one, of odd and even numbers
# of steps (two pairs of wavefronts take half each); windows of one to eight queues; just past eight windows, from the queues again.
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([40], 1, 1, 8), ([1], 2, 2, 3), ([260, 65], 16, 1, 8), ([1000, 900, 65, 7], 2, 1, 4),
                                                 ([1100], 16, 1, 16), ([700], 16, 2, 6), ([333], 8, 2, 16), ([8000], 1, 1, 8), ([8200], 1, 1, 8)])
def test_sparse_attn_backward_items_by_number(seqlens, Hq, Hkv, topk):
    test_sparse_attn_backward_dispatch(seqlens, Hq, Hkv, topk)


# Either side of the share up to which an item has two pairs of wavefronts (64 steps: 32 blocks x 64 steps of a call's 32768 rows each).
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([4096], 16, 1, 32), ([4097], 16, 1, 32), ([2048, 2048], 8, 1, 64), ([2049, 64], 8, 1, 64)])
def test_sparse_attn_backward_pairs(seqlens, Hq, Hkv, topk):
    test_sparse_attn_backward_dispatch(seqlens, Hq, Hkv, topk)


# Lists in which all blocks are equally popular, so that their items end at the same tokens: more than a bin holds (47 of 1125 items, 42 of
# 462, where a bin has three places and a window's tails), the rest from the list behind the queues.
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([10000], 2, 1, 16), ([1969, 1969], 6, 3, 3)])
def test_sparse_attn_backward_items_beyond_their_bin(seqlens, Hq, Hkv, topk):
    print("case attn backward bins", seqlens, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    gen = torch.Generator(device="cuda").manual_seed(79)
    B, T = len(seqlens), max(seqlens)
    q, do = (torch.randn((B, T, Hq, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn((B, Hkv, T, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    t = torch.arange(T)
    n = torch.clamp(t // 64 + 1, max=topk)
    i = torch.arange(topk)[None]
    idx = torch.where(i < n[:, None], ((t * n)[:, None] + i) % (t // 64 + 1)[:, None], -1)
    idx = idx.to(torch.int32)[None, None].expand(B, Hkv, T, topk).contiguous().cuda()
    sl = dev_i32(seqlens)
    out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx)
    dq, dk, dv = binding.sparse_attn_bwd(prm, q, k, v, out, do, lse, sl, T, idx)
    torch.cuda.synchronize()
    for b, l in enumerate(seqlens):
        wq, wk, wv, mq, mk, mv = ref.sparse_attn_bwd(to_bits(q[b, :l]), to_bits(k[b, :, :l]), to_bits(v[b, :, :l]), to_bits(do[b, :l]),
                                                     np.arange(l, dtype=np.int32), idx[b, :, :l].cpu().numpy(), oprm, want_mag=True)
        for got, want, mag in ((dq[b, :l], wq, mq), (dk[b, :, :l], wk, mk), (dv[b, :, :l], wv, mv)):
            assert grad_err(got.double().cpu().numpy(), want, mag) <= 1.0


# Walks that begin inside the list (from block 128 on): lists shorter than the workgroups that share an XCD are many, tiles of one and of
# several tokens, wavefronts that work alone and that split the list.  The gradients take the forward's out and lse in.
@pytest.mark.parametrize("seqlens,Hq,Hkv,topk", [([9001, 8400], 16, 1, 16), ([8500], 16, 1, 3), ([8450], 8, 1, 4), ([8777], 2, 1, 7)])
def test_sparse_attn_beyond_one_l2(seqlens, Hq, Hkv, topk):
    test_sparse_attn_backward_dispatch(seqlens, Hq, Hkv, topk)


# Longer buffers and other sequences beside it change no bit of a sequence's output and dq: where a walk begins and the order of its sums follow the
# token alone (wavefronts that work alone and that split the list, one and several tokens a tile).  What lies behind the end reads 0.
@pytest.mark.parametrize("l,others,cap,Hq,Hkv,topk", [
    (8777, [], 12345, 32, 2, 16), (8777, [9001, 64], 9100, 32, 2, 16), (8450, [300], 20000, 8, 1, 8), (8601, [], 131072, 4, 1, 12),
    (8300, [8200], 8999, 2, 2, 5), (4100, [500], 131072, 16, 2, 16)])
def test_results_do_not_depend_on_the_capacity(l, others, cap, Hq, Hkv, topk):
    print("case capacity", l, others, cap, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    gen = torch.Generator(device="cuda").manual_seed(l)
    T = (l + 63) // 64 * 64
    q, do = (torch.randn((1, T, Hq, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn((1, Hkv, T, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    sl = dev_i32([l])
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, binding.compress_keys(prm, k, sl, T), sl, T)
    out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx)
    want = out[0, :l], lse[0, :l], binding.sparse_attn_bwd(prm, q, k, v, out, do, lse, sl, T, idx)[0][0, :l]

    def longer(x, axis, fill=0):                           # the sequence among the others, last
        shape = list(x.shape)
        shape[0], shape[axis] = len(others) + 1, cap
        t = torch.full(shape, fill, dtype=x.dtype, device="cuda")
        for b, n in enumerate(others + [l]):
            t[b].narrow(axis - 1, 0, n).copy_(x[0].narrow(axis - 1, 0, min(n, T)) if n <= T else
                                              torch.cat([x[0], x[0]], axis - 1).narrow(axis - 1, 0, n))
        return t

    q, do, k, v, idx = longer(q, 1), longer(do, 1), longer(k, 2), longer(v, 2), longer(idx, 2, -1)
    lens = others + [l]
    out, lse = binding.sparse_attn_prefill(prm, q, k, v, dev_i32(lens), cap, idx)
    dq = binding.sparse_attn_bwd(prm, q, k, v, out, do, lse, dev_i32(lens), cap, idx)[0]
    torch.cuda.synchronize()
    for a, b in zip(want, (out[-1, :l], lse[-1, :l], dq[-1, :l])):
        assert torch.equal(a, b)
    for b, n in enumerate(lens):
        assert not bool(out[b, n:].any()) and not bool(lse[b, n:].any()) and not bool(dq[b, n:].any())


# The log-sum-exps against 64 bits: no more than the rounding of the results themselves (0.29 units in the last place, root mean square) and as much
# again for the sums; walks from the first block and, from 8192 tokens on, from inside the list; every form of the kernel.
@pytest.mark.parametrize("T,Hq,Hkv,topk", [(777, 32, 2, 8), (3000, 16, 1, 16), (12000, 32, 2, 16), (9000, 16, 2, 16), (9000, 4, 1, 12), (9000, 2, 2, 8)])
def test_log_sum_exps_are_as_near_as_fp32_allows(T, Hq, Hkv, topk):
    print("case lse", T, Hq, Hkv, topk, flush=True)
    prm, G = binding.Params(Hq, Hkv, topk=topk), Hq // Hkv
    gen = torch.Generator(device="cuda").manual_seed(T)
    q = torch.randn((1, T, Hq, 128), device="cuda", generator=gen).bfloat16()
    k, v = (torch.randn((1, Hkv, T, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    u = q[0].float().mean(0).reshape(Hkv, G, 128).mean(1)
    for j in range(2, T // 64 - 3, 16):                    # some blocks of keys along the mean query
        k[0, :, 64 * j:64 * j + 64] = (128 ** 0.5 * (u / u.norm(dim=-1, keepdim=True))[:, None] + 0.1 * k[0, :, 64 * j:64 * j + 64]).bfloat16()
    sl = dev_i32([T])
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, binding.compress_keys(prm, k, sl, T), sl, T)
    lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx)[1][0].double()
    err = []
    for t in range(T // 3, T, T // 150):
        for h in range(Hkv):
            b = idx[0, h, t][idx[0, h, t] >= 0].long()
            rows = (b[:, None] * 64 + torch.arange(64, device="cuda")).reshape(-1)
            z = q[0, t, h * G:(h + 1) * G].double() @ k[0, h, rows[rows <= t]].double().T * 128 ** -0.5
            want = torch.logsumexp(z, -1)
            err.append((lse[t, h * G:(h + 1) * G] - want) / torch.exp2(torch.floor(torch.log2(want)) - 23))
    assert float(torch.cat(err).square().mean().sqrt()) <= 0.58


def test_sparse_attn_backward_long_capacity():
    # buffers much longer than the sequences: the membership words and the dk / dv sums are laid out by the
    # capacity, the work items cut by 8192-token segments of the sequence; one that ends inside its third
    # segment and one just past its first, the rest of the capacity unused
    seqlens, Hq, Hkv, topk, cap = [20000, 8300], 16, 1, 8, 66000
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(57, seqlens, Hq, Hkv, n_planted=4)
    B = len(seqlens)
    rng = np.random.default_rng(10)
    do = synth.f32_to_bf16_bits(rng.standard_normal((B, T, Hq, 128), dtype=np.float32))

    def padded(x, axis):                                   # device copy with `cap` rows along the token axis
        shape = list(x.shape)
        shape[axis] = cap
        t = torch.zeros(shape, dtype=torch.bfloat16, device="cuda")
        t.narrow(axis, 0, x.shape[axis]).copy_(to_dev(x))
        return t

    qd, kd, vd, dod = padded(q, 1), padded(k, 2), padded(v, 2), padded(do, 1)
    sl = dev_i32(seqlens)
    idx = torch.full((B, Hkv, cap, topk), -1, dtype=torch.int32, device="cuda")
    want = [None] * B
    for b, l in enumerate(seqlens):
        _, ckb = ref.compress_keys(k[b, :, :l], oprm)
        pos = np.arange(l, dtype=np.int32)
        ib, _ = ref.select_blocks(q[b, :l], ckb, pos, oprm)
        idx[b, :, :l] = torch.from_numpy(ib).cuda()
        want[b] = ref.sparse_attn_bwd(q[b, :l], k[b, :, :l], v[b, :, :l], do[b, :l], pos, ib, oprm, want_mag=True)
    out, lse = binding.sparse_attn_prefill(prm, qd, kd, vd, sl, cap, idx)
    dq, dk, dv = binding.sparse_attn_bwd(prm, qd, kd, vd, out, dod, lse, sl, cap, idx)
    torch.cuda.synchronize()
    for b, l in enumerate(seqlens):
        wq, wk, wv, mq, mk, mv = want[b]
        eq = grad_err(dq[b, :l].double().cpu().numpy(), wq, mq)
        ek = grad_err(dk[b, :, :l].double().cpu().numpy(), wk, mk)
        ev = grad_err(dv[b, :, :l].double().cpu().numpy(), wv, mv)
        print("seq %d len %d: err/tol dq %.3f dk %.3f dv %.3f" % (b, l, eq, ek, ev), flush=True)
        assert eq <= 1.0 and ek <= 1.0 and ev <= 1.0
        assert bool((dq[b, l:] == 0).all()) and bool((dk[b, :, l:] == 0).all()) and bool((dv[b, :, l:] == 0).all())


# ------------------------------------------------------------------ query-block-shared selection (comparison variant)

@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,planted", [([1077, 333, 64, 1], 32, 2, 8, 5), ([700], 16, 2, 6, 3),
                                                          ([2500], 4, 1, 16, 4)])
def test_select_blocks_shared(seqlens, Hq, Hkv, topk, planted):
    print("case select shared", seqlens, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(61, seqlens, Hq, Hkv, n_planted=planted)
    qd, kd, sl = to_dev(q), to_dev(k), dev_i32(seqlens)
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks_shared(prm, qd, ck, sl, T)
    torch.cuda.synchronize()
    idx = idx.cpu().numpy()
    ckb = to_bits(ck)
    tot = near = 0
    for b, l in enumerate(seqlens):
        n_c = ref.num_kernels(l, 32, 16)
        want, margins, Rq = ref.select_blocks_shared(q[b, :l], ckb[b, :, :n_c], oprm, want_scores=True)
        n_qb = want.shape[1]
        n, e, nt, hard = compare_selection(idx[b, :, :n_qb], want, margins, Rq)
        assert not hard, hard[:3]
        assert np.all(idx[b, :, n_qb:] == -1)                          # query blocks past the end are not written
        tot, near = tot + n, near + nt
    assert near <= max(2, tot // 100)


@pytest.mark.parametrize("seqlens,Hq,Hkv,topk,planted", [([1077, 333, 64, 1, 0], 32, 2, 8, 5), ([700], 16, 2, 6, 3),
                                                          ([450], 2, 2, 5, 2), ([1500], 16, 1, 32, 5)])
def test_sparse_attn_prefill_shared(seqlens, Hq, Hkv, topk, planted):
    # the attention for per-query-block sets equals the per-token attention given the expanded sets
    print("case attn shared", seqlens, Hq, Hkv, topk, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(63, seqlens, Hq, Hkv, n_planted=planted)
    B = len(seqlens)
    n_qb = (T + 63) // 64
    idx_s = np.full((B, Hkv, n_qb, topk), -1, np.int32)
    want = [None] * B
    for b, l in enumerate(seqlens):
        if l == 0:
            continue
        _, ckb = ref.compress_keys(k[b, :, :l], oprm)
        ib, _ = ref.select_blocks_shared(q[b, :l], ckb, oprm)
        idx_s[b, :, :ib.shape[1]] = ib
        per_token = np.repeat(ib, 64, axis=1)[:, :l]                    # token t uses row t // 64
        want[b] = ref.sparse_attn(q[b, :l], k[b, :, :l], v[b, :, :l], np.arange(l, dtype=np.int32), per_token, oprm)
    qd, kd, vd, sl = to_dev(q), to_dev(k), to_dev(v), dev_i32(seqlens)
    out, lse = binding.sparse_attn_prefill_shared(prm, qd, kd, vd, sl, T, torch.from_numpy(idx_s).cuda())
    torch.cuda.synchronize()
    for b, l in enumerate(seqlens):
        if l == 0:
            continue
        eo = np.abs(out[b, :l].double().cpu().numpy() - want[b][0]).max()
        el = lse_err(lse[b, :l].double().cpu().numpy(), want[b][1])
        print("seq %d len %d: max|dO| %.3e LSE err/tol %.3f" % (b, l, eo, el), flush=True)
        assert eo <= OUT_TOL and el <= 1.0
        assert bool((out[b, l:] == 0).all())


@pytest.mark.parametrize("B,first", [(4, 4128), (17, 4128), (4, 8240), (17, 8240)])
def test_decode_step_many_sequences(B, first):
    # one step on a ragged batch, every sequence against the oracle (lengths include steps that complete a kernel); one kernel scores a row of up to
    # 8192 tokens; beyond, the selection has kernels of its own
    Hq, Hkv, topk = 32, 2, 8
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    rng = np.random.default_rng(77)
    lens = [int(rng.integers(40, 5000)) for _ in range(B)]
    lens[0], lens[1], lens[2] = first, 48, 1025                             # 4128, 8240 and 48 complete a kernel
    q, k, v, T = make_batch(97, lens, Hq, Hkv, n_planted=3)
    q1 = np.stack([q[b, l - 1] for b, l in enumerate(lens)])[:, None]
    kn = np.stack([k[b, :, l - 1] for b, l in enumerate(lens)])[:, :, None]
    vn = np.stack([v[b, :, l - 1] for b, l in enumerate(lens)])[:, :, None]
    k0, v0 = k.copy(), v.copy()
    for b, l in enumerate(lens):
        k0[b, :, l - 1] = 0
        v0[b, :, l - 1] = 0
    kc, vc, sl = to_dev(k0), to_dev(v0), dev_i32(lens)
    ck = binding.compress_keys(prm, kc, sl - 1, T)
    i1, o1, l1 = binding.decode_step(prm, to_dev(q1), to_dev(kn), to_dev(vn), kc, vc, ck, sl, T)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(kc), k) and np.array_equal(to_bits(vc), v)
    i1, ckb = i1.cpu().numpy(), to_bits(ck)
    for b, l in enumerate(lens):
        pos = np.array([l - 1], np.int32)
        _, ck_ref = ref.compress_keys(k[b, :, :l], oprm)
        assert np.array_equal(ckb[b, :, :ck_ref.shape[1]], ck_ref), b
        want, margins, R = ref.select_blocks(q1[b], ck_ref, pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(i1[b], want, margins, R)
        assert not hard, (b, hard)
        wo, wl = ref.sparse_attn(q1[b], k[b, :, :l], v[b, :, :l], pos, i1[b], oprm)
        assert out_err(o1[b].double().cpu().numpy(), wo) <= 1.0 and lse_err(l1[b].double().cpu().numpy(), wl[0]) <= 1.0


# The merge divides.  With queries of zero every key weighs 1, so an output is the exact mean of integer values: here one that lies halfway between two
# bf16 numbers, where the quotient rounds to the even one, and a product with the reciprocal, one rounding more, to its neighbour.  One merge kernel per
# top-k of up to 8, 16, 32 and 64; one to four blocks.
@pytest.mark.parametrize("L,topk", [(7, 8), (15, 16), (63, 32), (122, 64), (60, 8), (255, 24)])
def test_decoded_means_are_quotients(L, topk):
    print("case decoded means", L, topk, flush=True)
    Hq, Hkv, T = 4, 1, 320
    prm = binding.Params(Hq, Hkv, topk=topk)
    f = np.float32

    def bf16(x):
        return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(np.asarray(x, f)))

    odd = np.arange(257, 463, 2)                                          # halfway between the even integers that bf16 holds there
    tells = bf16((odd * L).astype(f) * (f(1) / f(L))) != bf16(odd)
    mean = np.resize(odd[tells], 128)
    v = np.zeros((T, 128), np.int64)
    for c, m in enumerate(mean):                                          # L integers of bf16 with that mean
        col = np.where(np.arange(L) < L // 2, m - 1, m + 1)
        if L % 2:                                                         # one odd value, below 256, and what it lacks over the others
            col[0] = 255
            more, rest = divmod(int(m * L - col.sum()) // 2, L - 1)
            col[1:] += 2 * more
            col[1:1 + rest] += 2
        assert col.sum() == m * L and (bf16(col) == col).all()
        v[:L, c] = col
    vd = torch.from_numpy(v).cuda().bfloat16().reshape(1, Hkv, T, 128)
    kd = torch.randn((1, Hkv, T, 128), device="cuda").bfloat16()
    q = torch.zeros((1, 1, Hq, 128), device="cuda", dtype=torch.bfloat16)
    sl = dev_i32([L])
    ck = binding.compress_keys(prm, kd, sl, T)
    want = torch.from_numpy(bf16(mean)).cuda().bfloat16().expand(Hq, 128)  # to nearest, ties to even
    idx = binding.select_blocks(prm, binding.MODE_DECODE, q, ck, sl, T)
    out, lse = binding.sparse_attn_decode(prm, q, kd, vd, sl, T, idx)
    torch.cuda.synchronize()
    assert torch.equal(out.reshape(Hq, 128), want), int((out.reshape(Hq, 128) != want).sum())
    assert float((lse - float(np.log(L))).abs().max()) <= 1e-5


# Where the workgroups that append sit: at the end of each row's chunks (3 per sequence here, up to 240 and beyond 1024 in all), behind all chunks, or
# behind the units of a short cache (more of them than a row has units).  The step against its parts, caches included.
@pytest.mark.parametrize("B,cap,topk", [(80, 8300, 8), (81, 8300, 8), (341, 8300, 4), (342, 8300, 4), (20, 2000, 8), (17, 900, 4), (8, 4096, 32), (7, 8192, 16)])
def test_decode_step_appends_to_every_sequence(B, cap, topk):
    print("case decode appends", B, cap, topk, flush=True)
    Hq, Hkv = 2, 1
    prm = binding.Params(Hq, Hkv, topk=topk)
    gen = torch.Generator(device="cuda").manual_seed(cap + B)
    q = torch.randn((B, 1, Hq, 128), device="cuda", generator=gen).bfloat16()
    kn, vn = (torch.randn((B, Hkv, 1, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn((B, Hkv, cap, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    lens = [cap - (37 * b) % (cap - 1) for b in range(B)]
    lens[1], lens[2], lens[3] = 32, cap + 1, 0                                          # completes the first kernel; neither of these is appended to
    sl = dev_i32(lens)
    ck = binding.compress_keys(prm, k, dev_i32([x - 1 if 0 < x <= cap else min(x, cap) for x in lens]), cap)
    parts, step = [x.clone() for x in (k, v, ck)], [x.clone() for x in (k, v, ck)]
    binding.append_kv(prm, kn, vn, parts[0], parts[1], sl, cap, ck=parts[2])
    idx = binding.select_blocks(prm, binding.MODE_DECODE, q, parts[2], sl, cap)
    out, lse = binding.sparse_attn_decode(prm, q, parts[0], parts[1], sl, cap, idx)
    got = binding.decode_step(prm, q, kn, vn, *step, sl, cap)
    torch.cuda.synchronize()
    for a, b in zip(parts + [idx, out, lse], step + list(got)):
        assert torch.equal(a.view(torch.int16) if a.dtype == torch.bfloat16 else a, b.view(torch.int16) if b.dtype == torch.bfloat16 else b)


def without_partial(q, ck, L, p, topk):
    """Block list of a decoding query whose log-sum-exps lack the p-th 128 kernels (p < 0: none).  q [Hq, d], ck [n_c, d] in 64 bits, one key-value
    head, 1 + 2 blocks forced."""
    z = q @ ck.T * q.shape[1] ** -0.5
    counted = np.where(np.arange(len(ck)) // 128 == p, -np.inf, z)
    m = counted.max(1, keepdims=True)
    r = np.exp(z - m - np.log(np.exp(counted - m).sum(1, keepdims=True))).mean(0)
    n = (L - 1) // 64 + 1
    r = np.concatenate([[-np.inf], r, np.full(4 * n + 4 - len(r), -np.inf)])                # block j: kernels 4j - 1 .. 4j + 3
    score = np.array([r[4 * j:4 * j + 5].max() for j in range(n)])
    picks = sorted(range(1, n - 2), key=lambda j: (-score[j], j))[:topk - 3]
    return np.array(sorted([0, n - 2, n - 1] + picks), np.int32)[None, None]


def rows_that_tell_partials(T, lens, Hq=16, topk=16, d=128):
    """A cache of T tokens, one key-value head, and four queries at its rows lens[i] - 1 whose picks move if a partial of their log-sum-exps is lost or
    counted for another head.  Half of a row's picks are blocks that two of its heads each put nearly all their weight on, in eight of the partials of
    128 kernels, the first, the last and those around the middle among them; which the others are follows from the heads' log-sum-exps.
    -> k, v [1, T, d], queries [4][Hq, d] as bits, what the oracle selects [4]."""
    oprm = ref.Params(Hq, 1, topk=topk)
    rng = np.random.default_rng(T)
    n_part = (ref.num_kernels(T, 32, 16) + 127) // 128
    u = rng.standard_normal((n_part, d)).astype(np.float32)
    u *= d ** 0.5 / np.linalg.norm(u, axis=1, keepdims=True)
    k = rng.standard_normal((T, d), dtype=np.float32) * np.exp(rng.standard_normal((T, 1), dtype=np.float32))
    for p in range(n_part):                               # a block of keys along u[p] within the kernels of every partial
        at = 2048 * p + (64 * (4 + 7 * p % 24) if 2048 * (p + 1) <= T - 1000 else 0)
        k[at:at + 64] = (u[p] + 0.1 * rng.standard_normal((64, d), dtype=np.float32))[:T - at]
    k = synth.f32_to_bf16_bits(k)[None]
    v = synth.f32_to_bf16_bits(rng.standard_normal((1, T, d), dtype=np.float32))
    qs, want, lost = [], [], 0
    for b, L in enumerate(lens):
        _, ck = ref.compress_keys(np.ascontiguousarray(k[:, :L]), oprm)
        n = (ck.shape[1] + 127) // 128
        parts = [(i * n // 8 + (0, 3, 5, n - 1 - 7 * n // 8)[b]) % n for i in range(8)]
        q = rng.standard_normal((Hq, d), dtype=np.float32)
        for h in range(Hq):
            q[h] += (8 + 6 * (5 * h % 16) / 15) * d ** -0.5 * u[parts[h % 8]]
        qs.append(synth.f32_to_bf16_bits(q))
        want.append(ref.select_blocks(qs[b][None], ck, np.array([L - 1], np.int32), oprm, want_scores=True))
        q64, ck64 = (synth.bf16_bits_to_f32(x).astype(np.float64) for x in (qs[b], ck[0]))
        assert not compare_selection(without_partial(q64, ck64, L, -1, topk), *want[b])[3]
        lost += sum(len(compare_selection(without_partial(q64, ck64, L, p, topk), *want[b])[3]) for p in parts)
    assert lost >= 24, "the inputs do not tell whether a partial is missing"     # of 32, by more than a near-tie
    return k, v, qs, want


# Decoding's tiles per workgroup follow sequences x heads x buffer (256 and 2048 workgroups of two tiles), and with them what a log-sum-exp is added
# up from: partials of 128 or of 256 kernels.  On either side of both lines, steps against the oracle.
@pytest.mark.parametrize("B,T", [(4, 131072), (4, 133000), (28, 17000), (29, 17000), (120, 32800), (121, 32800)])
def test_decode_tiles_by_workgroups(B, T):
    print("case decode tiles", B, T, flush=True)
    prm = binding.Params(16, 1, topk=16)
    lens = [T, T - 1000, T - 1000, T]
    k, v, qs, want = rows_that_tell_partials(T, lens)
    kd, vd = (to_dev(x).expand(B, 1, T, 128).contiguous() for x in (k, v))
    of = [b % 4 for b in range(B)]
    qd, sl = to_dev(np.stack(qs))[of][:, None], dev_i32([lens[b] for b in of])
    kn, vn = (to_dev(np.stack([x[:, L - 1:L] for L in lens]))[of] for x in (k, v))
    for b in range(B):
        kd[b, :, lens[of[b]] - 1:] = 0                    # (the step appends the last row; what lies behind it is not looked at)
        vd[b, :, lens[of[b]] - 1:] = 0
    ck = binding.compress_keys(prm, kd, sl - 1, T)
    idx, out, lse = binding.decode_step(prm, qd, kn, vn, kd, vd, ck, sl, T)
    alone = binding.select_blocks(prm, binding.MODE_DECODE, qd, ck, sl, T)
    torch.cuda.synchronize()
    assert torch.equal(alone, idx)
    for b in range(4, B):                                 # equal sequences, equal results
        assert torch.equal(idx[b], idx[of[b]]) and torch.equal(lse[b], lse[of[b]]), b
        assert torch.equal(out[b].view(torch.int16), out[of[b]].view(torch.int16)), b
    near = 0
    for b, L in enumerate(lens):
        got = idx[b].cpu().numpy()
        _, _, nt, hard = compare_selection(got, *want[b])
        assert not hard, (b, hard)
        near += nt
        wo, wl = ref.sparse_attn(qs[b][None], np.ascontiguousarray(k[:, :L]), np.ascontiguousarray(v[:, :L]), np.array([L - 1], np.int32), got,
                                 oracle_params(prm))
        assert out_err(out[b].double().cpu().numpy(), wo) <= 1.0 and lse_err(lse[b].double().cpu().numpy(), wl[0]) <= 1.0, b
    assert near <= 1


# Verification merges 64 partials of a log-sum-exp at a time: 8192 kernels, one more, and as many as a buffer may have.
@pytest.mark.parametrize("T", [131088, 131104, 262144])
def test_verify_selection_partials(T):
    print("case verify partials", T, flush=True)
    prm = binding.Params(16, 1, topk=16)
    lens = [T - 3, T - 2, T - 1, T]
    k, v, qs, want = rows_that_tell_partials(T, lens)
    kd, sl = to_dev(k)[None], dev_i32([T])
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks_verify(prm, to_dev(np.stack(qs))[None], ck, sl, T)
    torch.cuda.synchronize()
    near = 0
    for t in range(4):
        _, _, nt, hard = compare_selection(idx[0, :, t:t + 1].cpu().numpy(), *want[t])
        assert not hard, (t, hard)
        near += nt
    assert near <= 1


# Short prompts read keys and values where they lie: both sides of its lines, padded and interleaved token strides, an end inside a
# block, sequences of nothing; the same bits whatever the strides.
@pytest.mark.parametrize("seqlens,Hq,Hkv", [([1], 32, 2), ([64, 0, 17], 16, 1), ([190], 32, 2), ([193], 32, 2), ([383, 100], 8, 2), ([767], 8, 2),
                                            ([895], 4, 1), ([897], 4, 1), ([896, 1], 1, 1), ([333, 65], 2, 2), ([319], 32, 2), ([320], 32, 2),
                                            ([639], 16, 2), ([640, 1], 8, 1)])
def test_sparse_attn_prefill_direct(seqlens, Hq, Hkv):
    print("case direct", seqlens, Hq, Hkv, flush=True)
    prm, oprm = binding.Params(Hq, Hkv, topk=6), oracle_params(binding.Params(Hq, Hkv, topk=6))
    B, T = len(seqlens), max(seqlens)
    gen = torch.Generator(device="cuda").manual_seed(T)
    q = torch.randn((B, T, Hq, 128), device="cuda", generator=gen).bfloat16()
    pad = torch.randn((B, Hkv, T, 128 + 72), device="cuda", generator=gen).bfloat16()
    inter = torch.randn((B, T, Hkv + 1, 128), device="cuda", generator=gen).bfloat16()
    k, v = pad[..., :128], inter.transpose(1, 2)[:, :Hkv]                # token strides 200 and 128 (Hkv + 1)
    own = (torch.arange(T, device="cuda") // 64)[None, None, :, None]
    idx = own - torch.arange(6, device="cuda")[None, None, None, :] * torch.tensor([1, 2], device="cuda")[torch.arange(T, device="cuda") % 2][None, None, :, None]
    idx = torch.where(idx < 0, torch.full_like(idx, -1), idx).expand(B, Hkv, T, 6).to(torch.int32).contiguous()
    sl = dev_i32(seqlens)
    out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx)
    out2, lse2 = torch.full_like(q, 3.0), torch.full((B, T, Hq), 5.0, device="cuda")
    binding.sparse_attn_prefill(prm, q, k.contiguous(), v.contiguous(), sl, T, idx, out=out2, lse=lse2)
    torch.cuda.synchronize()
    for b, l in enumerate(seqlens):
        assert torch.equal(out[b, :l], out2[b, :l]) and torch.equal(lse[b, :l], lse2[b, :l])
        assert bool((out[b, l:] == 0).all()) and bool((lse[b, l:] == 0).all())
        assert bool((out2[b, l:] == 3.0).all()) and bool((lse2[b, l:] == 5.0).all())
        if l:
            pos = np.arange(l, dtype=np.int32)
            wo, wl = ref.sparse_attn(to_bits(q[b, :l]), to_bits(k[b, :, :l].contiguous()), to_bits(v[b, :, :l].contiguous()), pos, idx[b, :, :l].cpu().numpy(), oprm)
            assert np.abs(out[b, :l].double().cpu().numpy() - wo).max() <= OUT_TOL and lse_err(lse[b, :l].double().cpu().numpy(), wl) <= 1.0


# Tokens that share a tile with one that selected a block of infinities and NaNs must not see them: the rows that do not list
# the block (or list another head's) are what they are with ordinary values there, and its own rows stay reachable.
@pytest.mark.parametrize("T,Hq,Hkv", [(300, 4, 1), (770, 8, 1), (1700, 4, 2), (4100, 8, 2), (300, 1, 1), (3100, 2, 2), (600, 16, 1)])
@pytest.mark.parametrize("where", ["k", "v"])
def test_values_of_a_block_reach_only_the_tokens_that_selected_it(T, Hq, Hkv, where):
    print("case non-finite block", T, Hq, Hkv, where, flush=True)
    prm = binding.Params(Hq, Hkv, topk=3)
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, do = (torch.randn((1, T, Hq, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn((1, Hkv, T, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    own = (torch.arange(T, device="cuda") // 64)[None, :].expand(Hkv, T)
    lists = torch.arange(T, device="cuda")[None, :] % 3 == 1              # every third token selects block 1
    idx = torch.stack([torch.zeros_like(own), torch.where(lists, torch.ones_like(own), torch.full_like(own, -1)), own], -1)
    idx = torch.where((idx == 0) & (own == 0)[..., None] & (torch.arange(3, device="cuda") < 1), torch.full_like(idx, -1), idx)
    idx = torch.where((torch.arange(3, device="cuda") == 1) & (own <= 1)[..., None], torch.full_like(idx, -1), idx)[None].to(torch.int32).contiguous()
    sl = dev_i32([T])

    def both(k, v):
        out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, T, idx)
        clean = torch.nan_to_num(out, 0.0, 0.0, 0.0), torch.nan_to_num(lse, 0.0, 0.0, 0.0)
        return out, lse, binding.sparse_attn_bwd(prm, q, k, v, clean[0], do, clean[1], sl, T, idx)[0]

    want = both(k, v)
    k2, v2 = k.clone(), v.clone()
    bad = k2 if where == "k" else v2
    bad[:, :, 64 + 3, 5], bad[:, :, 64 + 40, 17], bad[:, :, 64 + 63] = float("nan"), float("inf"), -float("inf")
    got = both(k2, v2)
    torch.cuda.synchronize()
    free = ~lists[0] & (own[0] != 1)                                       # neither listed nor the own block
    assert bool((~torch.isfinite(got[0][:, ~free].float())).any())
    for x, y, name in zip(got, want, ("out", "lse", "dq")):
        x, y = x[:, free].double(), y[:, free].double()
        assert bool(torch.isfinite(x).all()), name
        # the same sums with the reference exponent perhaps placed differently: each side is within a bf16 rounding of the result
        # (outputs and gradients) and of the probabilities in it (whose errors average out over 64 keys and more), or fp32 for lse
        assert bool(((x - y).abs() <= (1e-4 if name == "lse" else 2.0 ** -7 * y.abs() + 2.0 ** -7 * y.pow(2).mean().sqrt())).all()), name


# Caches of up to 8192 tokens take the one-kernel selection: both sides of each of its lines (16, 32, 64, 128 blocks), the
# three-launch form for many rows, the long path from 8193 tokens on and around a list of 128 blocks, lengths that complete
# a kernel, are shorter than one, or select everything.
@pytest.mark.parametrize("cap,lens,Hq,Hkv,topk,forced", [
    (64, [1, 31, 32, 64], 32, 2, 16, (1, 2)), (1024, [1024, 1008, 1023], 32, 2, 8, (1, 2)), (1025, [1025, 48], 4, 2, 16, (0, 0)),
    (2048, [2048, 1040, 600], 8, 1, 12, (1, 2)), (2049, [2049, 2000], 16, 1, 64, (2, 3)), (4096, [4096, 4095, 3000], 2, 2, 16, (1, 2)),
    (4097, [4097, 100], 32, 2, 16, (0, 1)), (8192, [8192, 8191, 8176], 32, 2, 16, (1, 2)), (8192, [8192, 5008], 16, 2, 33, (1, 0)),
    (8193, [8193, 8192, 65], 32, 2, 16, (1, 2)), (16384, [16384, 8208], 4, 1, 64, (0, 0)), (16500, [16448, 16500], 32, 2, 16, (1, 2)),
    (2048, [33 + 49 * b for b in range(41)], 32, 2, 16, (1, 2)), (8192, [8192 - 176 * b for b in range(20)], 16, 1, 16, (1, 2))])
def test_decode_step_short_caches(cap, lens, Hq, Hkv, topk, forced):
    print("case short decode", cap, len(lens), Hq, Hkv, topk, forced, flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk, n_init_blocks=forced[0], n_local_blocks=forced[1])
    oprm = oracle_params(prm)
    B = len(lens)
    gen = torch.Generator(device="cuda").manual_seed(cap + B)
    q = torch.randn((B, 1, Hq, 128), device="cuda", generator=gen).bfloat16()
    k, v = (torch.randn((B, Hkv, cap, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    k[:, :, ::5] += 3 * q.float().mean(2)[:, 0, None, None, :].bfloat16()        # scores well apart
    sl = dev_i32(lens)
    at = (torch.tensor(lens, device="cuda") - 1)
    rows = torch.arange(B, device="cuda")
    kn, vn = k[rows, :, at][:, :, None].contiguous(), v[rows, :, at][:, :, None].contiguous()
    ck = binding.compress_keys(prm, k, sl - 1, cap)
    kc, vc = k.clone(), v.clone()
    for b, l in enumerate(lens):                            # what this step is about to write: a stale read shows
        kc[b, :, l - 1], vc[b, :, l - 1] = 90.0, 90.0
        if l >= 32 and (l - 32) % 16 == 0:
            ck[b, :, (l - 32) // 16] = 90.0
    kc2, vc2, ck2 = kc.clone(), vc.clone(), ck.clone()
    idx, out, lse = binding.decode_step(prm, q, kn, vn, kc, vc, ck, sl, cap)
    binding.append_kv(prm, kn, vn, kc2, vc2, sl, cap, ck=ck2)
    idx2 = binding.select_blocks(prm, binding.MODE_DECODE, q, ck2, sl, cap)
    out2, lse2 = binding.sparse_attn_decode(prm, q, kc2, vc2, sl, cap, idx2)
    torch.cuda.synchronize()
    for x, y in ((kc, k), (vc, v), (kc2, k), (ck, ck2), (idx, idx2), (out, out2), (lse, lse2)):
        assert torch.equal(x, y)
    for b in sorted(set(range(B)) if B < 5 else {0, 1, B // 2, B - 1}):
        l = lens[b]
        pos = np.array([l - 1], np.int32)
        kb, vb, qb = to_bits(k[b, :, :l]), to_bits(v[b, :, :l]), to_bits(q[b])
        _, ck_ref = ref.compress_keys(kb, oprm)
        assert np.array_equal(to_bits(ck[b])[:, :ck_ref.shape[1]], ck_ref), b
        want, margins, R = ref.select_blocks(qb, ck_ref, pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx[b].cpu().numpy(), want, margins, R)
        assert not hard, (b, hard)
        wo, wl = ref.sparse_attn(qb, kb, vb, pos, idx[b].cpu().numpy(), oprm)
        assert out_err(out[b].double().cpu().numpy(), wo) <= 1.0 and lse_err(lse[b].double().cpu().numpy(), wl[0]) <= 1.0


# An infinite value in the last selected block makes its channel infinite (as IEEE sums do), and no other: the merge rounds the top-k up
# and what it adds for the places past the end must not turn the infinity into a NaN.
@pytest.mark.parametrize("topk", [3, 8, 12, 16, 24, 33])
def test_decode_merge_keeps_an_infinity_of_the_last_block(topk):
    print("case infinite value", topk, flush=True)
    Hq, Hkv, L, n = 8, 2, 64 * 70 - 9, 3
    prm = binding.Params(Hq, Hkv, topk=topk)
    gen = torch.Generator(device="cuda").manual_seed(topk)
    q = torch.randn((1, n, Hq, 128), device="cuda", generator=gen).bfloat16()
    k, v = (torch.randn((1, Hkv, L, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    v[0, :, L - 20, 7], v[0, 1, L - 21, 100] = float("inf"), -float("inf")
    idx = torch.cat([torch.arange(topk - 1), torch.tensor([69])]).to(torch.int32).expand(1, Hkv, n, topk).contiguous().cuda()
    sl = dev_i32([L])
    q1, idx1 = q[:, -1:].contiguous(), idx[:, :, -1:].contiguous()
    out, lse = torch.zeros_like(q1), torch.zeros((1, Hq), dtype=torch.float32, device="cuda")
    results = [binding.sparse_attn_decode(prm, q1, k, v, sl, L, idx1), binding.sparse_attn_verify(prm, q, k, v, sl, L, idx),
               binding.sparse_attn_decode_noalloc(prm, q1, k, v, sl, L, idx1, out, lse)]
    for o, ls in results:
        o = o.float()
        assert bool((o[..., 7] == float("inf")).all()) and bool((o[:, :, Hq // Hkv:, 100] == -float("inf")).all())
        o[..., 7], o[:, :, Hq // Hkv:, 100] = 0.0, 0.0
        assert bool(torch.isfinite(o).all()) and bool(torch.isfinite(ls).all())


@pytest.mark.parametrize("B", [1, 4])
@pytest.mark.parametrize("rho", [2, 4])
def test_decode_step_approximate_lse_when_the_new_kernel_feeds_another_workgroup(rho, B):
    # One-call decode steps with the approximate log-sum-exp at the lengths where the semantic kernel the
    # new token completes is the last fine kernel of a coarse kernel that ANOTHER workgroup of the first
    # selection kernel owns (128 or 256 kernels per workgroup: one or four sequences).  That workgroup
    # must not read the row back from the compressed-key cache while it is being written: the row is
    # pre-filled with large values here, so a stale read changes the scores.
    Hq, Hkv, topk = 32, 2, 16
    prm = binding.Params(Hq, Hkv, topk=topk, lse_coarse_ratio=rho)
    oprm = oracle_params(prm)
    chunk_tokens = 16 * (128 if B < 4 else 256)
    base = 32 if rho == 2 else 64
    lens = [chunk_tokens * (1 + b % 2) + base for b in range(B)]
    q, k, v, T = make_batch(131 + rho, lens, Hq, Hkv, n_planted=3)
    q1 = np.stack([q[b, l - 1] for b, l in enumerate(lens)])[:, None]
    kn = np.stack([k[b, :, l - 1] for b, l in enumerate(lens)])[:, :, None]
    vn = np.stack([v[b, :, l - 1] for b, l in enumerate(lens)])[:, :, None]
    k0, v0 = k.copy(), v.copy()
    for b, l in enumerate(lens):
        k0[b, :, l - 1] = 0
        v0[b, :, l - 1] = 0
    kc, vc, sl = to_dev(k0), to_dev(v0), dev_i32(lens)
    ck = binding.compress_keys(prm, kc, sl - 1, T)
    for b, l in enumerate(lens):
        ck[b, :, (l - 32) // 16] = 100.0                                    # the row this step is about to write
    i1, o1, l1 = binding.decode_step(prm, to_dev(q1), to_dev(kn), to_dev(vn), kc, vc, ck, sl, T)
    torch.cuda.synchronize()
    i1, ckb = i1.cpu().numpy(), to_bits(ck)
    for b, l in enumerate(lens):
        print("case rho %d batch %d seq %d len %d" % (rho, B, b, l), flush=True)
        pos = np.array([l - 1], np.int32)
        _, ck_ref = ref.compress_keys(k[b, :, :l], oprm)
        assert np.array_equal(ckb[b, :, :ck_ref.shape[1]], ck_ref), b
        want, margins, R = ref.select_blocks(q1[b], ck_ref, pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(i1[b], want, margins, R)
        assert not hard, (b, hard)
        wo, wl = ref.sparse_attn(q1[b], k[b, :, :l], v[b, :, :l], pos, i1[b], oprm)
        assert out_err(o1[b].double().cpu().numpy(), wo) <= 1.0 and lse_err(l1[b].double().cpu().numpy(), wl[0]) <= 1.0


# ------------------------------------------------------------------ lengths outside [0, max_seqlen]

def test_out_of_range_lengths_are_clamped():
    # the interface clamps every entry of seqlens to [0, max_seqlen]; a decode step appends nothing for
    # an entry outside [1, max_seqlen]
    Hq, Hkv, topk = 32, 2, 8
    true_len = [0, 0, 700, 300]
    prm = binding.Params(Hq, Hkv, topk=topk)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(91, true_len, Hq, Hkv, n_planted=3)          # T = 700
    B = len(true_len)
    given = dev_i32([-3, 0, T + 50, 300])
    qd, kd, vd = to_dev(q), to_dev(k), to_dev(v)
    ck = binding.compress_keys(prm, kd, given, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, given, T)
    out, lse = binding.sparse_attn_prefill(prm, qd, kd, vd, given, T, idx)
    rng = np.random.default_rng(12)
    do = synth.f32_to_bf16_bits(rng.standard_normal((B, T, Hq, 128), dtype=np.float32))
    dq, dk, dv = binding.sparse_attn_bwd(prm, qd, kd, vd, out, to_dev(do), lse, given, T, idx)
    torch.cuda.synchronize()
    ckb, idx_np = to_bits(ck), idx.cpu().numpy()
    for b, l in enumerate(true_len):
        assert bool((out[b, l:] == 0).all()) and bool((dq[b, l:] == 0).all()) and bool((dk[b, :, l:] == 0).all())
        assert np.all(idx_np[b, :, l:] == -1)
        if l == 0:
            assert not ckb[b].any()
            continue
        pos = np.arange(l, dtype=np.int32)
        _, ck_ref = ref.compress_keys(k[b, :, :l], oprm)
        assert np.array_equal(ckb[b, :, :ck_ref.shape[1]], ck_ref) and not ckb[b, :, ck_ref.shape[1]:].any()
        want, margins, R = ref.select_blocks(q[b, :l], ck_ref, pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx_np[b, :, :l], want, margins, R)
        assert not hard, (b, hard[:3])
        wo, wl = ref.sparse_attn(q[b, :l], k[b, :, :l], v[b, :, :l], pos, idx_np[b, :, :l], oprm)
        assert out_err(out[b, :l].double().cpu().numpy(), wo) <= 1.0 and lse_err(lse[b, :l].double().cpu().numpy(), wl) <= 1.0
        wq, wk, wv, mq, mk, mv = ref.sparse_attn_bwd(q[b, :l], k[b, :, :l], v[b, :, :l], do[b, :l], pos, idx_np[b, :, :l], oprm,
                                                     want_mag=True)
        assert grad_err(dq[b, :l].double().cpu().numpy(), wq, mq) <= 1.0
        assert grad_err(dk[b, :, :l].double().cpu().numpy(), wk, mk) <= 1.0
        assert grad_err(dv[b, :, :l].double().cpu().numpy(), wv, mv) <= 1.0
    # one decode step with the same lengths: sequences 0-2 append nothing (2 decodes at position T - 1 on
    # the cache as it is), sequence 3 appends its row 299 again
    q1 = np.stack([q[b, max(l, 1) - 1] for b, l in enumerate(true_len)])[:, None]
    kn = np.stack([k[b, :, max(l, 1) - 1] for b, l in enumerate(true_len)])[:, :, None]
    vn = np.stack([v[b, :, max(l, 1) - 1] for b, l in enumerate(true_len)])[:, :, None]
    kn[2], vn[2] = 0x3F80, 0x3F80                                         # would be visible if it were appended
    kc, vc = to_dev(k), to_dev(v)
    i1, o1, l1 = binding.decode_step(prm, to_dev(q1), to_dev(kn), to_dev(vn), kc, vc, ck, given, T)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(kc), k) and np.array_equal(to_bits(vc), v) and np.array_equal(to_bits(ck), ckb)
    i1 = i1.cpu().numpy()
    for b, l in enumerate(true_len):
        if l == 0:
            assert np.all(i1[b] == -1) and bool((o1[b] == 0).all()) and bool(torch.isneginf(l1[b]).all())
            continue
        pos = np.array([l - 1], np.int32)
        want, margins, R = ref.select_blocks(q1[b], ckb[b, :, :ref.num_kernels(l, 32, 16)], pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(i1[b], want, margins, R)
        assert not hard, (b, hard)
        wo, wl = ref.sparse_attn(q1[b], k[b, :, :l], v[b, :, :l], pos, i1[b], oprm)
        assert out_err(o1[b].double().cpu().numpy(), wo) <= 1.0 and lse_err(l1[b].double().cpu().numpy(), wl[0]) <= 1.0


# ------------------------------------------------------------------ seeded random configurations, every entry point

@pytest.mark.parametrize("seed,wide", [(s, False) for s in range(24)] + [(s, True) for s in range(6)])
def test_random_configurations_all_entry_points(seed, wide):
    # wide: the limits of the interface (top-k up to 64, up to 64 drafted tokens) and longer sequences
    rng = np.random.default_rng((5000 if wide else 1000) + seed)
    G = int(rng.choice([1, 2, 4, 8, 16]))
    Hkv = int(rng.choice([1, 2, 3]))
    Hq = G * Hkv
    n_init, n_local = int(rng.integers(0, 5 if wide else 3)), int(rng.integers(0, 6 if wide else 4))
    topk = int(rng.integers(max(1, n_init + n_local), 65 if wide else 20))
    B = int(rng.integers(1, 6 if wide else 4))
    seqlens = [int(rng.integers(1, 2600 if wide else 900)) for _ in range(B)]
    if seed % 3 == 0:
        seqlens[0] = int(rng.choice([31, 32, 63, 64, 65, 128, 129]))
    if seed % 3 == 1:                                                 # around tile (256) and kernel (16) boundaries
        seqlens[-1] = int(rng.choice([255, 256, 257, 271, 272, 287, 288, 513, 527, 528, 543]))
    rho = 1
    if G == 16 and (n_init + n_local) * 64 >= 128 and seed % 2:
        rho = int(rng.choice([2, 4])) if (n_init + n_local) * 64 >= 8 * 16 else 2
    print("case random", seed, wide, dict(G=G, Hkv=Hkv, topk=topk, n_init=n_init, n_local=n_local, seqlens=seqlens, rho=rho), flush=True)
    prm = binding.Params(Hq, Hkv, topk=topk, n_init_blocks=n_init, n_local_blocks=n_local, lse_coarse_ratio=rho)
    oprm = oracle_params(prm)
    q, k, v, T = make_batch(200 + seed, seqlens, Hq, Hkv, n_planted=int(rng.integers(0, 4)), heavy=(0,) if seed % 4 == 0 else ())
    if seed % 5 == 0:                                                 # buffers larger than every sequence
        extra = int(rng.integers(1, 400))
        q = np.concatenate([q, np.zeros((B, extra, Hq, 128), np.uint16)], axis=1)
        k = np.concatenate([k, np.zeros((B, Hkv, extra, 128), np.uint16)], axis=2)
        v = np.concatenate([v, np.zeros((B, Hkv, extra, 128), np.uint16)], axis=2)
        T += extra
    # every seventh case: caches stored token-major and queries head-major (the ABI takes any strides with
    # a contiguous head_dim axis)
    lay = (lambda x: x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)) if seed % 7 == 3 else (lambda x: x)
    qd, kd, vd, sl = lay(to_dev(q)), lay(to_dev(k)), lay(to_dev(v)), dev_i32(seqlens)
    # prefill: compress, select, attend
    ck = binding.compress_keys(prm, kd, sl, T)
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, qd, ck, sl, T)
    torch.cuda.synchronize()
    ckb, idx_np = to_bits(ck), idx.cpu().numpy()
    idx_ref = np.full((B, Hkv, T, topk), -1, np.int32)
    near = 0
    for b, l in enumerate(seqlens):
        _, ck_ref = ref.compress_keys(k[b, :, :l], oprm)
        assert np.array_equal(ckb[b, :, :ck_ref.shape[1]], ck_ref)
        want, margins, R = ref.select_blocks(q[b, :l], ck_ref, np.arange(l, dtype=np.int32), oprm, want_scores=True)
        n, e, nt, hard = compare_selection(idx_np[b, :, :l], want, margins, R)
        assert not hard, hard[:3]
        near += nt
        idx_ref[b, :, :l] = want
    assert near <= 3
    idx_d = torch.from_numpy(idx_ref).cuda()
    out, lse = binding.sparse_attn_prefill(prm, qd, kd, vd, sl, T, idx_d)
    do = synth.f32_to_bf16_bits(rng.standard_normal((B, T, Hq, 128), dtype=np.float32))
    dq, dk, dv = binding.sparse_attn_bwd(prm, qd, kd, vd, out, lay(to_dev(do)), lse, sl, T, idx_d)
    torch.cuda.synchronize()
    for b, l in enumerate(seqlens):
        pos = np.arange(l, dtype=np.int32)
        wo, wl = ref.sparse_attn(q[b, :l], k[b, :, :l], v[b, :, :l], pos, idx_ref[b, :, :l], oprm)
        assert out_err(out[b, :l].double().cpu().numpy(), wo) <= 1.0
        assert lse_err(lse[b, :l].double().cpu().numpy(), wl, logit_mag(q[b, :l], k[b, :, :l], prm.softmax_scale)) <= 1.0
        wq, wk, wv, mq, mk, mv = ref.sparse_attn_bwd(q[b, :l], k[b, :, :l], v[b, :, :l], do[b, :l], pos, idx_ref[b, :, :l],
                                                     oprm, want_mag=True)
        assert grad_err(dq[b, :l].double().cpu().numpy(), wq, mq) <= 1.0
        assert grad_err(dk[b, :, :l].double().cpu().numpy(), wk, mk) <= 1.0
        assert grad_err(dv[b, :, :l].double().cpu().numpy(), wv, mv) <= 1.0
    # one decode step in one call: the last token of every sequence taken out of the cache and appended again
    last = np.array([l - 1 for l in seqlens])
    kn = np.stack([k[b, :, last[b]] for b in range(B)])[:, :, None]
    vn = np.stack([v[b, :, last[b]] for b in range(B)])[:, :, None]
    q1 = np.stack([q[b, last[b]] for b in range(B)])[:, None]
    k0, v0 = k.copy(), v.copy()
    for b in range(B):
        k0[b, :, last[b]] = 0
        v0[b, :, last[b]] = 0
    kc, vc = lay(to_dev(k0)), lay(to_dev(v0))
    ck1 = binding.compress_keys(prm, kc, dev_i32([l - 1 for l in seqlens]), T)
    i1, o1, l1 = binding.decode_step(prm, to_dev(q1), to_dev(kn), to_dev(vn), kc, vc, ck1, sl, T)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(kc), k) and np.array_equal(to_bits(vc), v)
    i1 = i1.cpu().numpy()
    for b, l in enumerate(seqlens):
        pos = np.array([l - 1], np.int32)
        _, ck_ref = ref.compress_keys(k[b, :, :l], oprm)
        assert np.array_equal(to_bits(ck1)[b, :, :ck_ref.shape[1]], ck_ref)
        want, margins, R = ref.select_blocks(q1[b], ck_ref, pos, oprm, want_scores=True)
        n, e, nt, hard = compare_selection(i1[b], want, margins, R)
        assert not hard, (b, hard)
        wo, wl = ref.sparse_attn(q1[b], k[b, :, :l], v[b, :, :l], pos, i1[b], oprm)
        assert out_err(o1[b].double().cpu().numpy(), wo) <= 1.0
        assert lse_err(l1[b].double().cpu().numpy(), wl[0], logit_mag(q1[b], k[b, :, :l], prm.softmax_scale)[0]) <= 1.0
    # verification of the last n tokens with a random tree, and the query-block-shared comparison variant
    n = int(rng.integers(1, 65 if wide else 9))
    qn = np.zeros((B, n, Hq, 128), np.uint16)
    masks = np.zeros((B, n), np.uint64)
    for b, l in enumerate(seqlens):
        masks[b] = tree_masks(rng, n, "tree")
        if l >= n:
            qn[b] = q[b, l - n:l]
    iv = binding.select_blocks_verify(prm, to_dev(qn), ck, sl, T)
    ov, lv = binding.sparse_attn_verify(prm, to_dev(qn), kd, vd, sl, T, iv, tree_mask=dev_masks(masks))
    torch.cuda.synchronize()
    iv = iv.cpu().numpy()
    for b, l in enumerate(seqlens):
        if l < n:
            assert np.all(iv[b] == -1)
            continue
        pos = np.arange(l - n, l, dtype=np.int32)
        want, margins, R = ref.select_blocks(qn[b], ckb[b, :, :ref.num_kernels(l, 32, 16)], pos, oprm, want_scores=True)
        nn, e, nt, hard = compare_selection(iv[b], want, margins, R)
        assert not hard, (b, hard)
        wo, wl = ref.sparse_attn_tree(qn[b], k[b, :, :l], v[b, :, :l], iv[b], masks[b], l - n, oprm)
        assert out_err(ov[b].double().cpu().numpy(), wo) <= 1.0
        assert lse_err(lv[b].double().cpu().numpy(), wl, logit_mag(qn[b], k[b, :, :l], prm.softmax_scale)) <= 1.0
    # the same verification step in one call, from the state before the drafts: equal bit for bit
    k0, v0 = k.copy(), v.copy()
    kn = np.zeros((B, Hkv, n, 128), np.uint16)
    vn = np.zeros((B, Hkv, n, 128), np.uint16)
    for b, l in enumerate(seqlens):
        if l >= n:
            kn[b], vn[b] = k[b, :, l - n:l], v[b, :, l - n:l]
            k0[b, :, l - n:l] = 0
            v0[b, :, l - n:l] = 0
    kc, vc = lay(to_dev(k0)), lay(to_dev(v0))
    ckv = binding.compress_keys(prm, kc, dev_i32([l - n if l >= n else l for l in seqlens]), T)
    i2, o2, l2 = binding.verify_step(prm, to_dev(qn), to_dev(kn), to_dev(vn), kc, vc, ckv, sl, T, tree_mask=dev_masks(masks))
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(kc), k) and np.array_equal(to_bits(vc), v) and np.array_equal(to_bits(ckv), ckb)
    assert np.array_equal(i2.cpu().numpy(), iv)
    assert torch.equal(o2.view(torch.int16), ov.view(torch.int16)) and torch.equal(l2, lv)
    if rho == 1:
        isd = binding.select_blocks_shared(prm, qd, ck, sl, T)
        osd, lsd = binding.sparse_attn_prefill_shared(prm, qd, kd, vd, sl, T, isd)
        torch.cuda.synchronize()
        isd = isd.cpu().numpy()
        for b, l in enumerate(seqlens):
            want, margins, Rq = ref.select_blocks_shared(q[b, :l], ckb[b, :, :ref.num_kernels(l, 32, 16)], oprm, want_scores=True)
            nn, e, nt, hard = compare_selection(isd[b, :, :want.shape[1]], want, margins, Rq)
            assert not hard, (b, hard)
            per_token = np.repeat(isd[b, :, :want.shape[1]], 64, axis=1)[:, :l]
            wo, wl = ref.sparse_attn(q[b, :l], k[b, :, :l], v[b, :, :l], np.arange(l, dtype=np.int32), per_token, oprm)
            assert out_err(osd[b, :l].double().cpu().numpy(), wo) <= 1.0
            assert lse_err(lsd[b, :l].double().cpu().numpy(), wl, logit_mag(q[b, :l], k[b, :, :l], prm.softmax_scale)) <= 1.0
