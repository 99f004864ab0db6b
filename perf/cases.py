"""The measured workloads: what a program that uses this framework has it do, through the public entry points.

  listed()             the fixed cases, smallest to largest
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  the inputs, caches and buffers such a program holds before the call, on the GPU
  run(state)           one pass, and everything it computes
  work(case)           bytes and operations of one pass that no implementation can do without
  tolerance(case)      how far two correct implementations may lie apart

A case is a dict of plain values:
  kind       "prefill"   compress_keys -> select_blocks -> sparse_attn_prefill over whole sequences
             "train"     the same, then sparse_attn_bwd: the attention's part of a training step
             "backward"  sparse_attn_bwd alone, on a finished forward
             "decode"    decode_step: append, select and attend for one new token per sequence
             "verify"    verify_step: the same for n_draft drafted tokens per sequence (a random tree, or a chain)
  batch, seq, seq_min    sequences, the longest and the shortest of them (lengths spread evenly between; for decode
                         and verify the lengths count the new tokens)
  hq, hkv, topk, rho     query heads, key-value heads, blocks per query, ratio of the approximate log-sum-exp (1 = exact)
  heavy                  leading sequences with heavy-tailed key norms
  keep                   True: the caller's own result buffers and workspaces, as a serving loop has them;
                         False: results and workspaces allocated by the call
  layers, graph          decode: caches of this many layers stepped one after the other; captured once in a HIP graph
  n_draft, tree          verify: drafted tokens, random tree instead of a chain

Inputs follow the recipe of paper_2506_07900_amd/synth.py, drawn on the GPU: N(0,1) queries, keys and values in bf16,
one planted block (keys along the mean query of the group) per 1024 tokens, optionally log-normal key norms.
"""
import numpy as np
import torch

from paper_2506_07900_amd import binding

D, BLOCK = 128, 64

_FIELDS = dict(kind="prefill", batch=1, seq=0, seq_min=0, hq=32, hkv=2, topk=16, rho=1, heavy=0, keep=True, layers=1,
               graph=False, n_draft=1, tree=False)


def _case(**kw):
    c = dict(_FIELDS, **kw)
    c["seq_min"] = c["seq_min"] or c["seq"]
    return c


def listed():
    return [
        # the smallest call: one chat turn's next token on a small model (4 query heads : 1), called eagerly
        _case(name="decode_2k_g4", kind="decode", seq=1999, hq=4, hkv=1, topk=8),
        # the next token of one 128K-token document: eight layers' attention in a captured HIP graph, as a latency-bound
        # serving loop replays it
        _case(name="decode_128k_graph", kind="decode", seq=131047, layers=8, graph=True),
        # a ragged serving batch, half of it with heavy-tailed keys, called eagerly
        _case(name="decode_ragged_b8", kind="decode", batch=8, seq=130999, seq_min=16411, heavy=4),
        # a full serving batch of long documents: the bandwidth end of decoding
        _case(name="decode_128k_b32", kind="decode", batch=32, seq=131061),
        # speculative decoding: 16 drafted tokens of a tree, verified at 128K
        _case(name="verify_128k_n16", kind="verify", seq=130991, n_draft=16, tree=True),
        # a short prompt, everything allocated by the calls: launches and host work count
        _case(name="prefill_777", seq=777, topk=8, keep=False),
        # a 2K prompt on the small model
        _case(name="prefill_2k_g4", seq=2048, hq=4, hkv=1, topk=8),
        # a ragged batch of prompts with the approximate log-sum-exp
        _case(name="prefill_ragged_b4_lse4", batch=4, seq=12289, seq_min=1500, rho=4),
        # a long document: the benchmark's headline workload
        _case(name="prefill_32k", seq=32768),
        # the longest document
        _case(name="prefill_128k", seq=131072),
        # fine-tuning on short sequences, eight query heads per key-value head, two sequences
        _case(name="train_4k_g8", kind="train", batch=2, seq=4096, seq_min=3333, hq=16, hkv=2, keep=False),
        # the backward of a long-document training step
        _case(name="backward_32k", kind="backward", seq=32768),
    ]


def _log_int(rng, lo, hi):
    return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "verify", "prefill", "prefill", "prefill", "train", "backward"])
    group = rng.choice([16, 16, 16, 8, 4, 2, 1])
    hkv = rng.choice([1, 2, 2, 4])
    c = dict(kind=kind, hq=group * hkv, hkv=hkv, topk=rng.choice([8, 12, 16, 16, 24, 32]))
    c["rho"] = rng.choice([1, 1, 1, 2, 4]) if group == 16 else 1
    c["keep"] = rng.random() < 0.6
    if kind in ("decode", "verify"):
        c["seq"] = _log_int(rng, 200, 131072)
        room = min(32, 8 * 131072 // (c["seq"] * hkv) * 4)           # at most what 32 sequences of 128K hold with two heads
        if kind == "decode":
            c["batch"] = _log_int(rng, 1, max(1, room))
            if c["batch"] == 1 and rng.random() < 0.5:
                c.update(layers=rng.randint(2, 6), graph=True, keep=True)
        else:
            c["batch"] = _log_int(rng, 1, 4)
            c["n_draft"] = rng.choice([2, 3, 4, 7, 8, 16, 16, 25, 32, 64])
            c["tree"] = rng.random() < 0.7
    else:
        # tokens x key-value heads bound the attention, tokens^2 x query heads the selection: both at most a fraction
        # of the largest listed case's
        most = {"prefill": 65536, "train": 16384, "backward": 32768}[kind] // hkv * 2
        if group < 16:
            most = min(most // 2, 16384)
        c["seq"] = _log_int(rng, 100, most)
        c["batch"] = _log_int(rng, 1, min(4, most // c["seq"])) if most >= 2 * c["seq"] else 1
    if c["batch"] > 1 and rng.random() < 0.7:
        c["seq_min"] = rng.randint(max(64, c["seq"] // 8), c["seq"]) if c["seq"] > 64 else c["seq"]
        c["heavy"] = rng.choice([0, 0, c["batch"] // 2])
    return _case(**c)


# ---- what a case means -----------------------------------------------------------------------------------------

def _lengths(c):
    b = c["batch"]
    if b == 1:
        return [c["seq"]]
    return [c["seq"] - (c["seq"] - c["seq_min"]) * i // (b - 1) for i in range(b)]


def _params(c):
    return binding.Params(c["hq"], c["hkv"], topk=c["topk"], lse_coarse_ratio=c["rho"])


def _kernels(n):
    return np.where(n < 32, 0, (n - 32) // 16 + 1)


# ---- inputs ----------------------------------------------------------------------------------------------------

def _planted_caches(c, lengths, cap, q_mean, gen):
    """k, v [batch, hkv, cap, D]; q_mean [batch, hkv, D]: the mean query row of each group."""
    b, h = c["batch"], c["hkv"]
    k = torch.zeros((b, h, cap, D), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros((b, h, cap, D), dtype=torch.bfloat16, device="cuda")
    u = q_mean / q_mean.norm(dim=-1, keepdim=True)
    for i, n in enumerate(lengths):
        k[i, :, :n].normal_(generator=gen)
        v[i, :, :n].normal_(generator=gen)
        last = n // BLOCK - 3
        count = min(last, max(2, n // 1024))
        if count > 0:
            rows = torch.arange(BLOCK, device="cuda")
            for j in range(h):
                at = torch.randperm(last, generator=gen, device="cuda")[:count] + 1
                eps = torch.randn((count * BLOCK, D), generator=gen, device="cuda")
                where = (at[:, None] * BLOCK + rows[None, :]).reshape(-1)
                k[i, j, where] = (D ** 0.5 * u[i, j][None, :] + 0.1 * eps).bfloat16()
        if i < c["heavy"]:
            z = torch.randn((h, n, 1), generator=gen, device="cuda")
            k[i, :, :n] = (k[i, :, :n].float() * torch.exp(z)).bfloat16()
    return k, v


def _group_mean(c, q):
    """q [batch, rows, hq, D] -> [batch, hkv, D]"""
    return q.float().mean(1).reshape(c["batch"], c["hkv"], -1, D).mean(2) if q.shape[1] <= 4096 else \
        q.mean(1, dtype=torch.float32).reshape(c["batch"], c["hkv"], -1, D).mean(2)


def _workspace(n):
    return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")


def _prepare_sequences(c, gen):
    lengths, cap, b = _lengths(c), c["seq"], c["batch"]
    prm = _params(c)
    q = torch.empty((b, cap, c["hq"], D), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    k, v = _planted_caches(c, lengths, cap, _group_mean(c, q), gen)
    s = {"c": c, "prm": prm, "q": q, "k": k, "v": v, "cap": cap,
         "sl": torch.tensor(lengths, dtype=torch.int32, device="cuda")}
    if c["kind"] != "prefill":
        s["dout"] = torch.empty_like(q).normal_(generator=gen)
    s["ck"] = s["idx"] = s["out"] = s["lse"] = s["ws_select"] = s["ws_attend"] = None
    s["dq"] = s["dk"] = s["dv"] = s["ws_backward"] = None
    if c["keep"]:
        s["ck"] = torch.zeros((b, c["hkv"], max(1, binding.num_kernels(cap, prm)), D), dtype=torch.bfloat16, device="cuda")
        s["idx"] = torch.full((b, c["hkv"], cap, c["topk"]), -1, dtype=torch.int32, device="cuda")
        s["out"] = torch.zeros_like(q)
        s["lse"] = torch.zeros((b, cap, c["hq"]), dtype=torch.float32, device="cuda")
        s["ws_select"] = _workspace(binding.workspace_bytes(binding.OP_SELECT_PREFILL, prm, b, cap))
        s["ws_attend"] = _workspace(binding.workspace_bytes(binding.OP_ATTN_PREFILL, prm, b, cap))
        if c["kind"] != "prefill":
            s["dq"], s["dk"], s["dv"] = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
            s["ws_backward"] = _workspace(binding.workspace_bytes(binding.OP_ATTN_BWD, prm, b, cap))
    if c["kind"] == "backward":
        s["idx"], s["out"], s["lse"] = _forward(s)[1:]
    return s


def _prepare_steps(c, gen):
    """decode and verify: caches that hold everything but the new tokens, per layer."""
    lengths, b, n = _lengths(c), c["batch"], c["n_draft"]
    prm = _params(c)
    cap = -(-(c["seq"] + 1) // 256) * 256
    sl = torch.tensor(lengths, dtype=torch.int32, device="cuda")
    layers = []
    verify = c["kind"] == "verify"
    ws = None
    if c["keep"]:
        ws = _workspace(binding.verify_workspace_bytes(binding.OP_VERIFY_STEP, prm, b, cap, n) if verify else
                        binding.workspace_bytes(binding.OP_DECODE_STEP, prm, b, cap))
    for _ in range(c["layers"]):
        q = torch.empty((b, n, c["hq"], D), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
        k, v = _planted_caches(c, [x - n for x in lengths], cap, _group_mean(c, q), gen)
        new = [torch.empty((b, c["hkv"], n, D), dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(2)]
        ck = torch.zeros((b, c["hkv"], max(1, binding.num_kernels(cap, prm)), D), dtype=torch.bfloat16, device="cuda")
        binding.compress_keys(prm, k, sl - n, cap, ck=ck)
        bufs = {}
        if c["keep"]:
            bufs = {"block_idx": torch.full((b, c["hkv"], n, c["topk"]), -1, dtype=torch.int32, device="cuda"),
                    "out": torch.zeros_like(q), "workspace": ws,
                    "lse": torch.zeros((b, n, c["hq"]) if verify else (b, c["hq"]), dtype=torch.float32, device="cuda")}
        layers.append((q, new[0], new[1], k, v, ck, bufs))
    mask = None
    if verify and c["tree"]:
        words = np.zeros((b, n), np.uint64)
        parents = torch.rand((b, n), generator=gen, device="cuda").cpu().numpy()
        for i in range(b):
            for t in range(n):                                  # token t: itself and its ancestors
                up = words[i, int(parents[i, t] * t)] if t else np.uint64(0)
                words[i, t] = up | (np.uint64(1) << np.uint64(t))
        mask = torch.from_numpy(words.view(np.int64)).cuda()
    s = {"c": c, "prm": prm, "cap": cap, "sl": sl, "layers": layers, "mask": mask, "graph": None}
    if c["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _steps(s)
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            s["result"] = _steps(s)
        s["graph"] = graph
    return s


def prepare(case, seed):
    c = dict(_FIELDS, **case)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    return _prepare_steps(c, gen) if c["kind"] in ("decode", "verify") else _prepare_sequences(c, gen)


# ---- one pass --------------------------------------------------------------------------------------------------

def _forward(s):
    prm, q, k, v, sl, cap = s["prm"], s["q"], s["k"], s["v"], s["sl"], s["cap"]
    ck = binding.compress_keys(prm, k, sl, cap, ck=s["ck"])
    idx = binding.select_blocks(prm, binding.MODE_PREFILL, q, ck, sl, cap, block_idx=s["idx"], workspace=s["ws_select"])
    out, lse = binding.sparse_attn_prefill(prm, q, k, v, sl, cap, idx, out=s["out"], lse=s["lse"], workspace=s["ws_attend"])
    return ck, idx, out, lse


def _backward(s, idx, out, lse):
    return binding.sparse_attn_bwd(s["prm"], s["q"], s["k"], s["v"], out, s["dout"], lse, s["sl"], s["cap"], idx,
                                   dq=s["dq"], dk=s["dk"], dv=s["dv"], workspace=s["ws_backward"])


def _steps(s):
    prm, sl, cap = s["prm"], s["sl"], s["cap"]
    results = []
    for q, k_new, v_new, k, v, ck, bufs in s["layers"]:
        if s["c"]["kind"] == "verify":
            r = binding.verify_step(prm, q, k_new, v_new, k, v, ck, sl, cap, tree_mask=s["mask"], **bufs)
        else:
            r = binding.decode_step(prm, q, k_new, v_new, k, v, ck, sl, cap, **bufs)
        results.append((r, k, v, ck))                           # the caches are updated in place
    return results


def run(state):
    kind = state["c"]["kind"]
    if kind in ("decode", "verify"):
        if state["graph"] is not None:
            state["graph"].replay()
            return state["result"]
        return _steps(state)
    if kind == "prefill":
        return _forward(state)
    if kind == "backward":
        return _backward(state, state["idx"], state["out"], state["lse"])
    ck, idx, out, lse = _forward(state)
    return ck, idx, out, lse, _backward(state, idx, out, lse)


# ---- what a pass cannot do without -----------------------------------------------------------------------------

def _attended(c, pos):
    """Keys attended by queries at positions pos: full lists of min(topk, own block + 1) blocks, causal in the own one."""
    own = pos // BLOCK
    return (np.minimum(c["topk"], own + 1) - 1) * BLOCK + pos % BLOCK + 1


def _scored(c, pos):
    """Semantic kernels a query has to score: none while every block is selected anyway."""
    n = np.where(pos // BLOCK + 1 > c["topk"], _kernels(pos + 1), 0)
    return n + (n // c["rho"] if c["rho"] > 1 else 0)


def work(case):
    c = dict(_FIELDS, **case)
    hq, hkv, n = c["hq"], c["hkv"], c["n_draft"]
    bytes_, flops = 0.0, 0.0
    for length in _lengths(c):
        if c["kind"] in ("decode", "verify"):
            pos = np.arange(length - n, length, dtype=np.int64)
            scored, seen = _scored(c, pos), _attended(c, pos)
            flops += float(scored.sum()) * hq * 2 * D + float(seen.sum()) * hq * 4 * D
            rows = (int(_kernels(np.int64(length))) if scored.max() > 0 else 0) + 2 * int(seen.max())
            bytes_ += c["layers"] * (rows * hkv * D * 2 + n * (2 * hq * D * 2 + 4 * hkv * D * 2 + hkv * c["topk"] * 4 + hq * 4))
            continue
        pos = np.arange(length, dtype=np.int64)
        pairs, scored = float(_attended(c, pos).sum()), float(_scored(c, pos).sum())
        qo, kv = length * hq * D * 2, length * hkv * D * 2
        small = length * (hkv * c["topk"] * 4 + hq * 4)
        if c["kind"] != "backward":
            bytes_ += 2 * qo + 2 * kv + small + int(_kernels(np.int64(length))) * hkv * D * 2
            flops += scored * hq * 2 * D + pairs * hq * 4 * D
        if c["kind"] != "prefill":                              # the backward reads q, out, dout, k, v, lse and the lists
            bytes_ += (4 if c["kind"] == "backward" else 2) * qo + (4 if c["kind"] == "backward" else 2) * kv + \
                (small if c["kind"] == "backward" else 0)
            flops += pairs * hq * 10 * D
    if c["kind"] in ("decode", "verify"):
        flops *= c["layers"]
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # bf16 results (outputs and gradients) of bf16 products with fp32 sums.  The log-sum-exps are fp32 and far closer;
    # the block lists are equal except where two blocks score the same to fp32 rounding, which moves a token's output
    # by less than its own size.
    return {"rel": 1e-2, "max": 0.5, "differ": 1e-3}
