"""Timed cases of the verification hot path, called as a decoding program calls it.

Three kinds of pass:
  iteration  one iteration of tree-based speculative decoding on the target's side: Hybrid Tree Attention on every
             layer over a capacity-sized KV cache (the last layer also leaves the chunk sums), greedy acceptance, chunk
             scores of the last accepted token with their top-k, the gather of the draft cache, and the commit of the
             accepted K/V rows
  attend     one attention layer of a draft model over its working cache
  prefill    causal self-attention of a prompt, or of a later piece of one
"""
import math
import random

import numpy as np
import torch

import paper_2505_20776_amd as sx
from workloads import chain_tree, eagle_style_tree, wide_tree

TREE_DEPTH = {"eagle": 6, "wide": 4}


def _iteration(name, **kw):
    case = dict(kind="iteration", dtype="bf16", out="bf16", layers=1, q_heads=32, kv_heads=8, head_dim=128,
                tree="eagle", nodes=60, chunk=32, top_k=32)
    case.update(kw)
    if name:
        case["name"] = name
    return case


def _attend(name, **kw):
    case = dict(kind="attend", dtype="bf16", out="bf16", layers=1, q_heads=32, kv_heads=8, head_dim=128, tree="eagle")
    case.update(kw)
    if name:
        case["name"] = name
    return case


def _prefill(name, **kw):
    case = dict(kind="prefill", dtype="bf16", out="bf16", q_heads=32, kv_heads=8, head_dim=128)
    case.update(kw)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the toy configuration: fp32, one layer of four heads of 64; all latency and launches
        _iteration("toy_f32", dtype="f32", out="f32", q_heads=4, kv_heads=1, head_dim=64, prefix=512, nodes=8, chunk=32,
                   top_k=4, tree="eagle"),
        # a Vicuna-68M-shaped draft layer checks a whole draft tree over its working cache of 1K tokens
        _attend("draft68m_1k", q_heads=12, kv_heads=12, head_dim=64, prefix=1024, nodes=60),
        # an EAGLE-style draft layer expands one level of the tree over its working cache of 2K tokens
        _attend("draft_level_2k", prefix=2048, nodes=8),
        # one layer of the target at a short prefix
        _iteration("layer_2k", prefix=2048),
        # one layer at a short prefix in fp32
        _iteration("layer_2k_f32", dtype="f32", out="f32", prefix=2048),
        # the retrieval parameter study: chunks smaller than the usual 32 tokens, a prefix that ends inside one
        _iteration("chunk16_4k", prefix=4096 + 13, chunk=16, top_k=64),
        # multi-head attention without grouping (Vicuna-7B / LongChat-7B targets), two layers, ragged prefix
        _iteration("multihead_8k", layers=2, kv_heads=32, prefix=8192 - 37, nodes=50),
        # the headline workload: all 32 layers of a Llama-3.1-8B-shaped target at a 16K prefix
        _iteration("step_16k", layers=32, prefix=16384),
        # a linear draft of 16 tokens behind a long ragged prefix: streaming the cache is all there is
        _iteration("chain16_32k", prefix=32768 - 37, tree="chain", nodes=16, chunk=64, top_k=16),
        # the largest tree behind the same prefix: matrix work
        _iteration("wide128_32k", prefix=32768 - 37, tree="wide", nodes=128, chunk=64, top_k=16),
        # a whole prompt
        _prefill("prefill_8k", q_len=8192, kv_len=8192),
        # a later piece of a long prompt that is processed in pieces
        _prefill("prefill_piece", q_len=512, kv_len=16384 - 21),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["iteration", "iteration", "iteration", "chunks", "f32", "small", "attend", "prefill", "prefill"])
    tree = rng.choice(["eagle", "eagle", "wide", "chain"])
    if what == "prefill":
        q_heads, kv_heads = rng.choice([(32, 8), (32, 8), (32, 32), (8, 2)])
        q_len = _log_int(rng, 64, 8192)
        kv_len = q_len if rng.random() < 0.5 else min(16384, q_len + _log_int(rng, 64, 16384))
        if kv_len != q_len:
            q_len = min(q_len, 2048)
        return _prefill(None, q_heads=q_heads, kv_heads=kv_heads, q_len=q_len, kv_len=max(kv_len, q_len),
                        out=rng.choice(["bf16", "bf16", "f32"]))
    if what == "attend":
        q_heads, kv_heads, d = rng.choice([(12, 12, 64), (32, 8, 128)])
        return _attend(None, q_heads=q_heads, kv_heads=kv_heads, head_dim=d, prefix=_log_int(rng, 256, 4096),
                       nodes=_log_int(rng, 1, 64), tree=tree)
    if what == "small":
        return _iteration(None, dtype="f32", out="f32", q_heads=rng.choice([4, 8]), kv_heads=rng.choice([1, 2]), head_dim=64,
                          prefix=_log_int(rng, 128, 2048), nodes=_log_int(rng, 2, 32), tree=tree,
                          chunk=rng.choice([16, 32]), top_k=rng.choice([4, 8]))
    if what == "f32":
        q_heads, kv_heads = rng.choice([(32, 8), (8, 2), (32, 32)])
        return _iteration(None, dtype="f32", out="f32", q_heads=q_heads, kv_heads=kv_heads, prefix=_log_int(rng, 512, 4096),
                          nodes=_log_int(rng, 1, 64), tree=tree, chunk=rng.choice([16, 32, 64]))
    if what == "chunks":
        return _iteration(None, prefix=_log_int(rng, 1024, 8192), nodes=_log_int(rng, 8, 64), tree=tree,
                          chunk=rng.choice([16, 48]), top_k=rng.choice([16, 32, 64]))
    kv_heads = rng.choice([8, 8, 32])
    prefix = _log_int(rng, 512, 131072 if kv_heads == 8 else 32768)
    return _iteration(None, layers=rng.choice([1, 1, 2]), kv_heads=kv_heads, prefix=prefix, nodes=_log_int(rng, 1, 128),
                      tree=tree, chunk=rng.choice([32, 32, 64]), top_k=rng.choice([16, 32, 64]),
                      out=rng.choice(["bf16", "bf16", "f32"]))


def _parents(case, seed):
    rng = np.random.default_rng(seed)
    n = case["nodes"]
    if case["tree"] == "chain" or n < 4:
        return chain_tree(n)
    if case["tree"] == "wide":
        return wide_tree(n, TREE_DEPTH["wide"], rng)
    return np.asarray(eagle_style_tree(n, TREE_DEPTH["eagle"], rng)[:n], dtype=np.int32)


def _tokens(parent, seed):
    """Drafted tokens (all different) and the target's choices: mostly one of the drafts below a node, as when the
    draft model is good; at the top the first root's token."""
    rng = random.Random(seed)
    n = len(parent)
    draft = rng.sample(range(1, 32000), n)
    target = []
    for i in range(n):
        below = [j for j in range(n) if parent[j] == i]
        target.append(draft[rng.choice(below)] if below and rng.random() < 0.8 else 0)
    return draft, target, draft[0]


def _dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _code(name):
    return sx.SPECEXT_BF16 if name == "bf16" else sx.SPECEXT_F32


class _Draw:
    """Seeded unit-variance values on the GPU (logits of standard deviation one, as attention has them)."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        self.dtype = dtype

    def __call__(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32).to(self.dtype)


def prepare(case, seed):
    torch.cuda.set_device(0)
    dt, odt = _dtype(case["dtype"]), _dtype(case["out"])
    rand = _Draw(seed, dt)
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    if case["kind"] == "prefill":
        tq, n = case["q_len"], case["kv_len"]
        return {"case": case, "q": rand(tq, hq, d), "k": rand(hkv, n, d), "v": rand(hkv, n, d),
                "out": torch.empty((tq, hq, d), dtype=odt, device="cuda"),
                "lse": torch.empty((hq, tq), dtype=torch.float32, device="cuda")}

    layers, plen, t = case["layers"], case["prefix"], case["nodes"]
    parent = _parents(case, seed)
    cap = plen + t
    state = {"case": case, "parent": torch.from_numpy(parent).cuda(),
             "k_cache": torch.empty((layers, hkv, cap, d), dtype=dt, device="cuda"),
             "v_cache": torch.empty((layers, hkv, cap, d), dtype=dt, device="cuda"),
             "q": rand(layers, t, hq, d), "k_tree": rand(layers, hkv, t, d), "v_tree": rand(layers, hkv, t, d),
             "out": torch.empty((layers, t, hq, d), dtype=odt, device="cuda"),
             "lse": torch.empty((layers, hq, t), dtype=torch.float32, device="cuda")}
    for y in range(layers):
        state["k_cache"][y] = rand(hkv, cap, d)
        state["v_cache"][y] = rand(hkv, cap, d)
    # every layer of a model holds its own tensors
    state["layers"] = [tuple(state[name][y] for name in ("q", "k_cache", "v_cache", "k_tree", "v_tree", "out", "lse"))
                       for y in range(layers)]
    common = dict(dtype=_code(case["dtype"]), out_dtype=_code(case["out"]), n_q_heads=hq, n_kv_heads=hkv, head_dim=d,
                  prefix_len=plen, n_tree=t, kp_stride_h=cap * d, kp_stride_l=d)
    state["desc"] = sx.make_desc(**common)
    if case["kind"] == "attend":
        state["workspace"] = torch.empty(sx.workspace_bytes(state["desc"]), dtype=torch.uint8, device="cuda")
        return state

    # the relevant chunks: the queries of a KV head's group share a direction that the keys of top_k chunks point along
    # too, so that these chunks score several times the others, which is what retrieval is for
    chunk, n_chunks = case["chunk"], -(-plen // case["chunk"])
    k = min(case["top_k"], n_chunks)
    along = torch.nn.functional.normalize(torch.randn((hkv, d), generator=rand.gen, device="cuda"), dim=-1)
    state["q"][-1] += (6.0 * along).repeat_interleave(hq // hkv, dim=0).to(dt)
    for c in random.Random(seed).sample(range(n_chunks), k):
        state["k_cache"][-1][:, c * chunk:min((c + 1) * chunk, plen)] += (4.0 * along).to(dt)[:, None, :]

    draft, target, first = _tokens(parent, seed)
    ints = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")  # noqa: E731
    kept = case["top_k"] * chunk
    state.update(
        top_k=case["top_k"], cap=cap, kept=kept,
        desc_scores=sx.make_desc(chunk_size=chunk, want_scores=True, **common),
        draft_token=ints(draft), target_token=ints(target), first_target=ints([first]),
        path=torch.empty(t, dtype=torch.int32, device="cuda"), n_accept=torch.empty(1, dtype=torch.int32, device="cuda"),
        next_token=torch.empty(1, dtype=torch.int32, device="cuda"),
        scores=torch.empty(n_chunks, dtype=torch.float32, device="cuda"),
        idx=torch.empty(case["top_k"], dtype=torch.int32, device="cuda"),
        n_idx=torch.empty(1, dtype=torch.int32, device="cuda"),
        # the draft model's cache: one layer of the target's KV shape, compacted into a working cache
        draft_k=rand(1, hkv, cap, d), draft_v=rand(1, hkv, cap, d),
        work_k=torch.zeros((1, hkv, kept, d), dtype=dt, device="cuda"),
        work_v=torch.zeros((1, hkv, kept, d), dtype=dt, device="cuda"),
        pos=torch.empty(kept, dtype=torch.int32, device="cuda"), length=torch.empty(1, dtype=torch.int32, device="cuda"))
    # all that the commit may write: every cache row behind the prefix
    state["k_new"], state["v_new"] = state["k_cache"][:, :, plen:], state["v_cache"][:, :, plen:]
    size = max(sx.workspace_bytes(state["desc"]), sx.workspace_bytes(state["desc_scores"]))
    state["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    return state


def run(state):
    s, case = state, state["case"]
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    if case["kind"] == "prefill":
        sx.prefill_attn(s["q"], s["k"], s["v"], s["out"], s["lse"], hq, hkv, d, case["q_len"], case["kv_len"],
                        dtype=_code(case["dtype"]), out_dtype=_code(case["out"]))
        return {"out": s["out"], "lse": s["lse"]}
    layers = case["layers"]
    last = layers - 1 if case["kind"] == "iteration" else -1
    parent, workspace = s["parent"], s["workspace"]
    for y, (q, k_cache, v_cache, k_tree, v_tree, out, lse) in enumerate(s["layers"]):
        sx.verify_attn(s["desc_scores"] if y == last else s["desc"], q, k_cache, v_cache, k_tree, v_tree, parent, out, lse,
                       workspace)
    if case["kind"] == "attend":
        return {"out": s["out"], "lse": s["lse"]}
    plen, t = case["prefix"], case["nodes"]
    elem = s["k_cache"].element_size()
    sx.accept_greedy(s["parent"], s["draft_token"], s["target_token"], s["first_target"], t, s["path"], s["n_accept"],
                     s["next_token"])
    sx.chunk_scores_select(s["desc_scores"], s["workspace"], 0, s["top_k"], s["idx"], s["n_idx"], scores=s["scores"],
                           path=s["path"], n_accept=s["n_accept"])
    sx.gather_draft_kv(s["draft_k"], s["draft_v"], s["work_k"], s["work_v"], s["idx"], s["n_idx"], s["top_k"], 1, hkv, plen,
                       s["kept"], d, case["chunk"], elem, s["pos"], s["length"], src_cap=s["cap"])
    sx.commit_tree_kv(s["k_tree"], s["v_tree"], s["k_cache"], s["v_cache"], s["path"], s["n_accept"], t, t, layers, hkv, d,
                      elem, plen, s["cap"])
    return {"out": s["out"], "lse": s["lse"], "path": s["path"], "n_accept": s["n_accept"], "next_token": s["next_token"],
            "scores": s["scores"], "idx": s["idx"], "n_idx": s["n_idx"], "work_k": s["work_k"], "work_v": s["work_v"],
            "pos": s["pos"], "length": s["length"], "k_new": s["k_new"], "v_new": s["v_new"]}


def work(case):
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    ein, eout = (2 if case["dtype"] == "bf16" else 4), (2 if case["out"] == "bf16" else 4)
    if case["kind"] == "prefill":
        tq, n = case["q_len"], case["kv_len"]
        pairs = tq * (n - tq) + tq * (tq + 1) // 2
        return {"bytes": tq * hq * d * (ein + eout) + 2 * hkv * n * d * ein + 4 * hq * tq, "flops": 4 * d * hq * pairs}
    layers, plen, t = case["layers"], case["prefix"], case["nodes"]
    row = t * hq * d
    total = layers * (2 * hkv * (plen + t) * d * ein + row * (ein + eout) + 4 * hq * t)
    if case["kind"] == "iteration":
        n_chunks = -(-plen // case["chunk"])
        kept = min(case["top_k"], n_chunks) * case["chunk"]
        total += 4 * n_chunks + 2 * 2 * hkv * min(kept, plen) * d * ein
    return {"bytes": total, "flops": layers * 4 * d * hq * t * plen}


def tolerance(case):
    # Four times the distance of output, log-sum-exp and chunk scores from the same attention in 64 bits.  2-norm: 9e-7 with
    # fp32 inputs, 2.4e-3 with bf16 ones (probabilities and results are rounded to bf16).  Largest difference: 1e-5 and
    # 1.5e-2; 5.4e-2 in a prompt, whose first rows are far larger than the mean one.  Tokens, chunk indices, positions and
    # copied rows are the same.
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 9e-3, "max": 0.2 if case["kind"] == "prefill" else 6e-2}
