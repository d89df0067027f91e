"""The work that a training or evaluation program has this package do, as cases that can be timed.

A case is a dict of plain values.  `what` says which calls one pass makes:

  train    one context-parallel rank's attention in a training step: schedule, forward, backward
  layers   the same for several layers that share one mask, hence one schedule
  step     a training step that starts from document lengths: sharding map, upload, schedule, forward, backward
  forward  schedule and forward only (evaluation)
  static   the forward for callers that may not allocate or hand over a workspace
  pack     the streaming packer over a pool of documents (host)

and the rest which documents, heads, head dimension and sharding it makes them for.  Document lengths
come from the recipes of `workloads.py` with a seed that belongs to the case, tensors are i.i.d. N(0, 1)
in bf16 drawn on the GPU from the seed given to `prepare`.
"""
import math

import numpy as np
import torch

from paper_2503_17924_amd import binding as B
from paper_2503_17924_amd import workloads as wl

WINDOW = 131072               # context window of the packing pool
COST_A, COST_B = 6, 640000    # packer cost model: picoseconds per token^2 and per token
PADDED, PER_SEQ, NOPAD = B.SHARD_PER_DOC_PADDED, B.SHARD_PER_SEQ, B.SHARD_PER_DOC_NOPAD


def _case(what, mix, doc_seed, tokens, lo, hi, hq, hkv, d, cp=1, rank=0, mode=PADDED, layers=1, **extra):
    return dict(extra, what=what, mix=mix, doc_seed=doc_seed, tokens=tokens, lo=lo, hi=hi, hq=hq, hkv=hkv, d=d, cp=cp, rank=rank,
                mode=mode, layers=layers)


def listed():
    return [
        # a 128K-token micro-batch on one of eight context-parallel ranks, one tensor-parallel share of a 70B-class
        # layer: the package's main workload
        _case("train", "mixture", 2, 131072, 16384, 131072, 8, 1, 128, cp=8, rank=3, name="train_128k_cp8"),
        # the largest pass: a 98304-token document followed by 979 tiny ones, all rows on one rank
        _case("train", "straggler", 4, 131072, 1, 64, 16, 2, 128, name="train_128k_straggler"),
        # a 32K-token micro-batch of an 8B-class layer without context parallelism
        _case("train", "mixture", 1, 32768, 8192, 32768, 32, 8, 128, name="train_32k_gqa"),
        # a 64K-token window with as many KV heads as query heads, two ranks
        _case("train", "mixture", 5, 65536, 8192, 65536, 8, 8, 128, cp=2, rank=1, name="train_64k_mha_cp2"),
        # the small-document regime (bound by memory): nothing but documents of 1 to 64 tokens
        _case("train", "uniform", 4, 32768, 1, 64, 16, 2, 128, name="train_tiny_docs"),
        # the same documents divided among four ranks: chunks of at most 8 tokens
        _case("train", "uniform", 4, 32768, 1, 64, 16, 2, 128, cp=4, rank=1, name="train_tiny_docs_cp4"),
        # head dimension 64 under contiguous (per-sequence) sharding, the baseline the sharding is compared with
        _case("train", "mixture", 2, 131072, 16384, 131072, 8, 1, 64, cp=8, rank=5, mode=PER_SEQ, name="train_128k_d64_per_seq"),
        # a short micro-batch of odd length in a model of four layers: one schedule, four forwards, four backwards
        _case("layers", "uniform", 7, 8191, 64, 1536, 8, 2, 128, layers=4, name="layers_8k"),
        # every micro-batch has documents of its own: sharding map without padding, upload and everything after it
        _case("step", "mixture", 8, 16381, 1024, 16384, 16, 4, 128, cp=4, rank=2, mode=NOPAD, name="step_16k_cp4_nopad"),
        # the smallest call: evaluation of 4096 tokens in short documents, head dimension 64, one of two ranks
        _case("forward", "uniform", 0, 4096, 64, 1536, 4, 4, 64, cp=2, rank=0, name="forward_4k_d64_cp2"),
        # evaluation under the no-allocation rule (graph capture, serving): 16K tokens, every call with its own mask
        _case("static", "mixture", 9, 16384, 1024, 16384, 32, 8, 128, name="forward_static_16k"),
        # the packer over a pool of 2000 documents in global batches of 8 windows, two waiting queues
        dict(name="pack_pool", what="pack", doc_seed=3, docs=2000, lo=8192, hi=131072, microbatches=8, queues=2),
    ]


_HEADS = [(4, 4), (8, 1), (8, 2), (8, 8), (16, 2), (16, 4), (32, 8)]


def draw(rng):
    what = rng.choice(["train"] * 6 + ["layers", "step", "forward", "forward", "static", "pack"])
    if what == "pack":
        return dict(what="pack", doc_seed=rng.randrange(1, 10**6), docs=int(math.exp(rng.uniform(math.log(100), math.log(2000)))), lo=8192, hi=131072,
                    microbatches=rng.choice([4, 8, 16]), queues=rng.choice([0, 1, 2]))
    most = {"layers": 16384, "static": 65536}.get(what, 131072)
    while True:
        tokens = int(math.exp(rng.uniform(math.log(1024), math.log(most))))
        mix = rng.choice(["mixture", "mixture", "uniform", "uniform", "straggler"])
        if mix == "mixture":
            lo, hi = max(tokens // 8, 2), max(tokens, 4)
        elif mix == "straggler":
            lo, hi = 1, 64
        else:
            lo, hi = rng.choice([(1, 64), (64, 1536), (500, 9000)])
        hq, hkv = rng.choice(_HEADS)
        cp = 1 if what == "static" else rng.choice([1, 1, 2, 4, 8])
        mode = rng.choice([PADDED, PADDED, NOPAD, PER_SEQ]) if cp > 1 else PADDED
        if mode == PER_SEQ:
            tokens -= tokens % (2 * cp)
        case = _case(what, mix, rng.randrange(1, 10**6), tokens, lo, min(hi, tokens), hq, hkv, rng.choice([64, 128, 128]), cp=cp,
                     rank=rng.randrange(cp), mode=mode, layers=4 if what == "layers" else 1)
        # no more than the largest listed case (4.83e9 pairs x 16 heads of 128)
        if _flops(case, _shard(case)["useful_pairs"]) <= 14 * 128 * 16 * 4.8e9:
            return case


def _docs(case):
    if case["mix"] == "mixture":
        return wl.mixture_docs_fill(case["doc_seed"], case["tokens"], case["lo"], case["hi"])
    if case["mix"] == "straggler":
        return wl.straggler_docs(case["doc_seed"], case["tokens"], case["tokens"] * 3 // 4, case["lo"], case["hi"])
    return wl.uniform_docs_until_overflow(case["doc_seed"], case["tokens"], case["lo"], case["hi"])


def _shard(case):
    return B.wlb_shard(_docs(case), case["cp"], case["rank"], case["mode"])


def _backward(case):
    return case["what"] in ("train", "layers", "step")


def _flops(case, pairs):
    """4 D per visible (query, key) pair and query head forward, 10 D backward."""
    return (14 if _backward(case) else 4) * case["d"] * case["hq"] * pairs * case["layers"]


def _pool(case, seed):
    """The case's documents, in an order of arrival that the seed gives."""
    return np.random.default_rng(seed).permutation(wl.mixture_pool(case["doc_seed"], case["docs"], case["lo"], case["hi"]))


def _global_batches(case, lengths):
    """The pool in arrival order, cut into global batches of `microbatches` windows' worth of tokens."""
    batch = np.cumsum(lengths.astype(np.int64)) // (case["microbatches"] * WINDOW)
    return np.split(lengths, np.searchsorted(batch, np.arange(1, batch[-1] + 1)))


def prepare(case, seed):
    if case["what"] == "pack":
        batches = _global_batches(case, _pool(case, seed))
        first = np.concatenate([[0], np.cumsum([len(b) for b in batches])])
        ids = [np.arange(first[i], first[i] + len(b), dtype=np.int64) for i, b in enumerate(batches)]
        thresholds = [WINDOW // 2, WINDOW * 3 // 4][:case["queues"]]
        # which step and micro-batch each document goes to (-1: still waiting at the end), and the micro-batches' costs
        return dict(case=case, batches=batches, ids=ids, thresholds=thresholds, step=np.empty(case["docs"], dtype=np.int32),
                    microbatch=np.empty(case["docs"], dtype=np.int32), cost=np.empty((len(batches), case["microbatches"]), dtype=np.int64))
    docs = _docs(case)
    sh = B.wlb_shard(docs, case["cp"], case["rank"], case["mode"])
    n_q, t, hq, hkv, d = len(sh["q_idx"]), int(sh["cu_seqlens_k"][-1]), case["hq"], case["hkv"], case["d"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    bf = torch.bfloat16

    def normal(n, h):
        return torch.randn((n, h, d), device="cuda", generator=gen, dtype=bf)

    layers = []
    for _ in range(case["layers"]):
        x = dict(q=normal(n_q, hq), k=normal(t, hkv), v=normal(t, hkv), o=torch.empty((n_q, hq, d), dtype=bf, device="cuda"),
                 lse=torch.empty((hq, n_q), dtype=torch.float32, device="cuda"))
        if _backward(case):
            x.update(do=normal(n_q, hq), dq=torch.empty_like(x["q"]), dk=torch.empty_like(x["k"]), dv=torch.empty_like(x["v"]))
        layers.append(x)
    state = dict(case=case, docs=docs, layers=layers, scale=1.0 / math.sqrt(d), t=t)
    if case["what"] == "static":
        state["q_idx"] = torch.from_numpy(sh["q_idx"]).cuda()
        state["cu"] = torch.from_numpy(sh["cu_seqlens_k"]).cuda()
        state["desc"] = B.AttnDesc(n_q, t, len(docs), hq, hkv, d, state["scale"], 0, sh["useful_pairs"])
    elif case["what"] != "step":
        state["attn"] = B.Attention(sh["q_idx"], sh["cu_seqlens_k"], t, hq, hkv, d, state["scale"], visible_pairs=sh["useful_pairs"])
    return state


def run(state):
    case = state["case"]
    if case["what"] == "pack":
        packer = B.Packer(case["microbatches"], WINDOW * 3 // 2, COST_A, COST_B, state["thresholds"])
        state["step"].fill(-1)
        state["microbatch"].fill(-1)
        for i, (ids, lengths) in enumerate(zip(state["ids"], state["batches"])):
            placed, _, microbatch, _, cost = packer.step(ids, lengths)
            state["step"][placed] = i
            state["microbatch"][placed] = microbatch
            state["cost"][i] = cost
        packer.close()
        return state["step"], state["microbatch"], state["cost"]
    x = state["layers"][0]
    if case["what"] == "static":
        B.wlb_attn_fwd_static(state["desc"], x["q"], x["k"], x["v"], state["q_idx"], state["cu"], x["o"], x["lse"])
        return x["o"], x["lse"]
    if case["what"] == "step":
        sh = B.wlb_shard(state["docs"], case["cp"], case["rank"], case["mode"])
        attn = B.Attention(sh["q_idx"], sh["cu_seqlens_k"], state["t"], case["hq"], case["hkv"], case["d"], state["scale"],
                           visible_pairs=sh["useful_pairs"])
    else:
        attn = state["attn"]
    attn.plan()
    for x in state["layers"]:
        attn.forward(x["q"], x["k"], x["v"], x["o"], x["lse"])
    if not _backward(case):
        return x["o"], x["lse"]
    for x in reversed(state["layers"]):
        attn.backward(x["q"], x["k"], x["v"], x["o"], x["lse"], x["do"], x["dq"], x["dk"], x["dv"])
    return [[x[name] for name in ("o", "lse", "dq", "dk", "dv")] for x in state["layers"]]


def work(case):
    if case["what"] == "pack":
        # length and id in; id, length and micro-batch out
        return {"bytes": case["docs"] * (4 + 8 + 8 + 4 + 4), "flops": 0}
    sh = _shard(case)
    n_q, t = len(sh["q_idx"]), int(sh["cu_seqlens_k"][-1])
    row, token = 2 * case["hq"] * case["d"], 2 * case["hkv"] * case["d"]    # bytes of a row of Q and of K
    size = n_q * (2 * row + 4 * case["hq"]) + t * 2 * token                 # Q, O, LSE; K, V
    if _backward(case):
        # the backward cannot start before the forward has ended: Q, O, dO, dQ, LSE; K, V, dK, dV
        size += n_q * (4 * row + 4 * case["hq"]) + t * 4 * token
    return {"bytes": size * case["layers"] + 4 * n_q, "flops": _flops(case, sh["useful_pairs"])}


def tolerance(case):
    if case["what"] == "pack":
        return "exact"
    # against the same attention in float64, over head dimensions, document mixes and shardings: outputs are off by 1.8e-3 to
    # 3.2e-3 (2-norm) and by at most 7.5e-2 in one element (probabilities and their gradients are bf16 operands)
    return {"rel": 1e-2, "max": 0.3}
