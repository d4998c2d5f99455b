"""What the speed of this library is judged by: calls that a block-diffusion decoder makes, one layer at a time.

A decoder that generates `gen` tokens after `prompt` tokens works through blocks of `block` positions.  For each block and
layer it makes one or two dense steps (the block's rows of attention over the whole sequence; the last of them also scores,
selects and copies the keys that the rest of the block will see) and then some thirty steps over the retained keys and the
block's own.  Kinds of a case:

  reuse   one sdllm_block_step of cache state 2: attention of the block's queries over the retained cache and the block
  full    one of state 0: the block's rows of dense attention over all keys
  update  one of state 1: the same plus scoring, pooling, top-k and compaction; the cache is part of the result
  block   all denoising steps of one block of one layer: state 0, state 1, then state 2 to the end
  score   sdllm_score_select on its own (cache managers that run their own attention), with the pooled scores
  dense   sdllm_dense_attn: every position over every position, which the rows outside the block need at states 0 and 1

Head counts and sizes are those of the repository's workloads (32 / 32 and 28 / 4 heads of 128), its tests (other groups,
head dimension 64, fp32, block lengths other than 32, odd prompts) and powers of two near them.
"""
import math

import torch

from paper_2508_02558_amd import binding as B

DEVICE = "cuda"
TYPES = {"bf16": (torch.bfloat16, 2, B.SDLLM_BF16), "f32": (torch.float32, 4, B.SDLLM_F32)}


def _case(kind, batch, q_heads, kv_heads, prompt, gen, **more):
    c = dict(kind=kind, batch=batch, q_heads=q_heads, kv_heads=kv_heads, head_dim=128, dtype="bf16", block=32, prompt=prompt,
             gen=gen, block_index=0, retention=0.5, pool=3, score="softmax_mean", select="per_segment", steps=1)
    c.update(more)
    return c


def listed():
    return [
        # the thirty-of-32 steps, from the smallest call (one sequence, 1k prompt: latency and launches) ...
        _case("reuse", 1, 32, 32, 1024, 256, name="reuse_mha_b1"),
        # ... over grouped-query heads and a batch ...
        _case("reuse", 8, 28, 4, 4096, 512, block_index=5, name="reuse_gqa_b8"),
        # ... to the repository's benchmark shape
        _case("reuse", 8, 32, 32, 4096, 256, name="reuse_mha_b8"),
        # a whole block of one layer at batch 1: what a single user's decoding is made of
        _case("block", 1, 28, 4, 4096, 256, block_index=3, steps=32, name="block_gqa_b1"),
        # cache rebuild: a small batch with odd lengths and the block off the tile grid; the benchmark shape; a long document
        _case("update", 3, 32, 32, 2037, 256, block_index=2, pool=5, name="update_mha_b3_odd"),
        _case("update", 8, 32, 32, 4096, 256, name="update_mha_b8"),
        _case("update", 1, 28, 4, 32768, 512, retention=0.25, name="update_gqa_long"),
        # dense block rows of grouped-query heads, 512-token generation
        _case("full", 8, 28, 4, 4096, 512, block_index=9, name="full_gqa_b8"),
        # block length 64, which some generation settings use
        _case("update", 2, 32, 32, 1024, 256, block=64, block_index=1, name="update_mha_block64"),
        # single precision, head dimension 64: the reference runs people compare against, at the smallest size
        _case("reuse", 1, 2, 2, 64, 96, head_dim=64, dtype="f32", name="reuse_f32_tiny"),
        # all rows of the sequence: a batch of 4k prompts, and one odd short sequence
        _case("dense", 8, 32, 32, 4096, 256, name="dense_mha_b8"),
        _case("dense", 1, 28, 4, 1181, 96, name="dense_gqa_odd"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["reuse"] * 4 + ["update"] * 3 + ["full", "block", "score", "dense", "dense"])
    q_heads, kv_heads = rng.choice([(32, 32), (32, 32), (28, 4), (28, 4), (32, 8), (16, 2), (12, 4), (8, 8)])
    c = _case(kind, _log_int(rng, 1, 8), q_heads, kv_heads, _log_int(rng, 100, 8000), rng.choice([192, 384, 576]))
    form = rng.random()
    if form < 0.15:
        c["block"] = rng.choice([8, 16, 24, 48, 64])
    elif form < 0.23:
        c["head_dim"] = 64
    elif form < 0.30:
        c.update(dtype="f32", head_dim=rng.choice([64, 128]))
    elif form < 0.42 and kind != "dense":
        # long documents, one sequence, grouped-query heads
        c.update(batch=1, q_heads=28, kv_heads=4, prompt=_log_int(rng, 8000, 32000), retention=0.25)
    if form < 0.30:
        c.update(batch=_log_int(rng, 1, 2), q_heads=8 if q_heads == kv_heads else 2 * q_heads // kv_heads,
                 kv_heads=8 if q_heads == kv_heads else 2, prompt=_log_int(rng, 60, 1000))
    c["block_index"] = rng.randrange(c["gen"] // c["block"])
    if c["retention"] == 0.5:
        c["retention"] = rng.choice([0.5, 0.5, 0.3, 0.7])
    c["pool"] = rng.choice([3, 3, 1, 5, 7])
    if kind == "block":
        c["steps"] = rng.choice([8, 16, 32])
        c["batch"] = min(c["batch"], 2)
    if kind == "dense":
        while c["batch"] > 1 and c["batch"] * c["q_heads"] * (c["prompt"] + c["gen"]) ** 2 > 8 * 32 * 4352 ** 2:
            c["batch"] -= 1
    if kind in ("update", "score") and rng.random() < 0.35:
        # the paper's algorithm taken literally: raw logits, one ranking over both sides of the block
        c.update(score="logit_mean", select="joint")
    return c


# ------------------------------------------------------------------ shapes and inputs
def _sizes(c):
    seq = c["prompt"] + c["gen"]
    off = c["prompt"] + c["block_index"] * c["block"]
    return seq, off, seq - off - c["block"]


def _kept(c):
    """(prefix quota, suffix quota), or (total, None) when both sides are ranked as one."""
    _, off, suf = _sizes(c)
    if c["select"] == "joint":
        return math.floor(c["retention"] * (off + suf) + 1e-9), None
    return math.ceil(c["retention"] * off - 1e-9), math.ceil(c["retention"] * suf - 1e-9)


def _shape(c):
    seq, off, _ = _sizes(c)
    return B.make_shape(batch=c["batch"], n_q_heads=c["q_heads"], n_kv_heads=c["kv_heads"], head_dim=c["head_dim"],
                        seq_len=seq, block_off=off, block_len=c["block"], dtype=TYPES[c["dtype"]][2], retention=c["retention"],
                        pool_kernel=c["pool"],
                        score_mode=B.SDLLM_SOFTMAX_MEAN if c["score"] == "softmax_mean" else B.SDLLM_LOGIT_MEAN,
                        select_mode=B.SDLLM_PER_SEGMENT if c["select"] == "per_segment" else B.SDLLM_JOINT,
                        k_rounding=B.SDLLM_CEIL if c["select"] == "per_segment" else B.SDLLM_FLOOR)


def _inputs(c, seed):
    """Queries, full-sequence K/V, the block's K/V of every step: normal values; two keys in a hundred lie along a direction
    that the queries lean to and stay salient for every query and step, which is what retention is for."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    t = TYPES[c["dtype"]][0]
    bt, hq, hkv, d, b = c["batch"], c["q_heads"], c["kv_heads"], c["head_dim"], c["block"]
    seq, off, _ = _sizes(c)

    def randn(*shape):
        return torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32)

    k, v, lean = randn(bt, hkv, seq, d), randn(bt, hkv, seq, d), randn(bt, hkv, 1, d)
    lean /= lean.norm(dim=-1, keepdim=True)
    salient = torch.rand((seq, 1), generator=g, device=DEVICE) < 0.02
    salient[off:off + b] = False
    k = torch.where(salient, 3.0 * k.norm(dim=-1, keepdim=True) * lean, k)
    lean = 0.5 * lean.repeat_interleave(hq // hkv, dim=1)
    rows = seq if c["kind"] == "dense" else b
    q = [(randn(bt, hq, rows, d) + lean).to(t) for _ in range(c["steps"])]
    blk = [(randn(bt, hkv, b, d).to(t), randn(bt, hkv, b, d).to(t)) for _ in range(c["steps"])]
    return dict(k=k.to(t), v=v.to(t), q=q, blk=blk, salient=salient[:, 0], g=g)


def _cache(c, x):
    """A retained cache for cases that start with one: the salient keys and a random choice of the others, ascending."""
    _, off, suf = _sizes(c)
    bt, hkv, d = c["batch"], c["kv_heads"], c["head_dim"]
    rank = torch.rand((bt, hkv, x["k"].shape[2]), generator=x["g"], device=DEVICE) + x["salient"]
    quota = _kept(c)
    parts = [rank[..., :off].topk(quota[0]).indices, rank[..., off + c["block"]:].topk(quota[1]).indices + off + c["block"]]
    idx = torch.cat(parts, dim=-1).sort(dim=-1).values[..., None].expand(-1, -1, -1, d)
    return x["k"].gather(2, idx), x["v"].gather(2, idx)


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    s = dict(case=c, shape=_shape(c), q=x["q"], k=x["k"], v=x["v"], blk=x["blk"])
    t = TYPES[c["dtype"]][0]
    if c["kind"] == "dense":
        s["out"] = torch.empty_like(x["q"][0])
        return s
    bt, hkv, d = c["batch"], c["kv_heads"], c["head_dim"]
    kept = sum(n or 0 for n in _kept(c))
    op = B.SDLLM_OP_SCORE_SELECT if c["kind"] == "score" else B.SDLLM_OP_BLOCK_STEP
    cache_rows = max(1, kept)
    s["shape"].cache_stride[:] = (hkv * cache_rows * d, cache_rows * d, d)
    s["ws"] = torch.empty(B.sdllm_workspace_bytes(s["shape"], op), dtype=torch.uint8, device=DEVICE)
    s["idx"] = torch.zeros((bt, hkv, kept), dtype=torch.int32, device=DEVICE)
    if c["kind"] == "score":
        n = x["k"].shape[2] - c["block"]
        s["pooled"], s["score"] = (torch.empty((bt, hkv, n), dtype=torch.float32, device=DEVICE) for _ in range(2))
        return s
    s["out"] = [torch.empty_like(q) for q in x["q"]]
    if c["kind"] == "reuse":
        s["kc"], s["vc"] = _cache(c, x)
    else:
        s["kc"], s["vc"] = (torch.empty((bt, hkv, cache_rows, d), dtype=t, device=DEVICE) for _ in range(2))
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "dense":
        B.sdllm_dense_attn(s["shape"], s["q"][0], s["k"], s["v"], s["out"])
        return s["out"]
    if kind == "score":
        B.sdllm_score_select(s["shape"], s["q"][0], s["k"], s["idx"], s["pooled"], s["score"], s["ws"])
        return {"idx": s["idx"], "pooled": s["pooled"], "score": s["score"]}
    first = {"full": 0, "update": 1, "reuse": 2, "block": 0}[kind]
    for t in range(c["steps"]):
        k_in, v_in = (s["k"], s["v"]) if first + t < 2 else s["blk"][t]
        B.sdllm_block_step(s["shape"], first + t, 1, s["q"][t], k_in, v_in, s["idx"], s["kc"], s["vc"], s["out"][t], s["ws"])
    if kind in ("reuse", "full"):
        return s["out"][0]
    return {"out": s["out"], "idx": s["idx"], "k_cache": s["kc"], "v_cache": s["vc"]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    seq, off, suf = _sizes(c)
    e = TYPES[c["dtype"]][1]
    bt, hq, hkv, d, b = c["batch"], c["q_heads"], c["kv_heads"], c["head_dim"], c["block"]
    kept = sum(n or 0 for n in _kept(c))
    q_out = 2 * bt * hq * b * d * e

    def attend(keys):
        return q_out + 2 * bt * hkv * keys * d * e, 4 * bt * hq * b * keys * d

    rebuild = bt * hkv * kept * (2 * d * e + 4)
    if c["kind"] == "dense":
        return {"bytes": 2 * bt * (hq + hkv) * seq * d * e, "flops": 4 * bt * hq * seq * seq * d}
    if c["kind"] == "score":
        n = off + suf
        logits = 2 * bt * hq * b * n * d if c["score"] == "softmax_mean" else 2 * bt * hkv * n * d
        return {"bytes": q_out // 2 + bt * hkv * (n * (d * e + 8) + kept * 4), "flops": logits}
    dense, sparse = attend(seq), attend(kept + b)
    if c["kind"] == "reuse":
        return {"bytes": sparse[0], "flops": sparse[1]}
    if c["kind"] == "full":
        return {"bytes": dense[0], "flops": dense[1]}
    if c["kind"] == "update":
        return {"bytes": dense[0] + rebuild, "flops": dense[1]}
    n = c["steps"] - 2
    return {"bytes": 2 * dense[0] + rebuild + n * sparse[0], "flops": 2 * dense[1] + n * sparse[1]}


def tolerance(case):
    # bf16: probabilities are rounded to 8 bits before the second product and results once more (measured: 1.7e-3 to 2.5e-3
    # against 64 bits); fp32: sums in another order.  Whole values are retained positions: two candidates whose scores agree
    # to the last bits may change places, which moves the positions between them by one.
    if case["kind"] == "score" or case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.01}
    return {"rel": 8e-3, "max": 0.1, "differ": 0.01}


# ------------------------------------------------------------------ the same in 64 bits
def _attend(q, k, v, group, step=1024):
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    for i in range(q.shape[0]):
        for h in range(q.shape[1]):
            kk, vv = k[i, h // group].double(), v[i, h // group].double()
            for r in range(0, q.shape[2], step):
                a = (q[i, h, r:r + step].double() @ kk.T) / math.sqrt(q.shape[3])
                out[i, h, r:r + step] = torch.softmax(a, dim=-1) @ vv
    return out


def _pool(score, width):
    return torch.nn.functional.max_pool1d(score, width, stride=1, padding=width // 2)


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    group = c["q_heads"] // c["kv_heads"]
    if c["kind"] == "dense":
        return _attend(x["q"][0], x["k"], x["v"], group)
    if c["kind"] == "reuse":
        kc, vc = _cache(c, x)
        kb, vb = x["blk"][0]
        return _attend(x["q"][0], torch.cat([kc, kb], dim=2), torch.cat([vc, vb], dim=2), group)
    if c["kind"] == "full":
        return _attend(x["q"][0], x["k"], x["v"], group)
    if c["kind"] in ("update", "block"):
        # which of two nearly equal candidates is retained hangs on rounding, and with it the cache and what follows from it
        dense = [_attend(q, x["k"], x["v"], group) for q in x["q"][:2]]
        return {"out": dense + [None] * (c["steps"] - len(dense)), "idx": None, "k_cache": None, "v_cache": None}
    seq, off, _ = _sizes(c)
    keys = torch.cat([x["k"][:, :, :off], x["k"][:, :, off + c["block"]:]], dim=2)
    score = torch.empty(keys.shape[:3], dtype=torch.float64, device=keys.device)
    for i in range(c["batch"]):
        for h in range(c["kv_heads"]):
            q = x["q"][0][i, h * group:(h + 1) * group].double().flatten(0, 1)
            a = (q @ keys[i, h].double().T) / math.sqrt(c["head_dim"])
            score[i, h] = (torch.softmax(a, dim=-1) if c["score"] == "softmax_mean" else a).mean(dim=0)
    if c["select"] == "joint":
        pooled = _pool(score, c["pool"])
    else:
        sides = [p for p in (score[..., :off], score[..., off:]) if p.shape[-1]]
        pooled = torch.cat([_pool(p, c["pool"]) for p in sides], dim=-1)
    return {"idx": None, "pooled": pooled, "score": score}
