"""The work that users of this library have it do, as cases that can be timed and compared.

A case is a dict of plain values.  `prepare` makes what a program holds before the call (tensors on
the GPU, the layout handle, workspaces, output buffers), `run` is one pass through the public entry
points of paper_2506_19225_amd.vxl and returns everything those calls write, `work` is what the pass
cannot do without, `tolerance` how far another correct implementation may be off.

Kinds of work:
  prefill   chunk-based pre-filling attention of one layer, once per video and layer
  query     a question arrives at a layer: relevance scores and selection, gather of the mixed KV set,
            attention of the question's tokens over it
  select    the same selection alone (a stack of layers selects at one layer and reuses it)
  mass      the selection by softmax attention mass instead of mean logits
  answer    the mixed KV set of a selection that another layer made, and the question's tokens over it
  step      one generated token over a mixed KV set that is there
  token     one generated token through a stack of layers, replayed from a HIP graph
  inplace   no mixed buffers: sparse KVs pooled, the question's tokens and the first generated token
            read dense and sparse rows in place
  chain     all four steps on one small prompt (pre-filling, selection, gather, decode)

Prompts look like long videos: a text prefix, then chunks of some frames, a few rows of every chunk
kept.  Queries share a direction and every chunk's keys carry a random amount of it, so that chunks
differ in relevance as they do for a real question.
"""
import functools
import math
import types

import numpy as np
import torch

from paper_2506_19225_amd import vxl

ELEM = {"bf16": 2, "f32": 4}
DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
SMALL = 1.0 / math.sqrt(128.0)          # value scale of the workloads at 7B-class shapes

_DEFAULTS = dict(dtype="bf16", hq=28, hkv=4, d=128, prefix=256, unit=1, keep=8, kept_random=False, window=0,
                 token_major=False, lse=False, batch=1, t=1, k=0, layers=1, scale=SMALL)


def _case(name, kind, **kw):
    c = dict(_DEFAULTS, kind=kind, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest prompt of the parity workloads, fp32, everything once: launches and latency
        _case("chain_f32_tiny", "chain", dtype="f32", hq=2, hkv=1, d=64, prefix=64, chunks=4, len_lo=128, len_hi=128,
              t=8, k=2, scale=1.0),
        # a clip of a few groups of frames with ragged chunks (the smoke test's prompt): too little work to fill the chip
        _case("prefill_clip", "prefill", hq=14, hkv=2, prefix=64, chunks=4, len_lo=130, len_hi=320, unit=2, scale=1.0),
        # 256 frames of 64 tokens, chunks of 4 frames
        _case("prefill_16k", "prefill", chunks=64, len_lo=256, len_hi=256),
        # 1,024 frames, chunk lengths from 128 to 1,024 tokens, several kept ratios, the tensors as a projection
        # writes them, a dense look-back window and the log-sum-exp wanted
        _case("prefill_66k_ragged", "prefill", chunks=114, len_lo=128, len_hi=1024, unit=64, keep=0, window=256,
              token_major=True, lse=True, scale=1.0),
        # 2,048 frames, chunks of 8 frames, 64 kept rows each at random places: the largest single call
        _case("prefill_131k", "prefill", chunks=256, len_lo=512, len_hi=512, kept_random=True),
        # a question of 32 tokens on the 16k prompt
        _case("query_16k", "query", chunks=64, len_lo=256, len_hi=256, t=32, k=8),
        # selection over the longest prompt: 10,240 frames in 640 chunks, a question of 128 tokens
        _case("select_164k", "select", chunks=640, len_lo=256, len_hi=256, keep=16, t=128, k=32),
        # the other relevance score on the 131k prompt
        _case("mass_131k", "mass", chunks=256, len_lo=512, len_hi=512, t=64, k=16, scale=1.0),
        # eight independent questions on the ragged prompt
        _case("answer_66k_batch8", "answer", chunks=114, len_lo=128, len_hi=1024, unit=64, keep=0, batch=8, t=32, k=32,
              scale=1.0),
        # one generated token at one layer, called directly
        _case("step_16k", "step", chunks=64, len_lo=256, len_hi=256, k=8),
        # one generated token through the 28 layers of the longest prompt
        _case("token_164k_28_layers", "token", chunks=640, len_lo=256, len_hi=256, keep=16, k=32, layers=28),
        # the gather-free form on the 131k prompt with pooled sparse KVs
        _case("inplace_131k_pooled", "inplace", chunks=256, len_lo=512, len_hi=512, t=64, k=16, scale=1.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another prompt, question and head count of the ranges above."""
    most = work(next(c for c in listed() if c["name"] == "prefill_131k"))
    kind = rng.choice(["chain", "prefill", "prefill", "prefill", "query", "select", "mass", "answer", "step", "token",
                       "inplace"])
    while True:
        hq, hkv, d = rng.choice([(28, 4, 128)] * 4 + [(14, 2, 128), (14, 2, 64), (8, 1, 128), (4, 4, 64)])
        kw = dict(hq=hq, hkv=hkv, d=d, prefix=rng.choice([0, 17, 64, 256, 256, 300]), scale=rng.choice([SMALL, 1.0]),
                  kept_random=rng.random() < 0.5, keep=rng.choice([0, 4, 8, 16, 32]))
        tokens = _log(rng, 600, 164000)
        mean = min(tokens, _log(rng, 64, 1024))
        if kind == "chain":                                   # fp32 is for small prompts
            tokens, mean = _log(rng, 200, 2500), _log(rng, 30, 300)
            kw.update(dtype="f32", hq=hkv * 2, prefix=rng.choice([0, 17, 64]), scale=1.0)
        chunks = max(1, round(tokens / mean))
        if rng.random() < 0.5:
            kw.update(chunks=chunks, len_lo=mean, len_hi=mean)
        else:
            kw.update(chunks=chunks, len_lo=max(1, mean // 2), len_hi=mean + mean // 2, unit=rng.choice([1, 1, 16]))
        if kind == "prefill":
            kw.update(window=rng.choice([0, 0, 100, 256]), token_major=rng.random() < 0.4, lse=rng.random() < 0.4)
        else:
            kw.update(k=min(chunks, rng.choice([0, chunks] + [_log(rng, 1, 64)] * 4)))
        if kind in ("query", "select", "mass", "answer", "inplace"):
            kw.update(t=_log(rng, 1, 128), batch=rng.choice([1, 1, 1, 2, 3, 8]) if kind != "inplace" else 1)
        elif kind in ("step", "token"):
            kw.update(t=rng.choice([1, 1, 1, 2, 4]), batch=rng.choice([1, 1, 2, 8]) if kind == "step" else 1,
                      layers=_log(rng, 2, 28) if kind == "token" else 1)
        elif kind == "chain":
            kw.update(t=_log(rng, 1, 32))
        c = _case(None, kind, **kw)
        w = work(c)
        if chunks <= vxl.MAX_CHUNKS and w["flops"] <= most["flops"] and w["bytes"] <= most["bytes"]:
            return c


# ---- prompts -----------------------------------------------------------------------------------
@functools.lru_cache(maxsize=64)
def _shape(prefix, chunks, lo, hi, unit, keep):
    """Chunk bounds and kept counts of a prompt: a property of the case, not of the seed."""
    rng = np.random.default_rng([prefix, chunks, lo, hi, unit, keep])
    lens = np.full(chunks, lo, np.int64) if lo == hi else rng.integers(lo // unit, hi // unit + 1, size=chunks) * unit
    lens = np.maximum(lens, 1)
    ratio = np.full(chunks, keep, np.int64) if keep else rng.choice([4, 8, 32], size=chunks)
    counts = np.maximum(lens // ratio, 1)
    return (np.concatenate([[prefix], prefix + np.cumsum(lens)]).astype(np.int32),
            np.concatenate([[0], np.cumsum(counts)]).astype(np.int32))


def _shape_of(c):
    return _shape(c["prefix"], c["chunks"], c["len_lo"], c["len_hi"], c["unit"], c["keep"])


def _kept(c, bounds, soff, seed):
    """Token ids of the kept rows: strided from the chunk's start, or at random places."""
    lens, counts = np.diff(bounds), np.diff(soff)
    if not c["kept_random"]:
        m = np.arange(soff[-1]) - np.repeat(soff[:-1], counts)
        return (np.repeat(bounds[:-1], counts) + m * np.repeat(lens // counts, counts)).astype(np.int32)
    rng = np.random.default_rng([seed, 7])
    return np.concatenate([b + np.sort(rng.permutation(n)[:m]) for b, n, m in zip(bounds[:-1], lens, counts)]
                          ).astype(np.int32)


def _mixed_rows(c):
    """Mean mixed length of a selection of k chunks."""
    bounds, soff = _shape_of(c)
    k = min(c["k"], c["chunks"])
    return c["prefix"] + float(soff[-1]) + k * float(bounds[-1] - bounds[0] - soff[-1]) / c["chunks"]


# ---- inputs ------------------------------------------------------------------------------------
def _randn(gen, shape, dtype, scale):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, scale, generator=gen)


def prepare(case, seed):
    c = dict(_DEFAULTS, **case)
    bounds, soff = _shape_of(c)
    n, dt, s = int(bounds[-1]), DTYPE[c["dtype"]], types.SimpleNamespace(c=c)
    hq, hkv, d, b, t, k, kind = (c[x] for x in ("hq", "hkv", "d", "batch", "t", "k", "kind"))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s.desc = vxl.make_desc(hq, hkv, d, c["dtype"], token_major=c["token_major"])
    s.layout = vxl.Layout(c["prefix"], bounds, soff, _kept(c, bounds, soff, seed), window=c["window"])
    cap = s.l_cap = s.layout.mixed_kv_capacity(k)

    def workspace(op, **kw):
        return vxl.alloc_workspace(vxl.workspace_bytes(op, s.layout, s.desc, **kw))

    if kind in ("prefill", "chain"):
        shape = (n, hq, d) if c["token_major"] else (hq, n, d)
        s.q = _randn(gen, shape, dt, c["scale"])
        s.o = torch.empty_like(s.q)
        s.o_lse = torch.empty((hq, n), dtype=torch.float32, device="cuda") if c["lse"] else None
        s.ws_prefill = workspace(vxl.OP_PREFILL)
    if kind in ("step", "token"):
        # mixed sets of another selection: rows past the length are what a buffer holds that was once zeroed
        mask = _some_chunks(gen, b, c["chunks"], k).cpu().numpy()
        lens = c["prefix"] + (mask * np.diff(bounds) + (1 - mask) * np.diff(soff)).sum(axis=1)
        s.mix_len = torch.tensor(lens, dtype=torch.int32, device="cuda")
        s.qd = [_randn(gen, (b, t, hq, d), dt, c["scale"]) for _ in range(c["layers"])]
        s.kmix = [_randn(gen, (b, hkv, cap, d), dt, c["scale"]) for _ in range(c["layers"])]
        s.vmix = [_randn(gen, (b, hkv, cap, d), dt, c["scale"]) for _ in range(c["layers"])]
        s.od = [torch.empty_like(x) for x in s.qd]
        s.od_lse = [torch.empty((b, t, hq), dtype=torch.float32, device="cuda") for _ in range(c["layers"])]
        s.ws_decode = workspace(vxl.OP_DECODE, batch=b, n_q_tokens=t, l_cap=cap)
        if kind == "token":
            _layers(s)                                       # the stack once before it is recorded
            torch.cuda.synchronize()
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph):
                _layers(s)
        return s
    # dense K and V, with a share of every question's direction in the keys of each chunk
    shape = (n, hkv, d) if c["token_major"] else (hkv, n, d)
    s.k, s.v = _randn(gen, shape, dt, c["scale"]), _randn(gen, shape, dt, c["scale"])
    if kind == "prefill":
        return s
    u = _randn(gen, (b, hkv, d), torch.float32, 0.5)
    s.qd = ((_randn(gen, (b, t, hkv, hq // hkv, d), torch.float32, 1.0) + u[:, None, :, None]) * c["scale"]
            ).reshape(b, t, hq, d).to(dt)
    share = _randn(gen, (c["chunks"], b), torch.float32, 0.5 * c["scale"])
    per_token = torch.cat([torch.zeros((c["prefix"], b), device="cuda"), torch.repeat_interleave(
        share, torch.tensor(np.diff(bounds), dtype=torch.int64, device="cuda"), dim=0)])
    for g in range(hkv):
        s.k[g] += (per_token @ u[:, g]).to(dt)
    if kind in ("query", "select", "mass", "chain"):
        s.idx = torch.zeros((b, min(k, c["chunks"])), dtype=torch.int32, device="cuda")
        s.mask = torch.zeros((b, c["chunks"]), dtype=torch.uint8, device="cuda")
        s.scores = torch.zeros((b, c["chunks"]), dtype=torch.float32, device="cuda")
        # the mean keys of the chunks are kept for the next question
        s.kbar = torch.zeros((hkv, c["chunks"], d), dtype=torch.float32, device="cuda")
        s.ws_score = (workspace(vxl.OP_SCORE_MASS, batch=b, n_q_tokens=t) if kind == "mass" else
                      workspace(vxl.OP_SCORE_TOPK, batch=b))
    else:
        s.mask = _some_chunks(gen, b, c["chunks"], k)
    if kind in ("query", "answer", "chain"):
        s.kmix = torch.zeros((b, hkv, cap, d), dtype=dt, device="cuda")
        s.vmix = torch.zeros_like(s.kmix)
        s.ws_decode = workspace(vxl.OP_DECODE, batch=b, n_q_tokens=t, l_cap=cap)
    s.mix_len = torch.zeros((b,), dtype=torch.int32, device="cuda")
    s.od = torch.empty_like(s.qd)
    s.od_lse = torch.empty((b, t, hq), dtype=torch.float32, device="cuda")
    if kind == "inplace":
        s.ksp = torch.empty((hkv, int(soff[-1]), d), dtype=dt, device="cuda")
        s.vsp = torch.empty_like(s.ksp)
        s.qd1 = s.qd[:, -1:].contiguous()
        s.od1, s.od1_lse = torch.empty_like(s.qd1), torch.empty((b, 1, hq), dtype=torch.float32, device="cuda")
        s.ws_decode = vxl.alloc_workspace(max(vxl.workspace_bytes(vxl.OP_DECODE_INPLACE, s.layout, s.desc, b, x, cap)
                                              for x in (1, t)))
    return s


def _some_chunks(gen, b, chunks, k):
    """Masks with k chunks each, chosen at random."""
    order = torch.argsort(torch.rand((b, chunks), device="cuda", generator=gen), dim=1)
    return torch.zeros((b, chunks), dtype=torch.uint8, device="cuda").scatter_(1, order[:, :k], 1)


# ---- one pass ----------------------------------------------------------------------------------
def _layers(s):
    for qd, kmix, vmix, od, lse in zip(s.qd, s.kmix, s.vmix, s.od, s.od_lse):
        vxl.bilevel_decode(s.desc, qd, kmix, vmix, s.mix_len, od, lse, s.ws_decode)


def run(s):
    kind, k = s.c["kind"], s.c["k"]
    if kind == "step":
        _layers(s)
        return s.od + s.od_lse
    if kind == "token":
        s.graph.replay()
        return s.od + s.od_lse
    out = []
    if kind in ("prefill", "chain"):
        vxl.chunk_prefill(s.layout, s.desc, s.q, s.k, s.v, s.o, s.o_lse, s.ws_prefill)
        out += [s.o, s.o_lse]
    if kind in ("query", "select", "chain"):
        vxl.chunk_score_topk(s.layout, s.desc, s.qd, s.k, k, s.idx, s.mask, s.scores, s.kbar, workspace=s.ws_score)
        out += [s.idx, s.mask, s.scores, s.kbar]
    if kind == "mass":
        vxl.chunk_score_topk_mass(s.layout, s.desc, s.qd, s.k, k, s.idx, s.mask, s.scores, workspace=s.ws_score)
        out += [s.idx, s.mask, s.scores]
    if kind in ("query", "answer", "chain"):
        vxl.gather_bilevel_kv(s.layout, s.desc, s.k, s.v, s.mask, s.kmix, s.vmix, s.mix_len)
        vxl.bilevel_decode(s.desc, s.qd, s.kmix, s.vmix, s.mix_len, s.od, s.od_lse, s.ws_decode)
        out += [s.kmix, s.vmix, s.mix_len, s.od, s.od_lse]
    if kind == "inplace":
        vxl.pool_sparse_kv(s.layout, s.desc, s.k, s.v, s.ksp, s.vsp)
        vxl.bilevel_decode_inplace(s.layout, s.desc, s.qd, s.k, s.v, s.ksp, s.vsp, s.mask, s.l_cap, s.od, s.od_lse,
                                   s.mix_len, s.ws_decode)
        vxl.bilevel_decode_inplace(s.layout, s.desc, s.qd1, s.k, s.v, s.ksp, s.vsp, s.mask, s.l_cap, s.od1, s.od1_lse,
                                   s.mix_len, s.ws_decode, map_ready=True)
        out += [s.ksp, s.vsp, s.mix_len, s.od, s.od_lse, s.od1, s.od1_lse]
    return [x for x in out if x is not None]


# ---- what a pass cannot do without ---------------------------------------------------------------
def work(case):
    c = dict(_DEFAULTS, **case)
    bounds, soff = _shape_of(c)
    n, e, kind = int(bounds[-1]), ELEM[c["dtype"]], c["kind"]
    hq, hkv, d, b, t = (c[x] for x in ("hq", "hkv", "d", "batch", "t"))
    kv = hkv * n * d * e                                     # dense K, or V
    mixed = b * hkv * _mixed_rows(c) * d * e                 # the K, or V, rows of the mixed sets
    qd, ints = b * t * hq * d * e, b * c["chunks"] * 5
    dec = 4.0 * d * hq * t * b * _mixed_rows(c)
    by, fl = 0.0, 0.0
    if kind in ("prefill", "chain"):
        by += 2 * hq * n * d * e + 2 * kv + (4 * hq * n if c["lse"] else 0)
        fl += 4.0 * d * hq * _pairs(c, bounds, soff)
    if kind in ("query", "select", "chain"):
        by += (kv if kind != "chain" else 0) + qd + ints + 4 * hkv * c["chunks"] * d
        fl += hkv * n * d + 2.0 * b * hkv * c["chunks"] * d
    if kind == "mass":
        by += kv + qd + ints
        fl += 2.0 * d * hq * t * b * n
    if kind == "query":
        by += 3 * mixed + qd                                 # V rows in, both mixed sets and O out
    if kind == "answer":
        by += 4 * mixed + 2 * qd                             # K and V rows in, both mixed sets and O out
    if kind == "chain":
        by += 2 * mixed + qd
    if kind in ("step", "token"):
        by += c["layers"] * (2 * mixed + 2 * qd)
    if kind == "inplace":
        by += 2 * kv + 2 * hkv * int(soff[-1]) * d * e + 2 * qd + 2 * hq * d * e
        dec *= (t + 1.0) / t
    if kind not in ("prefill", "select", "mass"):
        fl += c["layers"] * dec
    return {"bytes": float(by), "flops": float(fl)}


def _pairs(c, bounds, soff):
    """(query, key) pairs of the pre-filling mask: prefix and kept rows of earlier chunks, the look-back window
    (kept rows inside it once; their share is that of evenly spread rows), the causal half of the chunk itself."""
    lens, p = np.diff(bounds).astype(np.float64), float(c["prefix"])
    back = np.minimum(float(c["window"]), bounds[:-1] - p)
    lo = bounds[:-1] - back
    kept = np.interp(lo, bounds.astype(np.float64), soff.astype(np.float64))
    return p * (p + 1) / 2 + float((lens * (p + kept + back) + lens * (lens + 1) / 2).sum())


# ---- how far another correct implementation may be off --------------------------------------------
def tolerance(case):
    """Against float64 the cases show: fp32 storage, and the fp32 sums of the selection scores, relative errors up to
    6e-7 (values up to 2.5e-6); bf16 storage, whose probabilities and outputs are rounded to bf16 once (2^-9 each), up to
    2.3e-3 (values up to 1.6e-2).  About four times that.  Selections, lengths and gathered rows are exact: chunks differ
    in relevance by far more than the rounding of their scores."""
    if case["kind"] in ("select", "mass"):
        return {"rel": 2e-6, "max": 1e-5, "differ": 0.0}
    if case["dtype"] == "f32":
        return {"rel": 2.5e-6, "max": 1e-5, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.06, "differ": 0.0}
