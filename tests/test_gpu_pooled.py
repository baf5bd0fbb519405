"""GPU parity of the pooled sparse KVs (vxl_pool_sparse_kv, vxl_gather_bilevel_kv_pooled) and of
decoding over the mixed set built from them, against the float64 oracle.  Pooled values are
floating point: they are compared to within one unit in the last place of the storage dtype
(the device adds in fp32, the oracle in float64, both round once); everything that is a copy or
an index is compared bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import assert_close, desc_of, gpu_decode, gpu_gather, kept_rows, make_layout, storage_round

pytestmark = pytest.mark.gpu


def run_pool(w, lay, k, v, gl=None):
    gl = gl or make_layout(lay)
    desc = desc_of(w)
    dk, dv = vxl.to_device(k, w.dtype), vxl.to_device(v, w.dtype)
    s_total = int(lay.sparse_offsets[-1])
    ksp = torch.full((w.n_kv_heads, max(s_total, 1), w.head_dim), 7.0, dtype=dk.dtype, device="cuda")
    vsp = torch.full_like(ksp, 7.0)
    vxl.pool_sparse_kv(gl, desc, dk, dv, ksp, vsp)
    torch.cuda.synchronize()
    return gl, dk, dv, ksp, vsp


def check_pool(w, lay, k, v):
    gl, dk, dv, ksp, vsp = run_pool(w, lay, k, v)
    s_total = int(lay.sparse_offsets[-1])
    wk, wv = oracle.pool_sparse_kv(k, v, lay.chunk_bounds, lay.sparse_offsets)
    # one unit in the last place of the result (its single rounding) plus the fp32 summation error,
    # which scales with the summands, not with the (possibly cancelling) mean
    ulp = 2.0 ** -7 if w.dtype == "bf16" else 2.0 ** -22
    for got, want, src in ((vxl.to_host(ksp)[:, :s_total], wk, k), (vxl.to_host(vsp)[:, :s_total], wv, v)):
        ref = storage_round(w, want).astype(np.float64)
        assert np.isfinite(got).all()
        tol = ulp * np.abs(ref) + 2.0 ** -21 * np.abs(src).max()
        assert (np.abs(got - ref) <= tol).all(), np.abs(got - ref).max()
        if w.dtype == "bf16":
            assert (got == ref).mean() > 0.99                # the two roundings almost always agree
    return gl, dk, dv, ksp, vsp


def test_pool_config0_fp32_and_ragged_groups():
    w = wl.WORKLOADS["config0"]
    lay = wl.make_layout(w)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    check_pool(w, lay, k, v)
    rng = np.random.default_rng(91)
    for dtype, d in (("f32", 128), ("bf16", 64), ("bf16", 128)):
        w = wl.tiny_workload(dtype, 4, 2, d, T=2, B=2, k=2, seed=91)
        # odd chunk lengths and kept counts: groups of unequal size, one row per group, one group
        lay = wl.random_layout(rng, 3, 11, 1, 157, allow_empty_kept=True)
        _, k, v = wl.make_qkv(w, lay, with_q=False)
        check_pool(w, lay, k, v)


@pytest.mark.parametrize("dtype,d", [("f32", 128), ("bf16", 128), ("bf16", 64)])
@pytest.mark.parametrize("chunks", [1, 16, 17, 257, 300])
def test_pool_finds_chunks(dtype, d, chunks):
    """Chunk counts around the powers of the probes per row (8, 16 or 32), empty kept sets in runs and
    at both ends, group lengths around the four rows requested together."""
    rng = np.random.default_rng(chunks)
    w = wl.tiny_workload(dtype, 4, 2, d, T=1, B=1, k=1, seed=chunks)
    lay = wl.random_layout(rng, 5, chunks, 1, 19, allow_empty_kept=True)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    check_pool(w, lay, k, v)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
def test_pool_group_lengths(dtype, d):
    """Groups of 1 to 13 rows, which end in every remainder of the four rows requested together, side by side."""
    w = wl.tiny_workload(dtype, 2, 2, d, T=1, B=1, k=1, seed=96)
    lens = list(range(1, 14)) + [26, 7, 3]
    kept, start = [], 3
    for i, n in enumerate(lens):
        kept.append(np.arange(start, start + (1 if i < 13 else 2), dtype=np.int32))
        start += n
    lay = wl.layout_from_lists(3, lens, kept)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    check_pool(w, lay, k, v)


@pytest.mark.parametrize("name", ["config0", "config1", "config4"])
def test_pooled_chain(name):
    """select -> pool -> gather (pooled) -> decode, everything on the device; the gathered set is
    checked row by row against its sources, the decode output against the oracle's decode over
    the oracle's own pooled set."""
    w = wl.WORKLOADS[name]
    lay = wl.make_layout(w)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    gl, dk, dv, ksp, vsp = check_pool(w, lay, k, v)
    desc = desc_of(w)
    top_k = w.k
    scores = oracle.chunk_scores(qd, k, lay.chunk_bounds)
    _, masks = oracle.select_topk(scores, top_k)
    dm = torch.from_numpy(masks).cuda()
    l_cap = gl.mixed_kv_capacity(top_k)
    bsz = qd.shape[0]
    kmix = torch.full((bsz, w.n_kv_heads, l_cap, w.head_dim), 7.0, dtype=dk.dtype, device="cuda")
    vmix = torch.full_like(kmix, 7.0)
    mix_len = torch.full((bsz,), -1, dtype=torch.int32, device="cuda")
    src = torch.full((bsz, l_cap), -5, dtype=torch.int32, device="cuda")
    vxl.gather_bilevel_kv_pooled(gl, desc, dk, dv, ksp, vsp, dm, kmix, vmix, mix_len, src)
    torch.cuda.synchronize()
    # oracle structure (lengths, source codes) -- pooled values taken from the oracle's own pooling
    ok, ov = oracle.pool_sparse_kv(k, v, lay.chunk_bounds, lay.sparse_offsets)
    ok, ov = storage_round(w, ok), storage_round(w, ov)
    wk, wv, wlen, wsrc = oracle.gather_bilevel_pooled(k, v, ok, ov, masks, lay.n_prefix, lay.chunk_bounds,
                                                      lay.sparse_offsets, l_cap=l_cap)
    assert np.array_equal(mix_len.cpu().numpy(), wlen)
    hsrc = src.cpu().numpy()
    hk, hv = vxl.to_host(kmix), vxl.to_host(vmix)
    dsp_k, dsp_v = vxl.to_host(ksp), vxl.to_host(vsp)
    for b in range(bsz):
        n = int(wlen[b])
        assert np.array_equal(hsrc[b, :n], wsrc[b, :n])
        assert (hsrc[b, n:] == -5).all() and (hk[b, :, n:] == 7.0).all()          # rows beyond untouched
        s = hsrc[b, :n]
        dense = s >= 0
        assert np.array_equal(hk[b][:, :n][:, dense], k[:, s[dense]])             # copies: bit for bit
        assert np.array_equal(hv[b][:, :n][:, dense], v[:, s[dense]])
        assert np.array_equal(hk[b][:, :n][:, ~dense], dsp_k[:, -1 - s[~dense]])
        assert np.array_equal(hv[b][:, :n][:, ~dense], dsp_v[:, -1 - s[~dense]])
    got = gpu_decode(w, qd, kmix, vmix, mix_len)
    want = oracle.decode_mixed(qd, wk, wv, wlen)
    assert_close(got, want, w.dtype, head_axis=2, what=f"{name} decode over pooled mixed KV")


@pytest.mark.parametrize("n_kv_heads", [1, 3, 4, 5, 8, 11])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("bf16", 128)])
def test_gather_head_counts(dtype, d, n_kv_heads):
    """KV heads around the four whose pieces the gather requests together: every copied row bit for
    bit, the rows behind the mixed length untouched."""
    w = wl.tiny_workload(dtype, n_kv_heads, n_kv_heads, d, T=1, B=2, k=2, seed=93)
    lay = wl.random_layout(np.random.default_rng(93), 5, 7, 1, 61)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    gl, desc = make_layout(lay), desc_of(w)
    dk, dv = vxl.to_device(k, w.dtype), vxl.to_device(v, w.dtype)
    masks = np.array([[1, 0, 0, 1, 0, 0, 0], [0, 0, 1, 0, 0, 0, 1]], np.uint8)
    l_cap = gl.mixed_kv_capacity(2)
    kmix = torch.full((2, n_kv_heads, l_cap, d), 7.0, dtype=dk.dtype, device="cuda")
    vmix = torch.full_like(kmix, 7.0)
    mix_len = torch.zeros((2,), dtype=torch.int32, device="cuda")
    vxl.gather_bilevel_kv(gl, desc, dk, dv, torch.from_numpy(masks).cuda(), kmix, vmix, mix_len)
    torch.cuda.synchronize()
    hk, hv = vxl.to_host(kmix), vxl.to_host(vmix)
    for b in range(2):
        src = oracle.mixed_source_index(masks[b], lay.n_prefix, lay.chunk_bounds, lay.sparse_offsets, lay.sparse_idx)
        n = len(src)
        assert int(mix_len[b]) == n
        assert np.array_equal(hk[b, :, :n], k[:, src]) and np.array_equal(hv[b, :, :n], v[:, src])
        assert (hk[b, :, n:] == 7.0).all() and (hv[b, :, n:] == 7.0).all()


@pytest.mark.parametrize("pooled", [False, True])
@pytest.mark.parametrize("dtype,d", [("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_gather_four_heads_as_two_and_two(dtype, d, pooled):
    """Four KV heads take the instance that moves all heads of a row together, two heads the one that moves them one
    after the other: the same rows, lengths and untouched bytes behind them, bit for bit, also into buffers (by
    capacity; the sets are small) beyond the on-package cache."""
    w = wl.tiny_workload(dtype, 4, 4, d, T=1, B=3, k=2, seed=94)
    lay = wl.random_layout(np.random.default_rng(94), 5, 300, 1, 61)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    gl, desc = make_layout(lay), desc_of(w)
    dk, dv = vxl.to_device(k, w.dtype), vxl.to_device(v, w.dtype)
    masks = np.random.default_rng(95).random((3, 300)) < np.array([[0.3], [0.0], [1.0]])
    dm = torch.from_numpy(masks.astype(np.uint8)).cuda()
    need = lay.n_tokens
    sparse = ()
    if pooled:
        sparse = tuple(torch.empty((4, int(lay.sparse_offsets[-1]), d), dtype=dk.dtype, device="cuda") for _ in range(2))
        vxl.pool_sparse_kv(gl, desc, dk, dv, *sparse)
    call = vxl.gather_bilevel_kv_pooled if pooled else vxl.gather_bilevel_kv
    got = []
    for heads, l_cap in ((slice(0, 4), need), (slice(0, 4), max(need, (256 << 20) // (8 * 3 * d * dk.element_size()) + 1)),
                         (slice(0, 2), need), (slice(2, 4), need)):
        hkv = heads.stop - heads.start
        kmix = torch.full((3, hkv, l_cap, d), 7.0, dtype=dk.dtype, device="cuda")
        vmix = torch.full_like(kmix, 7.0)
        mix_len = torch.zeros((3,), dtype=torch.int32, device="cuda")
        call(gl, vxl.make_desc(hkv, hkv, d, dtype), dk[heads], dv[heads], *(x[heads] for x in sparse), dm, kmix, vmix, mix_len)
        torch.cuda.synchronize()
        assert (kmix[:, :, need:] == 7.0).all() and (vmix[:, :, need:] == 7.0).all()
        got.append((mix_len, kmix[:, :, :need].clone(), vmix[:, :, :need].clone()))
    (n2, k2, v2), (n3, k3, v3) = got[2:]
    assert torch.equal(n2, n3)
    got[2:] = [(n2, torch.cat([k2, k3], 1), torch.cat([v2, v3], 1))]
    assert got[0][0].tolist() == [5 + sum(int(b - a) if m else int(t - s) for m, a, b, s, t in zip(
        masks[q], lay.chunk_bounds, lay.chunk_bounds[1:], lay.sparse_offsets, lay.sparse_offsets[1:])) for q in range(3)]
    assert all(torch.equal(x, y) for other in got[1:] for x, y in zip(got[0], other))


@pytest.mark.parametrize("dtype,d,n_kv_heads", [("f32", 64, 3), ("bf16", 64, 2), ("bf16", 128, 3), ("bf16", 128, 4)])
def test_gather_beyond_the_on_package_cache(dtype, d, n_kv_heads):
    """Mixed buffers from 160 MB on, whose queries take turns: head counts that go one after the other and four, chunks of
    more than one scan round with empty ones among them, and a query that does not fit; every row bit for bit."""
    row, n_q = n_kv_heads * d * (4 if dtype == "f32" else 2), 13
    l_cap = (160 << 20) // (2 * n_q * row) + 1
    lens = np.random.default_rng(97).integers(1, 2 * l_cap // 1100 + 3, size=1100)
    lens[0] += max(0, l_cap + 1 - 5 - int(lens.sum()))                       # all chunks dense: does not fit
    starts = 5 + np.concatenate([[0], np.cumsum(lens)[:-1]])
    kept = [s + 1 + np.arange(n // 5, dtype=np.int32) for s, n in zip(starts, lens)]
    w = wl.tiny_workload(dtype, n_kv_heads, n_kv_heads, d, T=1, B=n_q, k=2, seed=96)
    lay = wl.layout_from_lists(5, lens.tolist(), kept)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    masks = (np.random.default_rng(98).random((n_q, 1100)) < np.linspace(0.0, 0.3, n_q)[:, None]).astype(np.uint8)
    masks[7] = 1
    kmix = torch.full((n_q, n_kv_heads, l_cap, d), 7.0, dtype=vxl.to_device(k[:, :1], dtype).dtype, device="cuda")
    vmix = torch.full_like(kmix, 7.0)
    mix_len = torch.zeros((n_q,), dtype=torch.int32, device="cuda")
    vxl.gather_bilevel_kv(make_layout(lay), desc_of(w), vxl.to_device(k, dtype), vxl.to_device(v, dtype),
                          torch.from_numpy(masks).cuda(), kmix, vmix, mix_len)
    torch.cuda.synchronize()
    for b in range(n_q):
        src = oracle.mixed_source_index(masks[b], lay.n_prefix, lay.chunk_bounds, lay.sparse_offsets, lay.sparse_idx)
        n = len(src) if len(src) <= l_cap else 0
        assert int(mix_len[b]) == (n if n else -len(src)) and (n > 0) == (b != 7)
        hk, hv = vxl.to_host(kmix[b]), vxl.to_host(vmix[b])
        assert np.array_equal(hk[:, :n], k[:, src[:n]]) and np.array_equal(hv[:, :n], v[:, src[:n]])
        assert (hk[:, n:] == 7.0).all() and (hv[:, n:] == 7.0).all()


def test_pooled_gather_without_sparse_rows_and_all_dense():
    w = wl.tiny_workload("bf16", 4, 2, 128, T=1, B=1, k=1, seed=92)
    lay = wl.layout_from_lists(4, [40, 24], [np.zeros(0, np.int32)] * 2)           # nothing kept: S_total = 0
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    gl = make_layout(lay)
    desc = desc_of(w)
    dk, dv = vxl.to_device(k, w.dtype), vxl.to_device(v, w.dtype)
    vxl.pool_sparse_kv(gl, desc, dk, dv, None, None)                               # nothing to write
    dm = torch.tensor([[1, 0]], dtype=torch.uint8, device="cuda")
    l_cap = gl.mixed_kv_capacity(1)
    kmix = torch.zeros((1, 2, l_cap, 128), dtype=dk.dtype, device="cuda")
    vmix = torch.zeros_like(kmix)
    mix_len = torch.zeros((1,), dtype=torch.int32, device="cuda")
    vxl.gather_bilevel_kv_pooled(gl, desc, dk, dv, None, None, dm, kmix, vmix, mix_len, None)
    torch.cuda.synchronize()
    assert int(mix_len[0]) == 44
    assert np.array_equal(vxl.to_host(kmix)[0, :, :44], k[:, :44])


@pytest.mark.parametrize("dtype,d,n_kv_heads", [("f32", 64, 1), ("bf16", 64, 2), ("bf16", 128, 3), ("bf16", 128, 4)])
def test_gather_past_the_caches_goes_by_rows(dtype, d, n_kv_heads):
    """Buffers from 160 MB on: a query that fills its own goes past the caches, one of few rows beside it does not."""
    row, n_q = n_kv_heads * d * (4 if dtype == "f32" else 2), 6
    l_cap = (160 << 20) // (2 * n_q * row) + 40
    lens = np.full(40, (l_cap - 39) // 40)
    lens[-1] += l_cap - 7 - int(lens.sum())
    kept = [s + np.arange(3, dtype=np.int32) for s in 7 + np.concatenate([[0], np.cumsum(lens)[:-1]])]
    w = wl.tiny_workload(dtype, n_kv_heads, n_kv_heads, d, T=1, B=n_q, k=2, seed=97)
    lay = wl.layout_from_lists(7, lens.tolist(), kept)
    rng = np.random.default_rng(97)
    shape = (n_kv_heads, lay.n_tokens, d)
    k, v = (wl.round_to_bf16(rng.random(shape, dtype=np.float32)) for _ in range(2))
    masks = np.ones((n_q, 40), np.uint8)
    masks[1::2] = rng.random((n_q // 2, 40)) < 0.3
    kmix, vmix, mix_len, _ = gpu_gather(w, lay, k, v, masks, l_cap)
    for b in range(n_q):
        src = oracle.mixed_source_index(masks[b], lay.n_prefix, lay.chunk_bounds, lay.sparse_offsets, lay.sparse_idx)
        n = len(src)
        assert int(mix_len[b]) == n and (2 * n_q * n * row > 160 << 20) == (b % 2 == 0)
        hk, hv = vxl.to_host(kmix[b]), vxl.to_host(vmix[b])
        assert np.array_equal(hk[:, :n], k[:, src]) and np.array_equal(hv[:, :n], v[:, src])
        assert (hk[:, n:] == 7.0).all() and (hv[:, n:] == 7.0).all()


@pytest.mark.parametrize("pooled", [False, True])
@pytest.mark.parametrize("n_kv_heads,d", [(1, 128), (3, 64), (4, 64)])
@pytest.mark.parametrize("n_chunks", [2499, 2500, 2501, 4096])
def test_gather_on_both_sides_of_the_chunk_table(n_chunks, n_kv_heads, d, pooled):
    """Where the source of a chunk's rows is kept beside the offsets, and where it is asked for (other head counts than
    four, more than 2,500 chunks): rows, lengths and the row map bit for bit, chunks without kept rows among them."""
    rng = np.random.default_rng(n_chunks + d)
    w = wl.tiny_workload("bf16", n_kv_heads, n_kv_heads, d, T=1, B=3, k=2, seed=98)
    lens = rng.integers(1, 5, size=n_chunks)
    starts = 11 + np.concatenate([[0], np.cumsum(lens)[:-1]])
    lay = wl.layout_from_lists(11, lens.tolist(), [s + np.arange(n // 2, dtype=np.int32) for s, n in zip(starts, lens)])
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    masks = (rng.random((3, n_chunks)) < np.array([0.0, 0.4, 1.0])[:, None]).astype(np.uint8)
    l_cap = lay.n_tokens
    if not pooled:
        kmix, vmix, mix_len, src_idx = gpu_gather(w, lay, k, v, masks, l_cap)
        ksp, vsp = (kept_rows(x, lay) for x in (k, v))
    else:
        dev = [vxl.to_device(x, "bf16") for x in (k, v)]
        gl, desc = make_layout(lay), desc_of(w)
        ksp, vsp = (wl.round_to_bf16(rng.standard_normal((n_kv_heads, len(lay.sparse_idx), d)).astype(np.float32)) for _ in range(2))
        kmix = torch.full((3, n_kv_heads, l_cap, d), 7.0, dtype=torch.bfloat16, device="cuda")
        vmix, mix_len = torch.full_like(kmix, 7.0), torch.zeros((3,), dtype=torch.int32, device="cuda")
        src_idx = torch.full((3, l_cap), -5, dtype=torch.int32, device="cuda")
        vxl.gather_bilevel_kv_pooled(gl, desc, *dev, vxl.to_device(ksp, "bf16"), vxl.to_device(vsp, "bf16"),
                                     torch.from_numpy(masks).cuda(), kmix, vmix, mix_len, src_idx)
    for b in range(3):
        src, sparse = [np.arange(11)], [np.full(11, -1)]            # token of every row; its kept row, or -1
        for c in range(n_chunks):
            lo, hi = lay.sparse_offsets[c], lay.sparse_offsets[c + 1]
            src.append(np.arange(lay.chunk_bounds[c], lay.chunk_bounds[c + 1]) if masks[b, c] else lay.sparse_idx[lo:hi])
            sparse.append(np.full(lens[c], -1) if masks[b, c] else np.arange(lo, hi))
        src, sparse = np.concatenate(src), np.concatenate(sparse)
        n = len(src)
        assert int(mix_len[b]) == n
        assert np.array_equal(src_idx[b, :n].cpu().numpy(), np.where(sparse >= 0, -1 - sparse, src) if pooled else src)
        for got, x, xs in ((kmix, k, ksp), (vmix, v, vsp)):
            want = np.where((sparse >= 0)[None, :, None], xs[:, np.maximum(sparse, 0)], x[:, src]) if pooled else x[:, src]
            assert np.array_equal(vxl.to_host(got[b])[:, :n], want) and (vxl.to_host(got[b])[:, n:] == 7.0).all()


def gather_together_and_apart(w, lay, masks, l_cap, pooled, shared):
    """The gather of all queries and that of each alone, head-major and token-major: the same rows, lengths, sources and
    untouched bytes, bit for bit; `shared` of the first kind by the kernel that reads a row once.  Returns the rows needed."""
    n_q, n_kv_heads, d, dtype = len(masks), w.n_kv_heads, w.head_dim, w.dtype
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    gl, n_sparse = make_layout(lay), int(lay.sparse_offsets[-1])
    need = [lay.n_prefix + sum(int(b - a) if m else int(t - s) for m, a, b, s, t in zip(
        mask, lay.chunk_bounds, lay.chunk_bounds[1:], lay.sparse_offsets, lay.sparse_offsets[1:])) for mask in masks]
    dm = torch.from_numpy(masks).cuda()
    for token_major in (False, True):
        dk, dv = vxl.to_device(k, dtype), vxl.to_device(v, dtype)
        desc = desc_of(w)
        if token_major:
            dk, dv = (x.transpose(0, 1).contiguous() for x in (dk, dv))
            desc = vxl.make_desc(n_kv_heads, n_kv_heads, d, dtype, token_major=True)
        sparse = ()
        if pooled:
            sparse = tuple(torch.empty((n_kv_heads, n_sparse, d), dtype=dk.dtype, device="cuda") for _ in range(2))
            vxl.pool_sparse_kv(gl, desc, dk, dv, *sparse)
        call = vxl.gather_bilevel_kv_pooled if pooled else vxl.gather_bilevel_kv

        def run(lo, hi):
            n = hi - lo
            kmix = torch.full((n, n_kv_heads, l_cap, d), 7.0, dtype=dk.dtype, device="cuda")
            vmix = torch.full_like(kmix, 7.0)
            mix_len = torch.full((n,), -9, dtype=torch.int32, device="cuda")
            src = torch.full((n, l_cap), -5_000_000, dtype=torch.int32, device="cuda")
            assert vxl.debug_gather_shared(desc, lay.n_tokens, n_sparse, lay.n_chunks, n, l_cap) == (shared and n > 1)
            call(gl, desc, dk, dv, *sparse, dm[lo:hi].contiguous(), kmix, vmix, mix_len, src)
            torch.cuda.synchronize()
            return kmix, vmix, mix_len, src

        together = run(0, n_q)
        assert together[2].tolist() == [x if x <= l_cap else -x for x in need]
        for b in range(n_q):
            assert all(torch.equal(x[b], y[0]) for x, y in zip(together, run(b, b + 1))), b
    return need


def capacity_of_large_sets(w, lay, n_q):
    """45 MB together, two rows per token, 128 blocks of 4,096 bytes per set."""
    row = w.head_dim * (4 if w.dtype == "f32" else 2)
    return max(45_000_000 // (2 * n_q * w.n_kv_heads * row) + 1, 2 * lay.n_tokens // n_q + 1, 128 * 4096 // row,
               make_layout(lay).mixed_kv_capacity(0))


@pytest.mark.parametrize("pooled", [False, True])
@pytest.mark.parametrize("dtype,n_kv_heads,d,n_q,prefix,chunks,longest", [
    ("bf16", 4, 128, 8, 5, 100, 61), ("bf16", 2, 128, 2, 0, 65, 61), ("bf16", 3, 64, 16, 17, 64, 61), ("bf16", 4, 64, 3, 5, 64, 61),
    ("f32", 1, 64, 16, 5, 1, 61), ("f32", 4, 128, 5, 33, 200, 61), ("f32", 2, 64, 16, 0, 31, 190), ("bf16", 1, 128, 15, 5, 33, 61),
    ("bf16", 8, 128, 3, 5, 70, 61), ("bf16", 16, 64, 4, 0, 40, 61), ("bf16", 6, 128, 9, 9, 20, 61), ("f32", 12, 64, 2, 1, 512, 9),
    ("bf16", 16, 128, 32, 17, 32, 200), ("bf16", 4, 64, 17, 5, 33, 61)])
def test_gather_for_many_queries_is_the_gather_for_each(dtype, n_kv_heads, d, n_q, prefix, chunks, longest, pooled):
    """Large sets of up to 16 queries, or 32 of many rows, are copied by the kernel that reads a row once for all of them, one
    query by the general one.  Queries that have every chunk dense, none, or do not fit; chunks without kept rows; counts around the 64 of a
    scan, the 32 queries and the 1,024 masks; KV heads in groups of four, two and one; token counts that are no multiple of a
    block's rows."""
    rng = np.random.default_rng(chunks + n_q)
    w = wl.tiny_workload(dtype, n_kv_heads, n_kv_heads, d, T=1, B=n_q, k=2, seed=chunks)
    lay = wl.random_layout(rng, prefix, chunks, 1, longest)
    masks = (rng.random((n_q, chunks)) < np.linspace(0.0, 1.0, n_q)[:, None]).astype(np.uint8)
    l_cap = capacity_of_large_sets(w, lay, n_q)
    need = gather_together_and_apart(w, lay, masks, l_cap, pooled, n_q <= 16 or longest == 200)
    assert longest != 190 or max(need) > l_cap                # one shape at least has a query that does not fit


@pytest.mark.parametrize("pooled", [False, True])
@pytest.mark.parametrize("n_kv_heads,d,n_q,prefix,dense", [
    (4, 128, 3, 0, []), (8, 64, 2, 40, []), (1, 128, 5, 0, [(4, 39)]), (8, 128, 4, 3, [(0, 0), (3, 20)])])
def test_gather_of_nearly_empty_sets(n_kv_heads, d, n_q, prefix, dense, pooled):
    """Most blocks have no row that anybody takes, the first one too, which writes the lengths all the same."""
    w = wl.tiny_workload("bf16", n_kv_heads, n_kv_heads, d, T=1, B=n_q, k=2, seed=d)
    lay = wl.random_layout(np.random.default_rng(d), prefix, 40, 20, 90)
    masks = np.zeros((n_q, 40), np.uint8)
    for at in dense:
        masks[at] = 1
    l_cap = 3 * capacity_of_large_sets(w, lay, n_q)
    assert max(gather_together_and_apart(w, lay, masks, l_cap, pooled, True)) < l_cap / 5
