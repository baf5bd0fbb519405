"""The fp32 matrix-instruction kernels at the sizes where a row block (16 stacked rows), a key tile (32) or the
slices of the waves that share a block's keys are partly filled or empty, and on both sides of the line between
one workgroup per row block and key splits in the decode.  Tolerance: the path's 1e-5 for fp32 storage."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import assert_close, desc_of, gpu_decode, gpu_decode_inplace, gpu_prefill, kept_rows, make_layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,prefix,lens,window", [
    (1, 1, 64, 0, [1, 2, 15, 16, 17], 0), (7, 1, 128, 1, [31, 32, 33, 5], 0), (6, 2, 64, 33, [127, 128, 129, 300], 40),
    (8, 1, 128, 130, [640, 700, 641], 0), (28, 4, 64, 64, [257, 1, 511], 100),
    (32, 1, 64, 0, [127, 1], 0), (32, 1, 64, 0, [128, 1], 0), (32, 1, 128, 5, [15, 17, 64, 3, 40], 20)], ids=lambda x: str(x).replace(" ", ""))
def test_prefill_f32_edges(hq, hkv, d, prefix, lens, window):
    rng = np.random.default_rng(len(lens) + d + hq)
    kept, start = [], prefix
    for n in lens:
        kept.append(np.sort(rng.choice(n, size=n // 3, replace=False)).astype(np.int32) + start)
        start += n
    lay = wl.layout_from_lists(prefix, lens, kept)
    w = wl.tiny_workload("f32", hq, hkv, d, T=1, B=1, k=1, seed=d + hq)
    q, k, v = wl.make_qkv(w, lay)
    got, lse = gpu_prefill(w, lay, q, k, v, want_lse=True, gl=make_layout(lay, window))
    want, wlse = oracle.prefill_blk(q, k, v, lay.n_prefix, lay.chunk_bounds, lay.sparse_offsets, lay.sparse_idx,
                                    window=window, return_lse=True)
    assert_close(got, want, "f32", what="prefill")
    assert np.abs(lse - wlse).max() <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,t_q,lens", [(2, 8, [1, 31, 32, 33]), (7, 5, [255, 256, 257, 513]), (3, 1, [0, 16, 1025, 7]),
                                         (16, 9, [512, 64, 5, 2000])], ids=lambda x: str(x).replace(" ", ""))
def test_decode_f32_edges(d, hq, t_q, lens):
    """Gathered rows, rows past the length NaN: they must never be read into O or LSE."""
    w = wl.tiny_workload("f32", hq, 1, d, T=t_q, B=len(lens), k=1, seed=d + t_q)
    rng = np.random.default_rng(d + t_q)
    cap = max(lens) + 3
    k, v = (rng.standard_normal((len(lens), 1, cap, d)).astype(np.float32) for _ in range(2))
    qd = wl.make_decode_queries(w)
    dk, dv = vxl.to_device(k, "f32"), vxl.to_device(v, "f32")
    for b, n in enumerate(lens):
        dk[b, :, n:] = dv[b, :, n:] = float("nan")
    got, lse = gpu_decode(w, qd, dk, dv, torch.tensor(lens, dtype=torch.int32, device="cuda"), want_lse=True)
    for b, n in enumerate(lens):
        if n == 0:
            assert (got[b] == 0).all() and np.isneginf(lse[b]).all()
            continue
        want, wlse = oracle.decode_lse(qd[b:b + 1], k[b:b + 1], v[b:b + 1], np.array([n], np.int32))
        assert_close(got[b:b + 1], want, "f32", head_axis=2, what=f"decode, {n} rows")
        assert np.abs(lse[b] - wlse[0]).max() <= 1e-5


@pytest.mark.parametrize("d,cap", [(64, 576), (64, 577), (128, 256), (128, 257), (64, 5000), (128, 5000)])
@pytest.mark.parametrize("hq,t_q", [(2, 1), (6, 11), (8, 16)])
def test_decode_f32_splits(d, cap, hq, t_q):
    """Both sides of the line, splits without keys among them (lengths far below the capacity), scratch full of NaN: the
    oracle's rows; the call without a workspace agrees within the tolerance, the one with static scratch bit for bit."""
    lens = [cap, 0, 1, cap // 2 + 1, 40]
    w = wl.tiny_workload("f32", hq, 2, d, T=t_q, B=len(lens), k=1, seed=d + cap)
    rng = np.random.default_rng(d + cap + t_q)
    k, v = (rng.standard_normal((len(lens), 2, cap, d)).astype(np.float32) for _ in range(2))
    dq = vxl.to_device(wl.make_decode_queries(w), "f32")
    dk, dv, ml = vxl.to_device(k, "f32"), vxl.to_device(v, "f32"), torch.tensor(lens, dtype=torch.int32, device="cuda")
    desc = desc_of(w)
    nbytes = vxl.workspace_bytes(vxl.OP_DECODE, None, desc, len(lens), t_q, cap)
    assert (nbytes > 256) == (cap > (576 if d == 64 else 256)) and nbytes <= 5 << 20
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    res = []
    for call in (lambda o, e: vxl.bilevel_decode(desc, dq, dk, dv, ml, o, e, ws),
                 lambda o, e: vxl.bilevel_decode_static(desc, dq, dk, dv, ml, o, e),
                 lambda o, e: vxl.bilevel_decode(desc, dq, dk, dv, ml, o, e, None)):
        out, lse = torch.full_like(dq, float("nan")), torch.full(dq.shape[:3], float("nan"), device="cuda")
        call(out, lse)
        res.append((vxl.to_host(out), vxl.to_host(lse)))
    (got, lse), (got_s, lse_s), (got_1, lse_1) = res
    assert np.array_equal(got, got_s) and np.array_equal(lse, lse_s)
    assert (got[1] == 0).all() and np.isneginf(lse[1]).all() and (got_1[1] == 0).all() and np.isneginf(lse_1[1]).all()
    some = [0, 2, 3, 4]
    want, wlse = oracle.decode_lse(vxl.to_host(dq)[some], k[some], v[some], np.array(lens, np.int32)[some])
    for o, e in ((got, lse), (got_1, lse_1)):
        assert_close(o[some], want, "f32", head_axis=2, what=f"decode, {cap} rows")
        assert np.abs(e[some] - wlse).max() <= 1e-5


def test_decode_inplace_f32_without_room_for_partials():
    """A workspace that holds the row map and no partial results still serves the call, within the tolerance of the one
    with room; one that does not hold the map is refused."""
    rng = np.random.default_rng(8)
    w = wl.tiny_workload("f32", 4, 2, 128, T=3, B=2, k=1, seed=8)
    lay = wl.random_layout(rng, 19, 9, 30, 90)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    masks = torch.from_numpy(rng.integers(0, 2, size=(2, lay.n_chunks)).astype(np.uint8)).cuda()
    dq, dk, dv = (vxl.to_device(x, "f32") for x in (wl.make_decode_queries(w), k, v))
    gl, desc = make_layout(lay), desc_of(w)
    full = vxl.workspace_bytes(vxl.OP_DECODE_INPLACE, gl, desc, 2, 3, lay.n_tokens)
    map_only = (2 * lay.n_tokens * 4 + 255) // 256 * 256 + 256 + 256
    assert map_only < full
    outs = []
    for n in (full, map_only, map_only - 1):
        ws, out = torch.full((n,), 255, dtype=torch.uint8, device="cuda"), torch.full_like(dq, float("nan"))
        try:
            vxl.bilevel_decode_inplace(gl, desc, dq, dk, dv, None, None, masks, lay.n_tokens, out, None, None, ws)
        except vxl.VxlError as e:
            assert e.status == vxl.VXL_ERR_WORKSPACE and n < map_only
            continue
        outs.append(vxl.to_host(out))
    assert len(outs) == 2 and np.isfinite(outs[0]).all() and np.abs(outs[0] - outs[1]).max() <= 1e-5


@pytest.mark.parametrize("d,compacted", [(64, False), (128, True), (128, False)])
def test_decode_inplace_f32(d, compacted):
    rng = np.random.default_rng(5 + d)
    w = wl.tiny_workload("f32", 6, 2, d, T=7, B=2, k=1, seed=5 + d)
    lay = wl.random_layout(rng, 19, 9, 1, 90)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    masks = rng.integers(0, 2, size=(2, lay.n_chunks)).astype(np.uint8)
    wk, wv, wlen, _ = oracle.gather_bilevel(k, v, masks, lay.n_prefix, lay.chunk_bounds, lay.sparse_offsets,
                                            lay.sparse_idx, l_cap=lay.n_tokens)
    sparse = (vxl.to_device(kept_rows(k, lay), "f32"), vxl.to_device(kept_rows(v, lay), "f32")) if compacted else None
    got, _, lens = gpu_decode_inplace(w, lay, qd, vxl.to_device(k, "f32"), vxl.to_device(v, "f32"), masks, lay.n_tokens,
                                      sparse)
    assert np.array_equal(lens, wlen)
    assert_close(got, oracle.decode_mixed(qd, wk, wv, wlen), "f32", head_axis=2, what="in place")


def expect_non_finite(got, finite, seen, bad):
    """Row-wise: `finite` is the result with the bad entries of V counted as 0; a row that sees a bad entry (bool
    `seen` [..., n_bad]) has that value in the entry's column, everything else is as without it."""
    want = finite.copy()
    with np.errstate(invalid="ignore"):                     # (inf - inf)
        for x, (d, value) in enumerate(bad):
            want[seen[..., x], d] += value
    ok = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), ok)
    assert np.abs(got[ok] - want[ok]).max() <= 1e-5
    inf = np.isinf(want)
    assert np.array_equal(got[inf], want[inf]) and np.isnan(got[~ok & ~inf]).all()


@pytest.mark.parametrize("hq,hkv,d,prefix,lens,window", [
    (7, 1, 128, 5, [31, 33, 64, 5], 0), (6, 2, 64, 33, [127, 128, 40], 40),            # keys shared by four waves
    (28, 4, 128, 20, [200, 257, 150], 30), (28, 4, 64, 0, [311, 290], 0)], ids=lambda x: str(x).replace(" ", ""))
def test_prefill_f32_row_depends_on_what_it_sees(hq, hkv, d, prefix, lens, window):
    """Infinities and NaN in V of single tokens reach the rows that see these tokens and no others."""
    rng = np.random.default_rng(d + hq)
    kept, start = [], prefix
    for n in lens:
        kept.append(np.sort(rng.choice(n, size=n // 3, replace=False)).astype(np.int32) + start)
        start += n
    lay = wl.layout_from_lists(prefix, lens, kept)
    w = wl.tiny_workload("f32", hq, hkv, d, T=1, B=1, k=1, seed=d + hq)
    q, k, v = wl.make_qkv(w, lay)
    n = lay.n_tokens
    bad = [(3, np.inf), (3, -np.inf), (d - 1, np.nan), (0, np.inf), (17, -np.inf)]
    tokens = [int(kept[0][-1]), prefix + lens[0] + 7, prefix + lens[0] - 1, n - 1, n - 2]
    finite_v = v.copy()
    for t, (col, value) in zip(tokens, bad):
        v[:, t, col], finite_v[:, t, col] = value, 0.0
    got, lse = gpu_prefill(w, lay, q, k, v, want_lse=True, gl=make_layout(lay, window))
    want, wlse = oracle.prefill_blk(q, k, finite_v, lay.n_prefix, lay.chunk_bounds, lay.sparse_offsets, lay.sparse_idx,
                                    window=window, return_lse=True)
    seen = oracle.allowed_mask(np.arange(n), lay.n_prefix, lay.chunk_bounds, lay.sparse_idx, window)[:, tokens]
    assert seen.any() and not seen.all()
    expect_non_finite(got, want, np.broadcast_to(seen, (hq, n, len(bad))), bad)
    assert np.abs(lse - wlse).max() <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
def test_decode_f32_non_finite(d):
    """The last key of a set repeats in the slots behind it; logits that are NaN or all -inf give NaN, not an empty row."""
    lens, t_q, hq = [33, 600, 17, 40, 40], 3, 4
    w = wl.tiny_workload("f32", hq, 1, d, T=t_q, B=len(lens), k=1, seed=d)
    rng = np.random.default_rng(d)
    k, v = (rng.standard_normal((len(lens), 1, max(lens), d)).astype(np.float32) for _ in range(2))
    qd = wl.make_decode_queries(w)
    finite_v = v.copy()
    bad = [(5, np.inf), (d - 2, -np.inf)]
    for b in range(3):
        for at, (col, value) in zip((lens[b] - 1, lens[b] // 2), bad):
            v[b, 0, at, col], finite_v[b, 0, at, col] = value, 0.0
    k[3, 0, 21] = np.nan
    qd[4] = np.abs(qd[4])
    k[4] = -np.inf
    got, lse = gpu_decode(w, qd, vxl.to_device(k, "f32"), vxl.to_device(v, "f32"),
                          torch.tensor(lens, dtype=torch.int32, device="cuda"), want_lse=True)
    want, wlse = oracle.decode_lse(qd[:3], k[:3], finite_v[:3], np.array(lens[:3], np.int32))
    expect_non_finite(got[:3], want, np.ones(want.shape[:3] + (len(bad),), bool), bad)
    assert np.abs(lse[:3] - wlse).max() <= 1e-4
    assert np.isnan(got[3:]).all() and np.isnan(lse[3:]).all()


@pytest.mark.parametrize("hq,n", [(2, 90), (28, 700)])
def test_prefill_f32_without_weight(hq, n):
    """A row whose visible logits are all -inf has neither output nor LSE."""
    lay = wl.layout_from_lists(0, [n], [np.zeros(0, np.int32)])
    w = wl.tiny_workload("f32", hq, 1, 64, T=1, B=1, k=1, seed=n)
    q, k, v = wl.make_qkv(w, lay)
    q, k[:, :40] = np.abs(q), -np.inf
    got, lse = gpu_prefill(w, lay, q, k, v, want_lse=True, gl=make_layout(lay))
    assert np.isnan(got[:, :40]).all() and np.isnan(lse[:, :40]).all()
    want, wlse = oracle.prefill_blk(q[:, 40:], k[:, 40:], v[:, 40:], 0, [0, n - 40], [0, 0], [], return_lse=True)
    assert np.abs(got[:, 40:] - want).max() <= 1e-5 and np.abs(lse[:, 40:] - wlse).max() <= 1e-4


def test_decode_f32_more_queries_than_a_grid_dimension_holds():
    """70,000 queries of one token over sets of 0 to 3 rows: past the 65,535 workgroups of a grid's y or z."""
    b, cap, d = 70000, 3, 64
    gen = torch.Generator(device="cuda").manual_seed(5)
    qd, km, vm = (torch.empty(s, device="cuda").normal_(generator=gen) for s in ((b, 1, 2, d), (b, 1, cap, d), (b, 1, cap, d)))
    ml = (torch.arange(b, device="cuda") % 4).to(torch.int32)
    desc = vxl.make_desc(2, 1, d, "f32")
    out, lse = torch.full_like(qd, float("nan")), torch.full((b, 1, 2), float("nan"), device="cuda")
    vxl.bilevel_decode(desc, qd, km, vm, ml, out, lse, vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_DECODE, None, desc, b, 1, cap)))
    s = (qd[:, 0, :, None].double() * km.double()).sum(-1) / d ** 0.5                    # [b, 2, cap]
    s = s.masked_fill(torch.arange(cap, device="cuda")[None, None] >= ml[:, None, None], float("-inf"))
    want = (torch.softmax(s, -1).nan_to_num(0.0)[..., None] * vm.double()).sum(-2)
    assert (out[:, 0].double() - want).abs().max().item() <= 1e-5
    some = ml > 0
    assert (lse[some, 0].double() - torch.logsumexp(s[some], -1)).abs().max().item() <= 1e-5
    assert (lse[~some] == float("-inf")).all()
