"""The fp32 matrix-instruction kernels at the sizes where a row block (16 stacked rows), a key tile (32) or the
slices of the waves that share a block's keys are partly filled or empty, and on both sides of the line between
shared and unshared keys (16 rows per SIMD of the chip).  Tolerance: the path's 1e-5 for fp32 storage."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import assert_close, gpu_decode, gpu_decode_inplace, gpu_prefill, kept_rows, make_layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,prefix,lens,window", [
    (1, 1, 64, 0, [1, 2, 15, 16, 17], 0), (7, 1, 128, 1, [31, 32, 33, 5], 0), (6, 2, 64, 33, [127, 128, 129, 300], 40),
    (8, 1, 128, 130, [640, 700, 641], 0), (28, 4, 64, 64, [257, 1, 511], 100)], ids=lambda x: str(x).replace(" ", ""))
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
    want = oracle.prefill_blk(q, k, v, lay.n_prefix, lay.chunk_bounds, lay.sparse_offsets, lay.sparse_idx, window=window)
    assert_close(got, want, "f32", what="prefill")
    assert np.isfinite(lse).all()


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
