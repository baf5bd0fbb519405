"""Scores and selection at the chunk counts where the kernels change form or a block, wave or key pair is only
partly filled: one launch up to 128 chunks, of short rows 192 (blocks for 16, 32 and 64 chunks at once), 16 chunks per score block and
64 per selection block beyond."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import desc_of, full_sort_selection, gpu_score_topk, make_layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_chunks", [1, 2, 15, 16, 17, 18, 31, 32, 33, 34, 63, 64, 65, 127, 128, 129, 143, 191, 193, 640, 1025, 4095, 4096])
def test_selection_is_a_full_sort_of_the_scores(n_chunks):
    """Every third chunk repeats one of a few contents, so that many scores tie exactly; the scores agree with the
    oracle to the rounding of 3 x 128 fp32 products (2e-5 of the largest), the selection is the full sort of them."""
    rng = np.random.default_rng(n_chunks)
    hkv, d, ln = (3, 128, 2) if n_chunks % 2 else (1, 64, 3)
    w = wl.tiny_workload("f32", 2 * hkv, hkv, d, T=3, B=2, k=1, seed=n_chunks)
    lay = wl.layout_from_lists(5, [ln] * n_chunks, [np.zeros(0, np.int32)] * n_chunks)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    blocks = k[:, 5:].reshape(hkv, n_chunks, ln, d)                        # (a view: k changes)
    for c in range(0, n_chunks, 3):
        blocks[:, c] = blocks[:, (c // 3) % min(4, n_chunks)]
    qd = wl.make_decode_queries(w)
    want = oracle.chunk_scores(qd, k, lay.chunk_bounds)
    for top_k in sorted({0, 1, n_chunks // 2, n_chunks}):
        print(n_chunks, top_k, flush=True)
        idx, mask, scores = gpu_score_topk(w, lay, qd, k, top_k)
        assert np.abs(scores - want).max() <= 2e-5 * np.abs(want).max()
        own_idx, own_mask = full_sort_selection(scores, top_k)
        assert np.array_equal(idx, own_idx) and np.array_equal(mask, own_mask)


@pytest.mark.parametrize("hkv,d", [(1, 64), (2, 64), (1, 128), (3, 64), (2, 128), (16, 128)])
def test_a_score_does_not_depend_on_the_number_of_chunks(hkv, d):
    """The first chunks of a prompt get the same bits from every form of the score kernel (rows of 16 to 512 pieces)."""
    rng = np.random.default_rng(hkv * d)
    counts, ln = (16, 17, 32, 33, 64, 65, 128, 129, 300), 2
    w = wl.tiny_workload("f32", 2 * hkv, hkv, d, T=3, B=2, k=1, seed=d)
    k = rng.standard_normal((hkv, 300 * ln, d)).astype(np.float32)
    qd = wl.make_decode_queries(w)
    want = None
    for n_chunks in counts:
        lay = wl.layout_from_lists(0, [ln] * n_chunks, [np.zeros(0, np.int32)] * n_chunks)
        _, _, scores = gpu_score_topk(w, lay, qd, np.ascontiguousarray(k[:, :n_chunks * ln]), 1)
        want = scores[:, :16].copy() if want is None else want
        assert np.array_equal(scores[:, :16].view(np.uint32), want.view(np.uint32)), n_chunks


@pytest.mark.parametrize("dtype,hkv,d,lens", [
    ("bf16", 2, 128, [700, 64, 1000, 333, 1, 31, 480, 481, 495, 1024]),    # 512 threads: every number of last rows
    ("f32", 2, 128, [400, 16, 47, 48, 49, 64, 300, 301]),
    ("f32", 1, 64, [900, 15, 500]),
    ("bf16", 3, 64, [900, 15, 500, 97]),                                   # short rows: 256 threads
    ("bf16", 2, 128, [300, 15, 16, 17, 63, 64, 65, 47]),                   # 256 threads: short chunks
])
def test_mean_keys_of_long_and_ragged_chunks(dtype, hkv, d, lens):
    """Scores of chunks whose rows leave threads with every remainder, the first two equal where they are as long; the
    rounding of sums of up to 1,024 fp32 values in parts of at most 32 is below 2e-6 of a mean's terms."""
    lens = lens[:1] + lens                                                 # (equal contents below: an exact tie)
    w = wl.tiny_workload(dtype, 2 * hkv, hkv, d, T=5, B=2, k=3, seed=d, value_scale=1.0)
    lay = wl.layout_from_lists(3, lens, [np.zeros(0, np.int32)] * len(lens))
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    k[:, 3 + lens[0]:3 + 2 * lens[0]] = k[:, 3:3 + lens[0]]
    qd = wl.make_decode_queries(w)
    want = oracle.chunk_scores(qd, k, lay.chunk_bounds)
    idx, mask, scores = gpu_score_topk(w, lay, qd, k, 3)
    assert np.abs(scores - want).max() <= 2e-5 * np.abs(want).max()
    assert np.array_equal(scores[:, 0], scores[:, 1])
    own_idx, own_mask = full_sort_selection(scores, 3)
    assert np.array_equal(idx, own_idx) and np.array_equal(mask, own_mask)


@pytest.mark.parametrize("dtype,hkv,d,lens", [
    ("bf16", 4, 128, [400, 333, 700, 1, 31, 32, 33, 64, 65, 127, 500]),     # 512 threads up to 128 chunks, then 256
    ("f32", 2, 128, [300, 1, 15, 16, 17, 31, 33, 500, 499]),                # 256 chunks
])
def test_means_do_not_depend_on_the_number_of_chunks(dtype, hkv, d, lens):
    """The first chunks' mean keys and scores have the same bits in a prompt of few long chunks, which 512 threads sum,
    and in one of more of them, which 256 do."""
    rng = np.random.default_rng(d + hkv)
    w = wl.tiny_workload(dtype, 2 * hkv, hkv, d, T=3, B=1, k=1, seed=d, value_scale=1.0)
    many = 512 // hkv + 1 - len(lens)
    k = rng.standard_normal((hkv, sum(lens) + 700 * many, d)).astype(np.float32)
    k = wl.round_to_bf16(k) if dtype == "bf16" else k
    qd, res = wl.make_decode_queries(w), []
    for all_lens in (lens + [700] * 4, lens + [700] * many):
        lay = wl.layout_from_lists(0, all_lens, [np.zeros(0, np.int32)] * len(all_lens))
        gl, desc = make_layout(lay), desc_of(w)
        dk, dq = vxl.to_device(np.ascontiguousarray(k[:, :lay.n_tokens]), dtype), vxl.to_device(qd, dtype)
        idx, mask = torch.zeros((1, 1), dtype=torch.int32, device="cuda"), torch.zeros((1, lay.n_chunks), dtype=torch.uint8, device="cuda")
        scores = torch.zeros((1, lay.n_chunks), device="cuda")
        kbar = torch.zeros((hkv, lay.n_chunks, d), device="cuda")
        vxl.chunk_score_topk(gl, desc, dq, dk, 1, idx, mask, scores, kbar,
                             workspace=vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_SCORE_TOPK, gl, desc, 1)))
        res.append((kbar[:, :len(lens)].cpu().numpy(), scores[:, :len(lens)].cpu().numpy()))
    for a, b in zip(*res):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("dtype,hq,hkv,d,bsz,t", [
    ("bf16", 28, 4, 128, 1, 8), ("bf16", 28, 4, 128, 2, 9),                # the last of one block per row, the first of four
    ("bf16", 14, 2, 128, 3, 17), ("bf16", 14, 2, 64, 1, 128), ("bf16", 8, 1, 128, 1, 127), ("bf16", 4, 4, 64, 2, 200),
    ("bf16", 64, 1, 64, 1, 33), ("bf16", 70, 1, 128, 1, 40),               # a piece per thread, more pieces than threads
    ("f32", 6, 2, 64, 2, 65), ("f32", 6, 2, 128, 1, 130)])
def test_scores_of_many_query_tokens(dtype, hq, hkv, d, bsz, t):
    """The mean over query tokens and heads by one thread per piece and by groups of them: rounding of fp32 sums (as above)."""
    rng = np.random.default_rng(t * d)
    w = wl.tiny_workload(dtype, hq, hkv, d, T=t, B=bsz, k=2, seed=t, value_scale=1.0)
    lay = wl.random_layout(rng, 9, 7, 1, 60)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = rng.standard_normal((bsz, t, hq, d)).astype(np.float32) + rng.standard_normal((1, 1, 1, d)).astype(np.float32)
    qd = wl.round_to_bf16(qd) if dtype == "bf16" else qd
    want = oracle.chunk_scores(qd, k, lay.chunk_bounds)
    _, _, scores = gpu_score_topk(w, lay, qd, k, 2)
    assert np.abs(scores - want).max() <= 2e-5 * np.abs(want).max()


def test_mean_query_does_not_depend_on_the_layout():
    """40 tokens; 20 long chunks, whose launch has 512 threads per block, and 300, whose has 256: the same scores, bit for bit."""
    ln, hkv, d = 320, 2, 128
    w = wl.tiny_workload("bf16", 14, hkv, d, T=40, B=2, k=1, seed=3, value_scale=1.0)
    gen = torch.Generator(device="cuda").manual_seed(3)
    k = torch.empty((hkv, 300 * ln, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=gen)
    qd = vxl.to_device(wl.make_decode_queries(w), "bf16")
    got = []
    for n in (20, 300):
        lay = wl.layout_from_lists(0, [ln] * n, [np.zeros(0, np.int32)] * n)
        gl, desc, kn = make_layout(lay), desc_of(w), k[:, :n * ln].contiguous()
        idx = torch.empty((2, 1), dtype=torch.int32, device="cuda")
        mask = torch.empty((2, n), dtype=torch.uint8, device="cuda")
        scores = torch.empty((2, n), dtype=torch.float32, device="cuda")
        vxl.chunk_score_topk(gl, desc, qd, kn, 1, idx, mask, scores,
                             workspace=vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_SCORE_TOPK, gl, desc, 2, 40)))
        got.append(scores[:, :20].cpu())
    assert torch.equal(*got)
