"""GPU parity of the softmax attention-mass relevance score (vxl_chunk_score_topk_mass) against
the float64 oracle.  Scores are compared numerically; the selection is compared bit for bit with
a full sort of the device's own fp32 scores (both sides decide in fp32) and, wherever the rank-k
margin of the oracle's scores exceeds the score tolerance, with the oracle's selection."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import check_selection_valid, full_sort_selection, gpu_score_topk_mass

pytestmark = pytest.mark.gpu

RTOL = 1e-4       # fp32 exponentials and sums of up to ~10^5 terms against float64


def check_mass(w, lay, qd, k, top_k, scale=0.0, rtol=RTOL):
    idx, mask, scores = gpu_score_topk_mass(w, lay, qd, k, top_k, scale=scale)
    want = oracle.chunk_scores_mass(qd, k, lay.n_prefix, lay.chunk_bounds, scale=scale or None)
    tol = rtol * np.abs(want).max()
    assert np.isfinite(scores).all()
    assert np.abs(scores - want).max() <= tol, (np.abs(scores - want).max(), tol)
    assert (scores.sum(axis=1) <= 1.0 + 1e-4).all()          # the prefix holds the rest of the mass
    # the device's selection is the full-sort selection of its own scores, bit for bit
    own_idx, own_mask = full_sort_selection(scores, top_k)
    assert np.array_equal(idx, own_idx) and np.array_equal(mask, own_mask)
    # and a valid selection for the oracle's scores: nothing clearly better is left out
    check_selection_valid(idx, mask, want, oracle.select_topk(want, top_k)[1], top_k, tol)
    return idx, mask, scores


def test_mass_config0_fp32():
    w = wl.WORKLOADS["config0"]
    lay = wl.make_layout(w)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    for top_k in (0, 1, w.k, lay.n_chunks + 3):
        check_mass(w, lay, qd, k, top_k, rtol=2e-5)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_mass_ragged_layouts(dtype, d):
    rng = np.random.default_rng(71 + d)
    # odd chunk lengths, a short prefix, 9 stacked rows per KV head (not a multiple of 32)
    w = wl.tiny_workload(dtype, 6, 2, d, T=3, B=3, k=2, seed=71)
    lay = wl.random_layout(rng, 5, 13, 1, 300)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    for top_k in (1, 4, 13):
        check_mass(w, lay, qd, k, top_k)
    # no prefix, one chunk longer than a piece (several items per chunk), 224 stacked rows (two
    # row tiles), a custom scale
    w = wl.tiny_workload(dtype, 14, 2, d, T=32, B=2, k=2, seed=72, value_scale=0.5)
    lay = wl.layout_from_lists(0, [2500, 77, 1024, 1025, 64], [np.zeros(0, np.int32)] * 5)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    check_mass(w, lay, qd, k, 2, scale=0.2)


def test_mass_exact_ties_go_to_the_lower_chunk():
    w = wl.tiny_workload("bf16", 4, 2, 128, T=2, B=1, k=2, seed=73, value_scale=0.3)
    ln = 70
    lay = wl.layout_from_lists(3, [ln] * 5, [np.zeros(0, np.int32)] * 5)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = np.abs(wl.make_decode_queries(w))
    blk = np.abs(k[:, 3 + ln:3 + 2 * ln]).copy()
    for c in (1, 3, 4):
        k[:, 3 + c * ln:3 + (c + 1) * ln] = blk
    for c in (0, 2):
        k[:, 3 + c * ln:3 + (c + 1) * ln] = -np.abs(k[:, 3 + c * ln:3 + (c + 1) * ln])
    idx, mask, scores = gpu_score_topk_mass(w, lay, qd, k, 2)
    assert scores[0, 1] == scores[0, 3] == scores[0, 4]
    assert list(idx[0]) == [1, 3] and list(mask[0]) == [0, 1, 0, 1, 0]


def test_mass_config1_and_sharp_queries():
    w = wl.WORKLOADS["config1"]
    lay = wl.make_layout(w)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    check_mass(w, lay, qd, k, w.k)
    # sharp softmax: queries scaled so that the logits have a standard deviation of about 3
    qs = wl.round_to_bf16(qd * np.float32(np.sqrt(128.0) * 3.0 * np.sqrt(128.0)))
    check_mass(w, lay, qs, k, w.k)


def test_mass_matrix_core_kernel_agrees_with_vector_kernel_on_device():
    rng = np.random.default_rng(74)
    w = wl.tiny_workload("bf16", 14, 2, 128, T=5, B=2, k=3, seed=74)
    lay = wl.random_layout(rng, 40, 9, 30, 700)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    _, mask_a, sc_a = gpu_score_topk_mass(w, lay, qd, k, 3)
    vxl.debug_force_simple(True)
    try:
        _, mask_b, sc_b = gpu_score_topk_mass(w, lay, qd, k, 3)
    finally:
        vxl.debug_force_simple(False)
    assert np.abs(sc_a - sc_b).max() <= 2e-5 * np.abs(sc_b).max()
    assert np.array_equal(mask_a, mask_b)


@pytest.mark.parametrize("name", ["config2", "config4"])
def test_mass_full_size(name):
    """Full-size layouts (131,328 tokens with T = 64; variable chunks with 8 queries)."""
    w = wl.WORKLOADS[name]
    lay = wl.make_layout(w)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    check_mass(w, lay, qd, k, w.k)


@pytest.mark.parametrize("d,t,lens", [(64, 1, [64, 65, 1, 200]), (128, 19, [63, 640, 129]), (128, 64, [1025, 300])])
def test_mass_reference_raised_inside_an_item(d, t, lens):
    """Logits that climb by far more than 2^30 (exp2 domain) from the first tile of an item to its last, fall again in
    the next chunk and differ in sign between the rows of a wave; row counts around the 128-row tile."""
    w = wl.tiny_workload("bf16", 14, 2, d, T=t, B=2, k=2, seed=75)
    lay = wl.layout_from_lists(5, lens, [np.zeros(0, np.int32)] * len(lens))
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    ramp = np.concatenate([np.linspace(-1, 1, 5)] + [np.linspace(-1, 1, n) * (1 - 2 * (i % 2)) for i, n in enumerate(lens)])
    k = wl.round_to_bf16(k * 0.1 + ramp[None, :, None].astype(np.float32) * np.sign(k[:, :1, :]))
    qd = wl.round_to_bf16((np.sign(qd) * np.float32(0.2) + np.sign(k[0, 0])) * 3)
    check_mass(w, lay, qd, k, 2, scale=1.0)


@pytest.mark.parametrize("n_items", [1, 8, 9, 16, 17, 63, 64, 65, 128, 130, 512, 513, 641])
def test_mass_row_statistics_at_the_edges_of_their_batches(n_items):
    """The items of a row are folded by 8 groups of 2 at a time, 16 groups of 4 or 32 of 4: around one batch of each, with
    items whose mass differs by orders of magnitude; 33 stacked rows, one more than a block holds."""
    rng = np.random.default_rng(76 + n_items)
    w = wl.tiny_workload("bf16", 6, 2, 64, T=11, B=2, k=1, seed=76)
    lay = wl.layout_from_lists(0, rng.integers(1, 40, n_items).tolist(), [np.zeros(0, np.int32)] * n_items)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    k = wl.round_to_bf16(k * np.repeat(rng.uniform(0.2, 6.0, n_items), np.diff(lay.chunk_bounds))[None, :, None].astype(np.float32))
    check_mass(w, lay, wl.make_decode_queries(w), k, min(3, n_items))


def test_mass_more_workgroups_than_a_grid_dimension_holds():
    """4,104 heads over 4,096 chunks of one token: 2^24 workgroups of 256 threads are 2^32 threads, a grid's limit in x."""
    h, c, d = 4104, 4096, 64
    gen = torch.Generator(device="cuda").manual_seed(6)
    k = torch.empty((h, c, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    qd = torch.empty((1, 1, h, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    layout = vxl.Layout(0, np.arange(c + 1, dtype=np.int32), np.zeros(c + 1, np.int32), np.zeros(0, np.int32))
    desc = vxl.make_desc(h, h, d, "bf16")
    idx, mask = torch.zeros((1, 1), dtype=torch.int32, device="cuda"), torch.zeros((1, c), dtype=torch.uint8, device="cuda")
    scores = torch.full((1, c), float("nan"), device="cuda")
    vxl.chunk_score_topk_mass(layout, desc, qd, k, 1, idx, mask, scores,
                              workspace=vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_SCORE_MASS, layout, desc, batch=1, n_q_tokens=1)))
    want = torch.zeros(c, dtype=torch.float64, device="cuda")
    for g in range(0, h, 216):
        logits = (k[g:g + 216].float() * qd[0, 0, g:g + 216, None].float()).sum(-1).double() / d ** 0.5
        want += torch.softmax(logits, -1).sum(0) / h
    assert (scores[0].double() - want).abs().max().item() <= RTOL * want.max().item()


@pytest.mark.parametrize("hq,hkv,t,bsz,d", [(8, 8, 1, 4, 128), (8, 8, 1, 4, 64), (32, 4, 33, 3, 128), (32, 4, 33, 3, 64),
                                            (8, 1, 3, 2, 128)])
def test_mass_items_in_turn_and_first_keys_far_off(hq, hkv, t, bsz, d):
    """Chunks of 1 to 130 keys, enough of them for a workgroup to take several in turn (the last case: too few), their
    first keys, whose logits an item's sums start from, tens of units above and below the others'."""
    rng = np.random.default_rng(77 + d)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=5, seed=77, value_scale=1.0)
    lay = wl.random_layout(rng, 70, 140, 1, 130)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    first = lay.chunk_bounds[:-1]
    k[:, first] = wl.round_to_bf16(k[:, first] * rng.choice([-30.0, 1.0, 30.0], size=len(first)).astype(np.float32)[None, :, None])
    check_mass(w, lay, wl.make_decode_queries(w), k, 5)


@pytest.mark.parametrize("hq,hkv,t,d", [(14, 2, 1, 128), (8, 1, 3, 64), (28, 4, 5, 128)])
def test_mass_of_a_query_does_not_depend_on_its_neighbours(hq, hkv, t, d):
    """Queries whose rows share a wave, every other one with logits that make it raise its references (tens of octaves):
    each query's scores are those of a call of its own, bit for bit."""
    rng = np.random.default_rng(99 + d)
    bsz = 6
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=3, seed=99, value_scale=1.0)
    lay = wl.random_layout(rng, 9, 24, 1, 400)
    _, k, _ = wl.make_qkv(w, lay, with_q=False)
    qd = wl.make_decode_queries(w)
    qd[1::2] = wl.round_to_bf16(qd[1::2] * np.float32(20.0))
    _, _, scores = check_mass(w, lay, qd, k, 3)
    for b in range(bsz):
        _, _, own = gpu_score_topk_mass(w, lay, qd[b:b + 1], k, 3)
        assert np.array_equal(own[0].view(np.uint32), scores[b].view(np.uint32)), b


@pytest.mark.parametrize("hq,t", [(1, 1), (1, 40)])
def test_mass_error_where_first_keys_lie_far_below(hq, t):
    """Chunks of a few keys whose first logit lies 19 octaves below the others, logits exact in fp32: against the largest
    logit of a tile the exponents that count are near 0 and exact, and the rest is some eight roundings of 2^-24 (the
    exponentials of a key, of its item and of its row, and the products), 1.7e-7 in root mean square.  An exponent
    of 19 is rounded by up to 2^-20, 3.8e-7 of the value in root mean square."""
    rng = np.random.default_rng(55 + t)
    lens = rng.integers(2, 6, size=200)
    w = wl.tiny_workload("bf16", hq, 1, 64, T=t, B=2, k=3, seed=55)
    lay = wl.layout_from_lists(0, lens.tolist(), [np.zeros(0, np.int32)] * len(lens))
    k = np.zeros((1, lay.n_tokens, 64), np.float32)
    k[0, :, 0] = rng.integers(208, 224, size=lay.n_tokens) / 16.0                  # exact in bf16: 13 to 14
    k[0, lay.chunk_bounds[:-1], 0] = 0.0
    qd = np.zeros((2, t, hq, 64), np.float32)
    qd[..., 0] = 1.0
    _, _, scores = check_mass(w, lay, qd, k, 3, scale=1.0)
    want = oracle.chunk_scores_mass(qd, k, 0, lay.chunk_bounds, scale=1.0)
    assert np.sqrt((((scores - want) / want) ** 2).mean()) <= 1.7e-7
