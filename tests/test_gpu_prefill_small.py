"""Small prompts, which take the pre-filling instances of four and eight waves without pre-pass and queue: the instance
that the library chooses and that of large prompts against the oracle on layouts on either side of the line between four
and eight waves (256 parts at D = 128) and on ragged ones, with a look-back window and token-major storage."""
import time

import numpy as np
import pytest
import torch

from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import assert_close, desc_of, gpu_prefill, make_layout, prefill_variant
from test_gpu_parity import oracle_prefill

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 2])
@pytest.mark.parametrize("hq,hkv,d,prefix,lens,window", [
    (8, 1, 128, 0, [256] * 16, 0),                 # 256 parts: the last size of the 4-wave instance
    (8, 1, 128, 1, [256] * 16, 0),                 # 258 parts
    (14, 2, 128, 64, [130, 319, 201, 256], 100),   # ragged bands: one row, one block, a full band
    (7, 1, 128, 33, [1, 31, 129, 128, 127], 40),
    (28, 4, 128, 64, [160, 161], 0),
    (4, 4, 64, 17, [200] * 5 + [64], 64),          # one head per KV head
    (14, 2, 64, 0, [97, 400], 0),
    (14, 2, 64, 30, [256] * 19, 0),                # two 4-wave workgroups per compute unit
    (8, 8, 64, 17, [97, 63, 200], 0),              # at most one, though two would fit
    (28, 4, 128, 0, [192] * 5, 0),                 # few keys for 220 parts
])
def test_small_prompts_match_the_oracle(variant, hq, hkv, d, prefix, lens, window):
    rng = np.random.default_rng(91 + sum(lens))
    starts = prefix + np.concatenate([[0], np.cumsum(lens)[:-1]])
    kept = [np.sort(s + rng.choice(n, max(1, n // 8), replace=False)).astype(np.int32) for s, n in zip(starts, lens)]
    lay = wl.layout_from_lists(prefix, lens, kept)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=1, B=1, k=1, seed=91, value_scale=1.0)
    q, k, v = wl.make_qkv(w, lay)
    vxl.debug_prefill_variant(variant)
    try:
        got, lse = gpu_prefill(w, lay, q, k, v, want_lse=True, gl=make_layout(lay, window=window))
    finally:
        vxl.debug_prefill_variant(0)
    want, wlse = oracle_prefill(q, k, v, lay, return_lse=True, window=window)
    assert_close(got, want, "bf16", what=f"{lens[:4]} variant {variant}")
    assert np.abs(lse - wlse).max() < 2e-2


@pytest.mark.parametrize("hq,hkv,d,prefix,lens,window,every", [
    (14, 2, 128, 0, [70, 1, 200, 64], 0, 3),           # four waves: history without a prefix, tile edges inside it
    (14, 2, 128, 63, [70, 1, 200, 64], 0, 3),          # a tile of prefix and kept rows
    (7, 1, 64, 64, [65, 129, 300], 0, 2),              # the prefix ends with a tile
    (7, 1, 64, 65, [65, 129, 300], 90, 2),
    (28, 4, 128, 17, [20] * 24, 0, 20),                # eight waves: many short segments, one kept row each
    (28, 4, 128, 130, [300] * 5 + [31], 256, 7),       # history that ends inside the prefix's last tile
    (8, 1, 128, 1, [256] * 17, 0, 8),                  # parts dealt to the XCDs in turn (eight heads on one KV head)
    (5, 1, 64, 40, [90] * 12, 33, 4),                  # row tiles of five heads
    (3, 3, 128, 40, [190] * 4, 0, 4),                  # KV heads that do not divide the eight XCDs
    (1, 1, 128, 0, [700] * 12 + [100], 0, 1),          # 8,500 kept rows: no room for their table
    (4, 2, 64, 256, [40] * 30, 0, 8),                  # chunks of one part, a prefix of two (four waves: of four)
    (12, 1, 128, 300, [33, 20, 64] * 6, 0, 8),         # a prefix of two bands, the last one ragged
    (6, 3, 64, 700, [50] * 12, 20, 8),                 # the same where one queue serves all heads
    (7, 1, 128, 130, [300, 20, 500], 0, 8),            # chunks with more parts than the prefix
])
def test_parts_and_history_without_queue_and_pre_pass(hq, hkv, d, prefix, lens, window, every):
    """What the library chooses, and the queue with late claims, against the oracle and against the instance of large
    prompts, whose tiles and row blocks are the same."""
    rng = np.random.default_rng(95 + sum(lens))
    starts = prefix + np.concatenate([[0], np.cumsum(lens)[:-1]])
    kept = [np.sort(s + rng.choice(n, max(1, n // every), replace=False)).astype(np.int32) for s, n in zip(starts, lens)]
    lay = wl.layout_from_lists(prefix, lens, kept)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=1, B=1, k=1, seed=95, value_scale=1.0)
    q, k, v = wl.make_qkv(w, lay)
    gl = make_layout(lay, window=window)
    res = []
    for variant in (0, 3, 2):
        with prefill_variant(variant):
            res.append(gpu_prefill(w, lay, q, k, v, want_lse=True, gl=gl))
    want, wlse = oracle_prefill(q, k, v, lay, return_lse=True, window=window)
    for got, lse in res:
        assert_close(got, want, "bf16", what=f"{prefix} + {lens[:4]}")
        assert np.abs(lse - wlse).max() < 2e-2
        assert np.array_equal(got, res[-1][0]) and np.array_equal(lse, res[-1][1])
    # token-major storage reads and writes the same rows
    desc = vxl.make_desc(hq, hkv, d, "bf16", token_major=True)
    ten = [vxl.to_device(x, "bf16").transpose(0, 1).contiguous() for x in (q, k, v)]
    out = torch.full_like(ten[0], float("nan"))
    vxl.chunk_prefill(gl, desc, *ten, out, None, vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_PREFILL, gl, desc)))
    assert np.array_equal(vxl.to_host(out.transpose(0, 1)), res[-1][0])


@pytest.mark.parametrize("d", [64, 128])
def test_small_prompt_token_major_equals_head_major(d):
    """The strided instance of the 4-wave form gives the dense one's bits; a replayed graph gives them again."""
    lay = wl.layout_from_lists(20, [150, 70, 300], [wl.strided_kept(20, 150, 10), wl.strided_kept(170, 70, 3),
                                                    wl.strided_kept(240, 300, 30)])
    w = wl.tiny_workload("bf16", 14, 2, d, T=1, B=1, k=1, seed=92)
    q, k, v = (vxl.to_device(x, "bf16") for x in wl.make_qkv(w, lay))
    gl = make_layout(lay)
    outs = []
    for token_major in (False, True):
        desc = vxl.make_desc(14, 2, d, "bf16", token_major=token_major)
        ten = [x.transpose(0, 1).contiguous() if token_major else x for x in (q, k, v)]
        o = torch.empty_like(ten[0])
        ws = torch.randint(0, 256, (vxl.workspace_bytes(vxl.OP_PREFILL, gl, desc),), dtype=torch.uint8, device="cuda")
        vxl.chunk_prefill(gl, desc, *ten, o, None, ws)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        first = o.clone()
        with torch.cuda.graph(graph):
            vxl.chunk_prefill(gl, desc, *ten, o, None, ws)
        for _ in range(3):
            o.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(o, first)
        outs.append(first.transpose(0, 1).contiguous() if token_major else first)
    assert torch.equal(*outs)


def test_host_time_does_not_grow_with_the_chunks():
    """The choice of the instance costs the same for one chunk and for as many as a layout takes (with a walk over them the
    call took 6.7 us for one chunk and 21.3 for 4,096; without 9.2)."""
    best = []
    for lens in ([4096], [1] * 4096):
        lay = wl.layout_from_lists(0, lens, [np.zeros(0, np.int32)] * len(lens))
        w = wl.tiny_workload("bf16", 7, 1, 64, T=1, B=1, k=1, seed=93)
        q, k, v = (vxl.to_device(x, "bf16") for x in wl.make_qkv(w, lay))
        gl, desc, o = make_layout(lay), desc_of(w), torch.empty_like(q)
        ws = vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_PREFILL, gl, desc))
        took = []
        for _ in range(60):
            start = time.perf_counter()
            vxl.chunk_prefill(gl, desc, q, k, v, o, None, ws)
            took.append(time.perf_counter() - start)
            torch.cuda.synchronize()
        best.append(min(took))
    assert best[1] < best[0] + 8e-6, best


@pytest.mark.parametrize("hq,hkv,d,prefix,lens,window,every", [
    (7, 1, 64, 65, [65, 129, 300], 90, 2), (4, 4, 64, 17, [200] * 5 + [64], 0, 1), (14, 2, 128, 63, [70, 1, 200, 64], 0, 3),
    (3, 3, 128, 0, [128, 129], 0, 8)])
def test_four_waves_with_pre_pass(hq, hkv, d, prefix, lens, window, every):
    """The instance of four waves with pre-pass and queue against the oracle and, bit for bit, the one of large prompts."""
    rng = np.random.default_rng(96 + sum(lens))
    starts = prefix + np.concatenate([[0], np.cumsum(lens)[:-1]])
    kept = [np.sort(s + rng.choice(n, max(1, n // every), replace=False)).astype(np.int32) for s, n in zip(starts, lens)]
    lay = wl.layout_from_lists(prefix, lens, kept)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=1, B=1, k=1, seed=96, value_scale=1.0)
    q, k, v = wl.make_qkv(w, lay)
    res = []
    for variant in (4, 2):
        with prefill_variant(variant):
            res.append(gpu_prefill(w, lay, q, k, v, want_lse=True, gl=make_layout(lay, window=window)))
    want, wlse = oracle_prefill(q, k, v, lay, return_lse=True, window=window)
    assert_close(res[0][0], want, "bf16", what=f"{lens[:4]}")
    assert np.abs(res[0][1] - wlse).max() < 2e-2
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])


@pytest.mark.parametrize("hq,hkv,d,prefix,chunks,length,every", [
    (4, 4, 64, 0, 170, 72, 8), (4, 4, 64, 256, 170, 72, 8),       # chunks of four cells at most, two workgroups per unit
    (4, 4, 64, 64, 100, 72, 4),                                    # the same, few of them: eight waves
    (4, 4, 64, 64, 250, 40, 2),                                    # no room for the kept rows of two: with the pre-pass
    (4, 2, 64, 0, 150, 72, 2),                                     # the same, 302 parts of eight waves
    (14, 2, 64, 256, 150, 40, 8),                                  # 1,200 parts of four waves
    (2, 1, 128, 256, 43, 160, 2),                                  # 60 tiles of history, a compute unit for every part
    (4, 4, 128, 64, 200, 40, 2), (4, 4, 128, 64, 240, 100, 8)])    # three parts per unit, one head per KV head: early claims
def test_chosen_instance_of_many_short_chunks(hq, hkv, d, prefix, chunks, length, every):
    """Prompts on the sides of the lines between the instances: bit for bit what the instance of large prompts gives."""
    lay = wl.layout_from_lists(prefix, [length] * chunks,
                               [wl.strided_kept(prefix + i * length, length, length // every) for i in range(chunks)])
    w = wl.tiny_workload("bf16", hq, hkv, d, T=1, B=1, k=1, seed=97, value_scale=1.0)
    gen = torch.Generator(device="cuda").manual_seed(chunks + d)
    dev = [torch.empty((h, lay.n_tokens, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=gen) for h in (hq, hkv, hkv)]
    res = []
    for variant in (0, 2):
        with prefill_variant(variant):
            res.append(gpu_prefill(w, lay, None, None, None, want_lse=True, dev=dev))
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])
