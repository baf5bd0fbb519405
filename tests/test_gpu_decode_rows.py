"""Decode calls whose stacked query rows fill several 32-row blocks over a short mixed set: the row blocks of a key
split as separate workgroups, gathered and in place, against the oracle at the edges of the row blocks, the key tiles and
the launch's grouping by eights."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import assert_close, desc_of, gpu_decode, gpu_decode_inplace, make_layout
from test_gpu_inplace import check_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,t,d,lens", [
    (11, 1, 6, 128, [700, 33, 0]),                 # 66 rows: two rows in the last block
    (14, 2, 5, 64, [1, 129]),                      # 35 rows, fewer tiles than waves
    (14, 2, 5, 128, [2500, 2113, 0, 31, 64, 2049, 7, 1000]),      # 35 rows, two tiles per wave
    (8, 1, 12, 64, [4097]),                        # 96 rows: whole blocks
    (28, 4, 32, 128, [4352]),                      # 224 rows over the mixed set of a 16k-token prompt
    (28, 4, 36, 128, [1029, 515]),                 # 252 rows, units that do not divide by eight
    (28, 4, 64, 128, [1031]),                      # 448 rows
    (7, 1, 128, 64, [300]),                        # 896 rows: 28 blocks on one XCD
    (28, 4, 96, 128, [700, 33, 0]),                # twelve units of 21 blocks: two on some XCDs
    (28, 4, 96, 64, [1400, 1399, 5]),
    (7, 1, 96, 128, [450, 1, 31, 32, 33, 64, 449, 0, 128]),       # nine units of 21 blocks
    (8, 1, 160, 128, [2600]),                      # 40 blocks: the ring kernel
    (8, 1, 160, 64, [1290]),                       # 40 blocks on one XCD, two per compute unit
    (2, 2, 1, 128, [700, 1, 0, 33]),               # one row: fewer floats than threads to merge them
    (2, 1, 1, 128, [300, 31]),                     # two rows: as many
    (3, 1, 1, 128, [300, 31]),                     # three: more
    (1, 1, 4, 64, [1100, 0, 65]),
    (5, 1, 1, 64, [1100, 0, 65]),
])
def test_row_blocks_match_the_oracle(hq, hkv, t, d, lens):
    rng = np.random.default_rng(81 + t)
    l_cap, bsz = max(lens), len(lens)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=1, seed=81)
    kmix = wl.round_to_bf16(rng.standard_normal((bsz, hkv, l_cap, d)).astype(np.float32))
    vmix = wl.round_to_bf16(rng.standard_normal((bsz, hkv, l_cap, d)).astype(np.float32))
    qd = wl.round_to_bf16(rng.standard_normal((bsz, t, hq, d)).astype(np.float32) * np.float32(0.5))
    dk, dv = vxl.to_device(kmix, "bf16"), vxl.to_device(vmix, "bf16")
    for b, n in enumerate(lens):                   # what lies past a length is never used
        dk[b, :, n:] = float("nan")
        dv[b, :, n:] = float("nan")
    dl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    got, lse = gpu_decode(w, qd, dk, dv, dl, want_lse=True)
    again, _ = gpu_decode(w, qd, dk, dv, dl, want_lse=True)
    assert np.array_equal(got, again)
    live = np.array(lens) > 0                      # (the oracle takes no empty set)
    want, wlse = oracle.decode_lse(qd[live], kmix[live], vmix[live], np.array(lens, np.int32)[live])
    assert_close(got[live], want, "bf16", head_axis=2, what=f"{hq * t // hkv} rows, d={d}")
    assert np.abs(lse[live] - wlse).max() < 2e-2
    assert not got[~live].any() and np.isneginf(lse[~live]).all()
    # no more partial results than one row per `rows` keys (what callers of the fixed scratch rely on)
    rows = hq // hkv * t
    bound = bsz * hkv * max(1, l_cap // rows) * rows * (d + 1) * 4 + 512
    assert vxl.workspace_bytes(vxl.OP_DECODE, None, desc_of(w), bsz, t, l_cap) <= bound


@pytest.mark.parametrize("mode", ["kept_in_place", "pooled"])
@pytest.mark.parametrize("hq,t,bsz,d", [(14, 6, 3, 128), (14, 11, 1, 64), (14, 23, 2, 128), (2, 1, 2, 128), (2, 3, 2, 128),
                                        (2, 4, 1, 64)])
def test_row_blocks_in_place(mode, hq, t, bsz, d):
    rng = np.random.default_rng(83 + t)
    w = wl.tiny_workload("bf16", hq, 2, d, T=t, B=bsz, k=3, seed=83, value_scale=0.5)
    lay = wl.random_layout(rng, 9, 12, 1, 300)
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    masks = (rng.random((bsz, 12)) < 0.4).astype(np.uint8)
    check_case(w, lay, k, v, wl.make_decode_queries(w), masks, mode)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("l_cap", [1, 129, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 12289, 32768])
def test_merge_of_every_number_of_splits(l_cap, d):
    """One row per KV head, a key split per 128 keys: one to 256 partial rows (the edges of the merge's batches of
    loads and of its choice of waves per row), some of them without keys."""
    rng = np.random.default_rng(l_cap)
    lens = [l_cap, max(1, l_cap // 3), 0] if l_cap < 20000 else [l_cap]
    w = wl.tiny_workload("bf16", 2 if l_cap < 20000 else 1, 2 if l_cap < 20000 else 1, d, T=1, B=len(lens), k=1, seed=82)
    shape = (len(lens), w.n_kv_heads, l_cap, d)
    kmix, vmix = (wl.round_to_bf16(rng.standard_normal(shape).astype(np.float32)) for _ in range(2))
    qd = wl.round_to_bf16(rng.standard_normal((len(lens), 1, w.n_q_heads, d)).astype(np.float32) * np.float32(0.5))
    got, lse = gpu_decode(w, qd, vxl.to_device(kmix, "bf16"), vxl.to_device(vmix, "bf16"),
                          torch.tensor(lens, dtype=torch.int32, device="cuda"), want_lse=True)
    live = np.array(lens) > 0
    want, wlse = oracle.decode_lse(qd[live], kmix[live], vmix[live], np.array(lens, np.int32)[live])
    assert_close(got[live], want, "bf16", head_axis=2, what=f"{l_cap} keys, d={d}")
    assert np.abs(lse[live] - wlse).max() < 2e-2
    assert not got[~live].any() and np.isneginf(lse[~live]).all()


@pytest.mark.parametrize("t,d,lens,l_cap", [
    (64, 128, [3000, 1, 63, 64, 65, 0], 3000),        # 448 rows, the ring: fewer tiles than splits, none, a ragged last one
    (64, 64, [700, 2500, 129], 9000),                 # lengths far below the capacity
    (100, 64, [15500, 4000], 15500),                  # 700 rows on four KV heads: more planned splits than one round holds
    (16, 128, [700, 650, 64] * 11, 800),              # 112 rows on 66 KV heads: the ring with four waves
])
def test_keys_dealt_out_by_length(t, d, lens, l_cap):
    rng = np.random.default_rng(t + l_cap)
    w = wl.tiny_workload("bf16", 14, 2, d, T=t, B=len(lens), k=1, seed=84)
    kmix, vmix = (wl.round_to_bf16(rng.standard_normal((len(lens), 2, l_cap, d)).astype(np.float32)) for _ in range(2))
    qd = wl.round_to_bf16(rng.standard_normal((len(lens), t, 14, d)).astype(np.float32) * np.float32(0.5))
    dk, dv = vxl.to_device(kmix, "bf16"), vxl.to_device(vmix, "bf16")
    for b, n in enumerate(lens):
        dk[b, :, n:] = float("nan")
        dv[b, :, n:] = float("nan")
    got, lse = gpu_decode(w, qd, dk, dv, torch.tensor(lens, dtype=torch.int32, device="cuda"), want_lse=True)
    live = np.array(lens) > 0
    want, wlse = oracle.decode_lse(qd[live], kmix[live], vmix[live], np.array(lens, np.int32)[live])
    assert_close(got[live], want, "bf16", head_axis=2, what=f"{7 * t} rows, d={d}")
    assert np.abs(lse[live] - wlse).max() < 2e-2
    assert not got[~live].any() and np.isneginf(lse[~live]).all()


@pytest.mark.parametrize("hq,hkv,t,d,lens", [
    (14, 2, 1, 128, [512, 1, 0, 129]),             # 7 rows: four tiles per wave
    (14, 2, 1, 128, [513, 481]),                   # one tile more: two splits and their merge
    (14, 2, 8, 128, [512, 33]),                    # 56 rows
    (28, 4, 36, 128, [31, 500, 0]),                # 252 rows, empty sets among them
    (8, 1, 8, 64, [384, 5]),                       # 64 rows, D = 64
    (8, 1, 9, 64, [768, 400]),                     # 72 rows
    (1, 1, 1, 64, [768]),                          # one row: fewer floats than threads
    (2, 2, 1, 128, [90, 0]),
    (14, 2, 40, 128, [300, 0, 64]),                # 280 rows
    (8, 1, 100, 128, [200, 0, 7, 64] * 16),        # 800 rows, one split: the ring
    (14, 2, 16, 64, [100, 0] * 17),                # 112 rows, one split: the ring with four waves
])
def test_calls_without_a_merge(hq, hkv, t, d, lens):
    """Mixed sets that one key split covers: the kernel writes O and LSE itself; O may be the buffer of the queries."""
    rng = np.random.default_rng(85 + t)
    l_cap, bsz = max(lens), len(lens)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=1, seed=85)
    kmix, vmix = (wl.round_to_bf16(rng.standard_normal((bsz, hkv, l_cap, d)).astype(np.float32)) for _ in range(2))
    qd = wl.round_to_bf16(rng.standard_normal((bsz, t, hq, d)).astype(np.float32) * np.float32(0.5))
    dk, dv = vxl.to_device(kmix, "bf16"), vxl.to_device(vmix, "bf16")
    for b, n in enumerate(lens):
        dk[b, :, n:] = float("nan")
        dv[b, :, n:] = float("nan")
    dl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    got, lse = gpu_decode(w, qd, dk, dv, dl, want_lse=True)
    live = np.array(lens) > 0
    want, wlse = oracle.decode_lse(qd[live], kmix[live], vmix[live], np.array(lens, np.int32)[live])
    assert_close(got[live], want, "bf16", head_axis=2, what=f"{hq * t // hkv} rows, d={d}")
    assert np.abs(lse[live] - wlse).max() < 2e-2
    assert not got[~live].any() and np.isneginf(lse[~live]).all()
    desc, q = desc_of(w), vxl.to_device(qd, "bf16")
    vxl.bilevel_decode(desc, q, dk, dv, dl, q, None, vxl.alloc_workspace(
        vxl.workspace_bytes(vxl.OP_DECODE, None, desc, bsz, t, l_cap)))
    assert np.array_equal(vxl.to_host(q), got)


def _rounded_tiles(qd, kmix, vmix, n, tile=32):
    """[B, T, Hq, D] attention over the first n rows as one tile of 32 keys per wave computes it: weights relative to the
    tile's own largest logit, rounded to bf16, everything else in float64."""
    b, t, hq, d = qd.shape
    g = hq // kmix.shape[1]
    out = np.empty(qd.shape)
    for i in range(b):
        for h in range(hq):
            x = qd[i, :, h].astype(np.float64) @ kmix[i, h // g, :n].astype(np.float64).T / d ** 0.5
            top, num, den = x.max(axis=1, keepdims=True), 0.0, 0.0
            for lo in range(0, n, tile):
                own = x[:, lo:lo + tile].max(axis=1, keepdims=True)
                p = wl.round_to_bf16(np.exp(x[:, lo:lo + tile] - own).astype(np.float32)).astype(np.float64)
                num = num + np.exp(own - top) * (p @ vmix[i, h // g, lo:min(lo + tile, n)].astype(np.float64))
                den = den + np.exp(own - top) * p.sum(axis=1, keepdims=True)
            out[i, :, h] = num / den
    return out


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("hq,hkv,t,bsz,d,n", [
    (28, 4, 1, 2, 128, 384), (28, 4, 8, 1, 128, 251), (7, 1, 16, 2, 128, 380), (2, 2, 1, 4, 128, 501),
    (14, 2, 1, 3, 64, 500), (14, 2, 20, 1, 64, 511), (4, 4, 3, 2, 64, 767), (8, 1, 8, 2, 64, 384)])
def test_one_workgroup_is_as_precise_as_a_tile_per_wave(hq, hkv, t, bsz, d, n, in_place):
    """Short sets that one workgroup walks, several tiles per wave: every tile's weights are rounded against the tile's
    own maximum.  Rounded alike, two results differ by fp32 sums, which move an output to its neighbour in bf16 (2^-8)
    in fewer than one of 2^8 elements: 2.5e-4 relative at most.  Rounded against another reference the weights differ by
    up to 2^-8 each, the results by 1e-3 and more."""
    rng = np.random.default_rng(n + hq)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=1, seed=n, value_scale=1.0)
    qd = wl.round_to_bf16(rng.standard_normal((bsz, t, hq, d)).astype(np.float32))
    k, v = (wl.round_to_bf16(rng.standard_normal((bsz, hkv, n, d)).astype(np.float32)) for _ in range(2))
    if in_place:                                                   # (all queries read the same rows)
        lay = wl.layout_from_lists(0, [n], [np.zeros(0, np.int32)])
        k[:], v[:] = k[:1], v[:1]
        got = gpu_decode_inplace(w, lay, qd, vxl.to_device(k[0], "bf16"), vxl.to_device(v[0], "bf16"),
                                 np.ones((bsz, 1), np.uint8), n)[0]
    else:
        got = gpu_decode(w, qd, vxl.to_device(k, "bf16"), vxl.to_device(v, "bf16"),
                         torch.full((bsz,), n, dtype=torch.int32, device="cuda"))
    want = wl.round_to_bf16(_rounded_tiles(qd, k, v, n).astype(np.float32)).astype(np.float64)
    assert np.linalg.norm(got - want) <= 2.5e-4 * np.linalg.norm(want)


@pytest.mark.parametrize("hq,hkv,d,bsz,t,l_cap,n,scale", [
    (28, 4, 128, 2, 32, 35410, 25500, 1.0), (28, 4, 128, 2, 32, 8000, 5000, 1.0), (14, 2, 64, 2, 95, 9000, 7000, 1.0),     # the ring
    (28, 4, 128, 8, 32, 9000, 6000, 0.0884), (28, 4, 128, 8, 16, 2000, 1500, 1.0), (28, 4, 128, 4, 1, 6000, 4000, 1.0),
    (28, 4, 128, 4, 8, 251, 251, 1.0), (14, 2, 64, 4, 20, 761, 700, 1.0), (28, 4, 128, 8, 1, 512, 501, 1.0)])
def test_decode_error_is_that_of_two_roundings(hq, hkv, d, bsz, t, l_cap, n, scale):
    """Wherever the keys are cut: the weights and the result are rounded to bf16 once.  Half a unit is 2^-8 of a value at
    most, 2^-8 * 0.42 of it in root mean square over mantissas that are uniform in their logarithm; the rows add the
    weights' roundings up as they do the weights.  sqrt(2) * 0.42 * 2^-8 = 2.35e-3, and 2 % for the sample."""
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=1, seed=1)
    desc, g, num, den = desc_of(w), hq // hkv, 0.0, 0.0
    gen = torch.Generator(device="cuda").manual_seed(l_cap)
    q, k, v = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, scale, generator=gen)
               for s in ((bsz, t, hq, d), (bsz, hkv, l_cap, d), (bsz, hkv, l_cap, d)))
    out = torch.empty_like(q)
    vxl.bilevel_decode(desc, q, k, v, torch.full((bsz,), n, dtype=torch.int32, device="cuda"), out, None,
                       vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_DECODE, None, desc, bsz, t, l_cap)))
    for b in range(bsz):
        for h in range(hkv):
            s = q[b, :, h * g:(h + 1) * g].reshape(-1, d).double() @ k[b, h, :n].double().T / d ** 0.5
            want = torch.softmax(s, -1) @ v[b, h, :n].double()
            num += (out[b, :, h * g:(h + 1) * g].reshape(-1, d).double() - want).pow(2).sum().item()
            den += want.pow(2).sum().item()
    assert (num / den) ** 0.5 <= 2.4e-3
