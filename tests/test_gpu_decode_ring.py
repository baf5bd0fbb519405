"""The ring decode with eight and with four waves per workgroup, gathered and in place, against the oracle: rows at the
edges of a wave's and a workgroup's rows, sets of few and of no keys, more splits than tiles, one split, both head
dimensions."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import DECODE_128, DECODE_RING, assert_close, decode_kernel, desc_of, gpu_decode, make_layout
from test_gpu_inplace import check_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,t,d,waves,lens,l_cap", [
    (28, 4, 43, 128, 4, [5300, 0], 5300),                  # 301 rows: a last workgroup of 45, two waves without rows
    (14, 2, 55, 128, 4, [9000, 130, 1], 9000),             # 385 rows: one in the last workgroup
    (8, 1, 160, 128, 4, [5000, 4937, 63], 5000),           # 1,280: whole workgroups
    (8, 1, 33, 64, 4, [9000, 64, 65], 9000),               # 264 rows, D = 64
    (14, 2, 77, 64, 4, [3000, 2999, 1, 0], 3000),          # 539
    (7, 1, 257, 128, 4, [70, 64, 1, 0] * 8, 70),           # 1,799 rows, one split
    (28, 4, 36, 128, 8, [8000, 7937] * 4, 8000),           # 252 rows of eight queries: longer walks
    (14, 2, 129, 64, 8, [30000, 29937], 30000),
    (28, 4, 5, 128, 4, [1500, 0, 64, 65] * 9, 1500),       # 35 rows: two waves without any
    (28, 4, 18, 64, 4, [777, 1, 63] * 9, 777),             # 126 rows
    (14, 2, 19, 128, 4, [200, 129] * 17, 200)])            # 133 rows in two workgroups, one split
def test_either_number_of_waves(hq, hkv, t, d, waves, lens, l_cap):
    rng = np.random.default_rng(t + l_cap)
    bsz = len(lens)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=1, seed=86)
    kernel = decode_kernel(w, bsz, t, l_cap)
    assert kernel in (DECODE_128, DECODE_RING)
    assert (4 if kernel == DECODE_128 else vxl.debug_decode_ring_waves(desc_of(w), bsz, t, l_cap)) == waves
    k, v = (torch.empty((bsz, hkv, l_cap, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1) for _ in range(2))
    qd = wl.round_to_bf16(rng.standard_normal((bsz, t, hq, d)).astype(np.float32) * np.float32(0.5))
    for b, n in enumerate(lens):                           # what lies past a length is never used
        k[b, :, n:] = float("nan")
        v[b, :, n:] = float("nan")
    dl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    got, lse = gpu_decode(w, qd, k, v, dl, want_lse=True)
    again, _ = gpu_decode(w, qd, k, v, dl, want_lse=True)
    assert np.array_equal(got, again)
    live = np.array(lens) > 0
    q = torch.from_numpy(qd).cuda().double()
    g = hq // hkv
    for b in np.flatnonzero(live):
        for h in range(hkv):
            s = q[b, :, h * g:(h + 1) * g].reshape(-1, d) @ k[b, h, :lens[b]].double().T / d ** 0.5
            want = (torch.softmax(s, -1) @ v[b, h, :lens[b]].double()).reshape(t, g, d).cpu().numpy()
            assert_close(got[b, :, h * g:(h + 1) * g], want, "bf16", head_axis=1, what=f"query {b}, {lens[b]} keys")
            wlse = torch.logsumexp(s, -1).reshape(t, g).cpu().numpy()
            assert np.abs(lse[b, :, h * g:(h + 1) * g] - wlse).max() < 2e-2
    assert not got[~live].any() and np.isneginf(lse[~live]).all()


@pytest.mark.parametrize("mode", ["kept_in_place", "pooled"])
@pytest.mark.parametrize("hq,t,d,waves,chunks,length", [
    (14, 150, 128, 4, 15, 800), (14, 300, 64, 4, 20, 800), (14, 55, 128, 8, 90, 900), (14, 55, 64, 8, 90, 900)])
def test_either_number_of_waves_in_place(mode, hq, t, d, waves, chunks, length):
    rng = np.random.default_rng(87 + t)
    w = wl.tiny_workload("bf16", hq, 2, d, T=t, B=1, k=3, seed=87, value_scale=0.5)
    lay = wl.random_layout(rng, 9, chunks, max(1, length // 2), length)
    masks = np.ones((1, chunks), np.uint8)
    masks[0, rng.choice(chunks, chunks // 4, replace=False)] = 0
    desc = desc_of(w)
    lengths = np.where(masks[0], np.diff(lay.chunk_bounds), np.diff(lay.sparse_offsets))
    l_cap = int(lay.n_prefix + lengths.sum())
    assert decode_kernel(w, 1, t, l_cap, True) == DECODE_RING
    assert vxl.debug_decode_ring_waves(desc, 1, t, l_cap, True) == waves
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    check_case(w, lay, k, v, wl.make_decode_queries(w), masks, mode, l_cap=l_cap)


@pytest.mark.parametrize("hq,hkv,t,d,bsz,l_cap,blocks", [
    (28, 4, 10, 128, 8, 5200, 2),                          # 70 rows, 21 tiles per wave of row blocks in two splits
    (16, 1, 6, 64, 8, 38000, 10)])                         # 96 rows, 30 tiles in ten splits
def test_long_walks_and_the_scratch_that_row_blocks_take(hq, hkv, t, d, bsz, l_cap, blocks):
    """The ring, whose splits need more scratch memory, and with as much as row blocks need those: both against float64; a
    byte less is refused."""
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=1, seed=88)
    desc, g, rows = desc_of(w), hq // hkv, hq // hkv * t
    kernel, n_split = vxl.debug_decode_plan(desc, bsz, t, l_cap)
    assert kernel == DECODE_128 and n_split > blocks
    gen = torch.Generator(device="cuda").manual_seed(l_cap)
    q, k, v = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=gen)
               for s in ((bsz, t, hq, d), (bsz, hkv, l_cap, d), (bsz, hkv, l_cap, d)))
    lens = torch.tensor([l_cap, l_cap - 1, 65, 64, 1, l_cap // 2, 0, l_cap - 64], dtype=torch.int32)
    for b, n in enumerate(lens.tolist()):
        k[b, :, n:] = float("nan")
        v[b, :, n:] = float("nan")
    dl = lens.cuda()
    small = sum((bsz * hkv * blocks * rows * n * 4 + 255) // 256 * 256 for n in (d, 1))
    full = vxl.workspace_bytes(vxl.OP_DECODE, None, desc, bsz, t, l_cap)
    assert small < full
    with pytest.raises(vxl.VxlError):
        vxl.bilevel_decode(desc, q, k, v, dl, torch.empty_like(q), None,
                           torch.empty(small - 1, dtype=torch.uint8, device="cuda"))
    for size in (full, small):
        out, lse = torch.full_like(q, float("nan")), torch.full((bsz, t, hq), float("nan"), device="cuda")
        vxl.bilevel_decode(desc, q, k, v, dl, out, lse, torch.empty(size, dtype=torch.uint8, device="cuda"))
        for b, n in enumerate(lens.tolist()):
            if n == 0:
                assert not out[b].any() and torch.isneginf(lse[b]).all()
                continue
            for h in range(hkv):
                s = q[b, :, h * g:(h + 1) * g].reshape(-1, d).double() @ k[b, h, :n].double().T / d ** 0.5
                want = (torch.softmax(s, -1) @ v[b, h, :n].double()).reshape(t, g, d).cpu().numpy()
                got = vxl.to_host(out[b, :, h * g:(h + 1) * g].contiguous())
                assert_close(got, want, "bf16", head_axis=1, what=f"query {b}, {n} keys, {size} bytes")
                wlse = torch.logsumexp(s, -1).reshape(t, g)
                assert (lse[b, :, h * g:(h + 1) * g].double() - wlse).abs().max() < 2e-2


@pytest.mark.parametrize("pooled", [False, True])
def test_long_walks_in_place_and_the_scratch_that_row_blocks_take(pooled):
    """The same in place, where the row map comes before the partial rows: 70 rows of eight queries, 21 tiles per wave of row
    blocks in two splits, by the ring, by row blocks (the bytes that those need) and refused (one byte less)."""
    hq, hkv, t, d, bsz, l_cap, blocks = 28, 4, 10, 128, 8, 5200, 2
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=1, seed=89, value_scale=0.5)
    rng, g, rows = np.random.default_rng(89), hq // hkv, hq // hkv * t
    lens = [330] * 20
    lay = wl.layout_from_lists(9, lens, [np.sort(rng.choice(330, 40, replace=False)).astype(np.int32) + 9 + 330 * c
                                         for c in range(20)])
    masks = np.zeros((bsz, 20), np.uint8)
    for b, n in enumerate((15, 14, 15, 0, 1, 15, 20, 7)):     # (20 dense chunks do not fit)
        masks[b, rng.choice(20, n, replace=False)] = 1
    desc, gl = desc_of(w), make_layout(lay)
    kernel, n_split = vxl.debug_decode_plan(desc, bsz, t, l_cap, True)
    assert kernel == DECODE_128 and n_split > blocks
    _, k, v = wl.make_qkv(w, lay, with_q=False)
    dk, dv, qd = vxl.to_device(k, "bf16"), vxl.to_device(v, "bf16"), vxl.to_device(wl.make_decode_queries(w), "bf16")
    dm, sp = torch.from_numpy(masks).cuda(), (None, None)
    kmix = torch.zeros((bsz, hkv, l_cap, d), dtype=torch.bfloat16, device="cuda")
    vmix, need = torch.zeros_like(kmix), torch.zeros(bsz, dtype=torch.int32, device="cuda")
    if pooled:
        sp = tuple(torch.empty((hkv, 800, d), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        vxl.pool_sparse_kv(gl, desc, dk, dv, *sp)
        vxl.gather_bilevel_kv_pooled(gl, desc, dk, dv, *sp, dm, kmix, vmix, need)
    else:
        vxl.gather_bilevel_kv(gl, desc, dk, dv, dm, kmix, vmix, need)

    def partials(n):
        return sum((bsz * hkv * n * rows * x * 4 + 255) // 256 * 256 for x in (d, 1))

    full = vxl.workspace_bytes(vxl.OP_DECODE_INPLACE, gl, desc, bsz, t, l_cap)
    small = full - partials(n_split) + partials(blocks)
    with pytest.raises(vxl.VxlError):
        vxl.bilevel_decode_inplace(gl, desc, qd, dk, dv, *sp, dm, l_cap, torch.empty_like(qd), None, None,
                                   torch.empty(small - 1, dtype=torch.uint8, device="cuda"))
    for size in (full, small):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        for map_ready in (False, True):
            out, lse = torch.full_like(qd, float("nan")), torch.full((bsz, t, hq), float("nan"), device="cuda")
            vxl.bilevel_decode_inplace(gl, desc, qd, dk, dv, *sp, dm, l_cap, out, lse, None, ws, map_ready)
            for b, n in enumerate(need.tolist()):
                if n <= 0:
                    assert not out[b].any() and torch.isneginf(lse[b]).all()
                    continue
                for h in range(hkv):
                    s = qd[b, :, h * g:(h + 1) * g].reshape(-1, d).double() @ kmix[b, h, :n].double().T / d ** 0.5
                    want = (torch.softmax(s, -1) @ vmix[b, h, :n].double()).reshape(t, g, d).cpu().numpy()
                    got = vxl.to_host(out[b, :, h * g:(h + 1) * g].contiguous())
                    assert_close(got, want, "bf16", head_axis=1, what=f"query {b}, {n} keys, {size} bytes")
                    wlse = torch.logsumexp(s, -1).reshape(t, g)
                    assert (lse[b, :, h * g:(h + 1) * g].double() - wlse).abs().max() < 2e-2
