"""The instances that read past the caches, just above the sizes from which they are taken (32 MB of keys or mixed rows, 96
MB for mean keys, 256 MB for pooling): against float64 on the device from the same stored values."""
import numpy as np
import pytest
import torch

from paper_2506_19225_amd import vxl, workloads as wl

from gpu_util import DECODE_BLOCKS, DECODE_RING, assert_close, decode_kernel, desc_of

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def randn(seed, shape, dtype):
    return torch.empty(shape, dtype=DT[dtype], device="cuda").normal_(0, 1, generator=torch.Generator(device="cuda").manual_seed(seed))


def ragged_layout(n_tokens, mean, kept=1):
    """A prefix of 5 tokens and chunks of about `mean`, every one of another length, whose first `kept` rows are kept."""
    lens = [mean + (i * 37) % 61 - 30 for i in range((n_tokens - 5) // mean)]
    lens[-1] += n_tokens - 5 - sum(lens)
    bounds = np.concatenate([[5], 5 + np.cumsum(lens)]).astype(np.int32)
    soff = (kept * np.arange(len(lens) + 1)).astype(np.int32)
    sidx = (bounds[:-1, None] + np.arange(kept)).reshape(-1).astype(np.int32)
    return bounds, vxl.Layout(5, bounds, soff, sidx)


@pytest.mark.parametrize("d,hq,hkv,t,bsz", [(128, 7, 1, 1, 1), (128, 7, 1, 18, 1), (128, 14, 2, 1, 8), (64, 4, 1, 1, 2), (64, 8, 2, 16, 2)])
def test_mass_past_the_caches(d, hq, hkv, t, bsz):
    """One row tile of all stacked rows; chunks of several full tiles and a ragged tail.  fp32 sums of up to 263,000 terms:
    the tolerance of the score, 1e-4 of the largest, as in the other tests of it."""
    n = (32 << 20) // (2 * hkv * d) + 77
    bounds, gl = ragged_layout(n, 700)
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=3, seed=d)
    k, qd = randn(1, (hkv, n, d), "bf16"), randn(2, (bsz, t, hq, d), "bf16")
    c = len(bounds) - 1
    idx, mask = torch.zeros((bsz, 3), dtype=torch.int32, device="cuda"), torch.zeros((bsz, c), dtype=torch.uint8, device="cuda")
    scores = torch.full((bsz, c), float("nan"), device="cuda")
    vxl.chunk_score_topk_mass(gl, desc_of(w), qd, k, 3, idx, mask, scores, workspace=vxl.alloc_workspace(
        vxl.workspace_bytes(vxl.OP_SCORE_MASS, gl, desc_of(w), bsz, t)))
    want = torch.zeros((bsz, c), dtype=torch.float64, device="cuda")
    g, ends = hq // hkv, torch.from_numpy(bounds.astype(np.int64)).cuda()
    for h in range(hkv):
        for b in range(bsz):
            p = torch.softmax(qd[b, :, h * g:(h + 1) * g].reshape(-1, d).double() @ k[h].double().T / d ** 0.5, -1).sum(0)
            total = torch.cat([torch.zeros(1, dtype=torch.float64, device="cuda"), torch.cumsum(p, 0)])
            want[b] += (total[ends[1:]] - total[ends[:-1]]) / (t * hq)
    assert (scores.double() - want).abs().max().item() <= 1e-4 * want.max().item()
    assert torch.equal(torch.argsort(scores, dim=1, descending=True, stable=True)[:, :3].int(), idx)


@pytest.mark.parametrize("d,hq,hkv,t,bsz,kernel", [
    (64, 4, 4, 1, 3, DECODE_BLOCKS), (64, 8, 4, 2, 2, DECODE_BLOCKS), (64, 28, 4, 1, 2, DECODE_BLOCKS),   # 1, 4 and 7 rows
    (128, 2, 2, 1, 2, DECODE_BLOCKS), (128, 4, 2, 1, 3, DECODE_BLOCKS), (128, 14, 2, 4, 1, DECODE_BLOCKS),
    (64, 28, 4, 32, 4, DECODE_RING), (128, 28, 4, 32, 4, DECODE_RING)])
def test_decode_past_the_caches(d, hq, hkv, t, bsz, kernel):
    l_cap = (32 << 20) // (4 * bsz * hkv * d) + 33
    w = wl.tiny_workload("bf16", hq, hkv, d, T=t, B=bsz, k=1, seed=d)
    assert decode_kernel(w, bsz, t, l_cap) == kernel
    k, v, qd = randn(3, (bsz, hkv, l_cap, d), "bf16"), randn(4, (bsz, hkv, l_cap, d), "bf16"), randn(5, (bsz, t, hq, d), "bf16")
    lens = [l_cap, l_cap // 3 + 1, 1, 0][:bsz] if bsz > 1 else [l_cap - 5]
    for b, n in enumerate(lens):
        k[b, :, n:], v[b, :, n:] = float("nan"), float("nan")
    out, lse = torch.full_like(qd, float("nan")), torch.full((bsz, t, hq), float("nan"), device="cuda")
    vxl.bilevel_decode(desc_of(w), qd, k, v, torch.tensor(lens, dtype=torch.int32, device="cuda"), out, lse,
                       vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_DECODE, None, desc_of(w), bsz, t, l_cap)))
    g = hq // hkv
    for b, n in enumerate(lens):
        if n == 0:
            assert not out[b].any() and torch.isneginf(lse[b]).all()
            continue
        want = torch.empty((t, hq, d), dtype=torch.float64, device="cuda")
        wlse = torch.empty((t, hq), dtype=torch.float64, device="cuda")
        for h in range(hkv):
            s = qd[b, :, h * g:(h + 1) * g].reshape(-1, d).double() @ k[b, h, :n].double().T / d ** 0.5
            want[:, h * g:(h + 1) * g] = (torch.softmax(s, -1) @ v[b, h, :n].double()).reshape(t, g, d)
            wlse[:, h * g:(h + 1) * g] = torch.logsumexp(s, -1).reshape(t, g)
        assert_close(vxl.to_host(out[b]), want.cpu().numpy(), "bf16", head_axis=1, what=f"{n} of {l_cap} rows")
        assert (lse[b].double() - wlse).abs().max().item() < 2e-2


@pytest.mark.parametrize("dtype,hkv,d,mean", [("bf16", 4, 128, 1000), ("bf16", 4, 128, 250), ("bf16", 2, 64, 900), ("f32", 4, 64, 1500),
                                              ("f32", 2, 128, 300)])
def test_mean_keys_past_the_caches(dtype, hkv, d, mean):
    """256 and 512 threads per chunk.  A mean of up to 1,600 values: fp32 sums in parts of at most 32 and a tree of
    six levels, below 2^-19 of the values' deviation."""
    n = (96 << 20) // (hkv * d * (2 if dtype == "bf16" else 4)) + 77
    bounds, gl = ragged_layout(n, mean)
    w = wl.tiny_workload(dtype, hkv, hkv, d, T=2, B=1, k=1, seed=d)
    k, qd, c = randn(6, (hkv, n, d), dtype), randn(7, (1, 2, hkv, d), dtype), len(bounds) - 1
    idx, mask = torch.zeros((1, 1), dtype=torch.int32, device="cuda"), torch.zeros((1, c), dtype=torch.uint8, device="cuda")
    scores, kbar = torch.zeros((1, c), device="cuda"), torch.full((hkv, c, d), float("nan"), device="cuda")
    vxl.chunk_score_topk(gl, desc_of(w), qd, k, 1, idx, mask, scores, kbar,
                         workspace=vxl.alloc_workspace(vxl.workspace_bytes(vxl.OP_SCORE_TOPK, gl, desc_of(w), 1)))
    for i in range(c):
        want = k[:, bounds[i]:bounds[i + 1]].double().mean(1)
        assert (kbar[:, i].double() - want).abs().max().item() <= 2.0 ** -19, i


@pytest.mark.parametrize("dtype,hkv,d", [("bf16", 4, 64), ("bf16", 2, 128), ("f32", 2, 64), ("f32", 4, 128)])
def test_pooling_past_the_caches(dtype, hkv, d):
    """Groups of 1 to 700 rows.  fp32 sums in row order, rounded once: 700 roundings of 2^-24 of a sum of some 26
    deviations over 700 of them are below 2^-17, to which bf16 adds half a unit (2^-8 of the value)."""
    n = (256 << 20) // (2 * hkv * d * (2 if dtype == "bf16" else 4)) + 77
    bounds, gl = ragged_layout(n, 700, kept=3)
    w = wl.tiny_workload(dtype, hkv, hkv, d, T=1, B=1, k=1, seed=d)
    k, v, c = randn(8, (hkv, n, d), dtype), randn(9, (hkv, n, d), dtype), len(bounds) - 1
    ksp = torch.full((hkv, 3 * c, d), float("nan"), dtype=DT[dtype], device="cuda")
    vsp = torch.full_like(ksp, float("nan"))
    vxl.pool_sparse_kv(gl, desc_of(w), k, v, ksp, vsp)
    for i in range(0, c, 7):
        for m in range(3):
            lo, hi = (int(bounds[i] + x * (bounds[i + 1] - bounds[i]) // 3) for x in (m, m + 1))
            for got, x in ((ksp, k), (vsp, v)):
                want = x[:, lo:hi].double().mean(1)
                err = (got[:, 3 * i + m].double() - want).abs()
                assert (err <= 2.0 ** -17 + (want.abs() * 2.0 ** -8 if dtype == "bf16" else 0)).all(), (i, m)
