"""The choice between the decode kernels, which is made on the host and needs no GPU: where 32-row blocks take the place
of the ring kernel, they are the shorter call by the times of a tile, a round of workgroups on the busiest XCD, and a
call."""
import numpy as np
import pytest

from paper_2506_19225_amd import vxl

RING, BLOCKS = 1, 2


def plan(hq, hkv, d, b, t, l_cap, in_place=False):
    return vxl.debug_decode_plan(vxl.make_desc(hq, hkv, d, "bf16"), b, t, l_cap, in_place)


def ring_splits(units, rows, l_cap):
    """Key splits of the ring kernel: as many as give each of 256 compute units a workgroup, no more partial rows than keys."""
    tiles, want = -(-l_cap // 64), -(-256 // (units * -(-rows // 256)))
    per = -(-tiles // max(1, min(want, l_cap // rows, tiles)))
    return -(-tiles // per)


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_row_blocks_are_the_shorter_call(d, in_place):
    chosen = 0
    for g, hkv in [(8, 1), (7, 1), (7, 2), (7, 4), (16, 1), (1, 8)]:
        for b in (1, 2, 3, 5, 9, 12):
            for t in (37, 64, 92, 128, 129, 160, 256, 512, 2000):
                rows, units = g * t, hkv * b
                if rows <= 256:                    # (fewer rows: the ring of 128 rows may be the other choice)
                    continue
                for l_cap in (300, 1000, 1300, 1800, 4096, 16384, 45000):
                    kernel, n_split = plan(g * hkv, hkv, d, b, t, l_cap, in_place)
                    n_ring = ring_splits(units, rows, l_cap)
                    if kernel == RING:
                        assert n_split == n_ring
                        continue
                    assert kernel == BLOCKS
                    chosen += 1
                    blocks = -(-rows // 32)
                    per_xcd = np.bincount(np.arange(units * n_split) % 8).max() * blocks
                    lds = 1024 * d + 1024 + (16384 if in_place else 0)            # (tiles, statistics, row map)
                    rounds = -(-per_xcd // (32 * (163840 // lds)))
                    tiles, ring_tiles = -(-l_cap // (128 * n_split)), -(-l_cap // (64 * n_ring))
                    assert rounds * (8 + 0.8 * tiles) < 14 + ring_tiles, (g, hkv, b, t, l_cap, n_split)
                    assert n_split <= n_ring and units * n_split * blocks <= 256
    assert chosen > 50


@pytest.mark.parametrize("hq,hkv,d,b,t,l_cap,kernel", [
    (8, 1, 128, 1, 128, 4096, BLOCKS), (8, 1, 128, 1, 160, 4096, RING), (8, 1, 128, 1, 160, 16384, RING),
    (8, 1, 64, 1, 160, 4096, BLOCKS), (8, 1, 64, 1, 160, 16384, RING), (8, 1, 128, 1, 512, 4096, RING),
    (28, 4, 128, 3, 96, 1300, BLOCKS), (28, 4, 128, 3, 96, 2000, RING), (28, 4, 64, 3, 96, 2000, BLOCKS),
    (7, 1, 128, 9, 128, 1300, BLOCKS), (28, 4, 128, 1, 160, 4096, RING), (28, 4, 128, 1, 32, 4352, BLOCKS),
    (8, 1, 128, 1, 353, 148, RING), (14, 2, 128, 1, 137, 1171, BLOCKS), (8, 1, 128, 1, 266, 640, RING)])
def test_measured_sides_of_the_line(hq, hkv, d, b, t, l_cap, kernel):
    """Shapes on either side whose two kernels were timed against each other."""
    assert plan(hq, hkv, d, b, t, l_cap)[0] == kernel


@pytest.mark.parametrize("hq,hkv,d,b,t,l_cap,kernel", [
    (7, 1, 64, 3, 154, 6680, RING), (8, 1, 128, 1, 272, 583, RING), (8, 1, 128, 1, 341, 1985, RING),
    (14, 2, 128, 1, 138, 2486, BLOCKS), (7, 1, 64, 1, 95, 2297, BLOCKS)])
def test_measured_sides_of_the_line_in_place(hq, hkv, d, b, t, l_cap, kernel):
    assert plan(hq, hkv, d, b, t, l_cap, True)[0] == kernel


@pytest.mark.parametrize("hq,hkv,d,b,t,l_cap,in_place,waves", [
    (28, 4, 64, 8, 188, 1094, True, 8), (32, 8, 64, 3, 340, 35009, True, 8), (16, 16, 64, 8, 395, 1411, True, 8),
    (16, 16, 64, 2, 1237, 1097, True, 8), (16, 16, 64, 3, 1126, 2986, True, 8), (4, 4, 64, 8, 545, 1674, True, 4),
    (16, 8, 64, 8, 178, 2042, True, 4), (16, 16, 128, 3, 722, 272, True, 8), (16, 16, 64, 3, 1233, 856, False, 8), (16, 8, 64, 8, 350, 967, False, 8),
    (28, 4, 64, 8, 198, 42803, False, 8), (28, 4, 128, 1, 64, 10368, False, 4), (28, 4, 128, 8, 43, 23830, False, 8)])
def test_measured_waves_of_the_ring(hq, hkv, d, b, t, l_cap, in_place, waves):
    """Shapes that were timed with workgroups of four and of eight waves: the faster by 2 to 38 %."""
    desc = vxl.make_desc(hq, hkv, d, "bf16")
    assert plan(hq, hkv, d, b, t, l_cap, in_place)[0] == RING
    assert vxl.debug_decode_ring_waves(desc, b, t, l_cap, in_place) == waves


def test_which_gathers_read_a_row_once():
    """Both sides of every line of the rule."""
    def shared(b=8, l_cap=16384, n=8000, chunks=100, hkv=4, d=128, dtype="bf16"):
        return vxl.debug_gather_shared(vxl.make_desc(hkv, hkv, d, dtype), n, 400, chunks, b, l_cap)

    assert shared() and shared(b=2) and not shared(b=1)
    assert shared(b=16, chunks=64) and not shared(b=16, chunks=65)
    assert shared(b=17, n=9766, chunks=10) and not shared(b=17, n=9765, chunks=10)      # 20 MB of K and V
    assert shared(b=32, n=9766, chunks=32) and not shared(b=33, n=9766, chunks=10)
    assert shared(chunks=128) and not shared(chunks=129)
    assert shared(n=65536) and not shared(n=65537)
    assert shared(l_cap=2747, n=1000) and not shared(l_cap=2746, n=1000)           # 45 MB
    assert shared(b=16, l_cap=2048, n=1000, hkv=16, chunks=9) and not shared(b=16, l_cap=2047, n=1000, hkv=16, chunks=9)
    assert shared(b=16, l_cap=4096, n=1000, hkv=16, d=64, chunks=9) and not shared(b=16, l_cap=4095, n=1000, hkv=16, d=64, chunks=9)
    assert shared(hkv=7, d=64, l_cap=6280, n=1000) and shared(dtype="f32", l_cap=1374, n=1000)
