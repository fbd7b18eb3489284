"""CPU emulation of the bf16 expert FFN's narrow tiles (narrow_gemm of
expert_ffn.hip): tile order, load addresses, the stage ring and the output
columns, replayed in numpy where a slip would fault the GPU."""
import numpy as np
import pytest

from tests import test_ffn_tiling_emulation as E

NB_N = 128


def ring(bm):
    stage = (bm + NB_N) * E.ROW_B
    return stage, E.STAGES * E.STAGE_BYTES // stage


def schedule(counts, max_rows, bm):
    offs = np.concatenate([[0], np.cumsum(counts)])
    b = np.clip(offs[:-1], 0, max_rows)
    e = np.maximum(b, np.clip(offs[1:], 0, max_rows))
    return b, e, np.concatenate([[0], np.cumsum((e - b + bm - 1) // bm)])


def decode(t, pref, b, e, n_tiles, bm):
    l = int(np.flatnonzero(pref[:-1] <= t // n_tiles)[-1])
    # the kernel's binary search returns the last expert whose prefix is <= the m-tile
    while pref[l + 1] == pref[l]:
        l -= 1
    cnt = int(pref[l + 1] - pref[l])
    u = t - int(pref[l]) * n_tiles
    nt, j = u // cnt, u % cnt
    row0 = int(b[l]) + j * bm
    return l, row0, min(bm, int(e[l]) - row0), nt


def find_expert(pref, m):
    lo, hi = 0, len(pref) - 2
    while lo < hi:
        mid = (lo + hi + 1) >> 1
        if pref[mid] <= m:
            lo = mid
        else:
            hi = mid - 1
    return lo


@pytest.mark.parametrize("counts,max_rows,d,inter", [
    ([24, 22, 0, 18, 66, 44, 34, 29], 8192, 1024, 256), ([1], 1, 256, 128), ([0, 0, 3], 3, 256, 128),
    ([63, 64, 65, 128, 129, 1000], 1400, 512, 384), ([2] * 40 + [0] * 30, 75, 256, 128)])
@pytest.mark.parametrize("gu", [True, False])
@pytest.mark.parametrize("bm", [64, 128])
def test_narrow_tiles_in_bounds(counts, max_rows, d, inter, gu, bm):
    b, e, pref = schedule(counts, max_rows, bm)
    stage, depth = ring(bm)
    K, N_out = (d, inter) if gu else (inter, d)
    n_tiles = N_out // (NB_N // 2) if gu else N_out // NB_N
    total = int(pref[-1]) * n_tiles
    pitch, lane = K * 2, np.arange(64)
    seen = set()
    for t in range(total):
        l = find_expert(pref, t // n_tiles)
        assert pref[l] <= t // n_tiles < pref[l + 1]
        l2, row0, rows, nt = decode(t, pref, b, e, n_tiles, bm)
        assert l2 == l and 1 <= rows <= bm and 0 <= nt < n_tiles and row0 + rows <= min(max_rows, e[l])
        assert (l, row0, nt) not in seen
        seen.add((l, row0, nt))
        covered = {}
        for w in range(8):
            for j in range(bm // 64):
                r = np.minimum(64 * j + 8 * w + E.LD_ROW, rows - 1)
                off = r * pitch + E.COL_B[w & 1] + (K // 64 - 1) * 128
                assert off.max() + 16 <= rows * pitch
                assert (8 * j + w) % 2 == w & 1 and 64 * E.ROW_B * j + w * 1024 + 1024 <= bm * E.ROW_B
            first = (l * N_out + nt * (NB_N // 2) + (w >> 1) * 16) if gu else (l * N_out + nt * NB_N + w * 16)
            for i in range(2):
                assert 0 <= first + 8 * i and first + 8 * i + 8 <= (l + 1) * N_out
                lds = bm * E.ROW_B + w * 2048 + i * 1024
                assert ((lds // E.ROW_B) // 8) % 2 == i           # swizzle parity of the 8-row block
                assert lds + 1024 <= stage
                covered[lds // E.ROW_B - bm] = (("w3" if w & 1 else "w1") if gu else "w2", first + 8 * i)
        assert sorted(covered) == list(range(0, NB_N, 8))
        for row, (arr, src) in covered.items():                   # what the epilogue takes block by block
            wn, h = row // 32, (row // 16) % 2
            if gu:
                assert arr == ("w3" if h else "w1") and src == l * N_out + nt * 64 + wn * 16 + row % 16
            else:
                assert src == l * N_out + nt * 128 + row
    assert len(seen) == total
    assert depth >= 3 and depth * stage <= E.STAGES * E.STAGE_BYTES
    # fragment rows: block i of wave row wm is rows (2 i + wm) * 16 .. + 15, each of the tile's once
    assert sorted((2 * i + wm) * 16 for i in range(bm // 32) for wm in range(2)) == list(range(0, bm, 16))
    # output columns: 4 q + 0..3 of 16-column blocks, each once
    q = lane >> 4
    cols = [wn * 16 + 4 * q + k for wn in range(4) for k in range(4)] if gu else \
           [wn * 32 + 16 * j + 4 * q + k for wn in range(4) for j in range(2) for k in range(4)]
    assert sorted(set(np.concatenate(cols).tolist())) == list(range(64 if gu else 128))


@pytest.mark.parametrize("KT,tiles", [(2, 1), (2, 7), (4, 3), (32, 2)])
@pytest.mark.parametrize("bm", [64, 128])
def test_narrow_ring_order(KT, tiles, bm):
    """Stages issued RING - 1 ahead over the tiles of a workgroup (the last one again past the end): when a stage is
    computed its loads have landed (at most (RING - 2) stages' loads younger), and a buffer is overwritten only after
    the barrier that follows its last read."""
    n, RING = KT * tiles, ring(bm)[1]
    issued = list(range(RING - 1))                     # stage issued i-th, into buffer i % RING
    for s in range(n):
        landed = len(issued) - (RING - 2)              # wait_vm((RING - 2) * LOADS)
        assert s < landed
        # the barrier; then the next issue takes the buffer of stage s - 1, read before the barrier
        buf = len(issued) % RING
        assert buf == (s - 1) % RING
        issued.append(min(len(issued), n - 1))
        assert issued[s] == min(s, n - 1) and s % RING != buf
