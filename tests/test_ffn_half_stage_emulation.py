"""CPU emulation of the bf16 expert FFN's stage pipeline (k_loop, load_half0
and load_half1 of expert_ffn.hip).

A stage (K = 64 of a 256 x 256 tile) is loaded in parts (A, and the four
quarters of B, two of them a half), each issued as soon as the LDS space it
overwrites has been read by every wave.  The test
replays the program order of the loader and compute waves on the host:

* the loader waves' direct loads cover every 8-row block of a stage once, with
  the operand row the fragment reads and the epilogue expect there, inside the
  weight arrays;
* no fragment is read before the loads that fill it have landed (the loader's
  counted vmcnt wait, then a barrier), and no load is issued into rows that a
  wave may still read (a completed read, then a barrier).
"""
import numpy as np
import pytest

from tests import test_ffn_tiling_emulation as E

HALF_B = E.BLD // 2


def b_loads(half, lw):
    """(first LDS row of the B tile, quarter slot, 8-row block index) of a loader's B loads in one half."""
    first = (lw >> 1) * E.WN + half * 64 + (lw & 1) * 16
    return [(first + 32 * q + 8 * i, q, i) for q in range(2) for i in range(HALF_B // 2)]


def b_source_row(gu, lw, half, q, i, nt, expert, N_out):
    """(array, row) that tile_loads and load_b address for that block's first row."""
    wn, h = lw >> 1, lw & 1
    if gu:
        row = expert * N_out + nt * (E.BN // 2) + wn * (E.WN // 2) + h * 16
        return ("w3" if q else "w1"), row + half * 32 + i * 8
    row = expert * N_out + nt * E.BN + wn * E.WN + h * 16
    return "w2", row + 32 * q + half * 64 + i * 8


@pytest.mark.parametrize("gu", [True, False])
def test_half_stage_loads_cover_the_stage(gu):
    N_out = 2048 if gu else 7168
    n_tiles = N_out // (E.BN // 2) if gu else N_out // E.BN
    for expert, nt in ((0, 0), (7, n_tiles - 1), (3, 5)):
        seen = {}
        for lw in range(E.NL):
            for half in range(2):
                for lds_row, q, i in b_loads(half, lw):
                    arr, row = b_source_row(gu, lw, half, q, i, nt, expert, N_out)
                    assert lds_row % 8 == 0 and 0 <= lds_row < E.BN and lds_row not in seen
                    # the swizzle of the block's rows depends on the block's parity: col_b[i & 1] of lane_map
                    assert (lds_row // 8) % 2 == i % 2
                    # the half holds exactly the wave columns' quarters 2 half, 2 half + 1
                    assert (lds_row % E.WN) // 64 == half
                    assert 0 <= row and row + 8 <= (expert + 1) * N_out
                    seen[lds_row] = (arr, row)
        assert len(seen) == E.BN // 8
        for lds_row, (arr, row) in seen.items():
            if gu:      # 32-row blocks of W1 and W3 alternate
                pair, r = lds_row // 64, lds_row % 32
                assert arr == ("w3" if (lds_row // 32) % 2 else "w1")
                assert row == expert * N_out + nt * 128 + 32 * pair + r
            else:
                assert (arr, row) == ("w2", expert * N_out + nt * 256 + lds_row)


@pytest.mark.parametrize("rows", range(1, E.BM + 1, 3))
def test_loaders_of_waves_with_rows_load_a(rows):
    """A loader brings A rows if its own wave row w // 2 has rows (a_on): then every 64-row block that a computing wave
    reads is loaded, and a tile of at most 64 rows has two loaders' A loads, not four."""
    a_on = [w // E.WAVES_N * E.WM < rows for w in range(E.NL)]
    for wm in range(E.BM // E.WM):
        assert not wm * E.WM < rows or a_on[wm]
    assert sum(a_on) == (2 if rows <= E.WM else 4)


@pytest.mark.parametrize("loads_a", [True, False])
@pytest.mark.parametrize("KT", [2, 4, 12, 22, 112])
def test_half_stage_pipeline_order(KT, loads_a):
    """Program order of one tile over the parts A, Q0..Q3 of its stages; an epoch is the time between two
    barriers, which all waves share.  loads_a: the loader brings A rows (its own wave has rows), or only B; its waits
    count what it has in flight."""
    a_ld = E.ALD if loads_a else 0
    loads_of = {"A": a_ld, "Q0": HALF_B // 2, "Q1": HALF_B // 2, "Q2": HALF_B // 2, "Q3": HALF_B // 2}
    queue, landed = [], {}                # the loader's loads in order; landed[stage, part]: the epoch it is safe from
    reads, issues = [], []                # (epoch, stage, part)
    epoch = 0

    def issue(kt, *parts):
        for p in parts:
            issues.append((epoch, kt, p))
            queue.append((kt, p, loads_of[p]))

    def wait(n):
        left = n
        for kt, p, cnt in reversed(queue):
            if left > 0:                  # may still be in flight (whole or in part)
                left -= cnt
            else:
                landed.setdefault((kt, p), epoch + 1)

    def read(kt, *parts):
        reads.extend((epoch, kt, p) for p in parts)

    issue(0, "A", "Q0", "Q1", "Q2", "Q3")
    wait(0)
    epoch += 1
    issue(1, "A", "Q0", "Q1")
    read(0, "Q0", "A")
    for kt in range(KT):
        next1, next2 = kt + 1 < KT, kt + 2 < KT
        read(kt, "A", "Q1")
        if next1:
            issue(kt + 1, "Q2", "Q3")
        wait(a_ld + 8 if next1 else 0)
        epoch += 1                                        # barrier a
        read(kt, "Q2", "Q3")
        if next2:
            issue(kt + 2, "A")
        if next1:
            wait(a_ld + 4 if next2 else 4)
        epoch += 1                                        # barrier c
        if next1:
            read(kt + 1, "Q0", "A")
        if next2:
            issue(kt + 2, "Q0", "Q1")
    assert len(issues) == 5 * KT
    for ep, kt, part in reads:
        assert landed[kt, part] <= ep, (kt, part)
    last_read = {}
    for ep, kt, part in reads:
        last_read[kt, part] = max(last_read.get((kt, part), 0), ep)
    for ep, kt, part in issues:
        if kt >= 2:                                       # the reads completed before a barrier that precedes the issue
            assert last_read[kt - 2, part] < ep, (kt, part)
    # the next tile's stage 0 goes to buffer 0 after barrier a of the last stage
    assert max(ep for ep, kt, _ in reads if kt == KT - 2) < 2 + 2 * (KT - 1)
    assert KT % 2 == 0
