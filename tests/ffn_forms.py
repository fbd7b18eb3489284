"""Which tiles a call of the expert FFN runs on: a host copy of the kernels' rules (build_call and f32_large_from of
expert_ffn.hip) with their constants read from the source, so that a test of one form notices when a change of the
rule moves its call to another."""
import os
import re

_SRC = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_05116_amd", "csrc",
                         "expert_ffn.hip")).read()


def _const(name):
    return int(re.search(rf"\b{name} = (\d+)[,;]", _SRC).group(1))


NARROW_MAX_ROWS = _const("kNarrowMaxRows")
CLK = {256: _const("kWideClk"), 64: _const("kNarrow64Clk"), 128: _const("kNarrow128Clk")}


def _up(a, b):
    return -(-a // b)


def m_tiles(counts, rows):
    return sum(_up(n, rows) for n in counts)


def bf16_tiles(counts, rows, d, inter):
    """(gate/up, down) tiles of `rows` rows: 128 H columns and 256 output columns a wide tile, half as many a narrow."""
    gu, dn = (128, 256) if rows == 256 else (64, 128)
    return m_tiles(counts, rows) * (inter // gu), m_tiles(counts, rows) * (d // dn)


def bf16_form(counts, d, inter, cus):
    """Rows of the call's tiles: 64, 128 (narrow) or 256 (wide)."""
    if max(counts, default=0) > NARROW_MAX_ROWS:
        return 256

    def cost(rows):
        gu, dn = bf16_tiles(counts, rows, d, inter)
        return (_up(gu, cus) * (d // 64) + _up(dn, cus) * (inter // 64)) * CLK[rows]

    narrow = min(64, 128, key=cost)
    return narrow if cost(narrow) < cost(256) else 256


_F32 = re.search(r"f32_large_from\(int K\) \{ return K <= (\d+) \? (\d+) : K < (\d+) \? (\d+) : (\d+); \}", _SRC)


def _f32_from(K):
    """Twice the small tiles per CU from which a GEMM takes large ones."""
    k1, t1, k2, t2, t3 = (int(v) for v in _F32.groups())
    return t1 if K <= k1 else t2 if K < k2 else t3


def f32_open(cap, E_loc, K, N, cus):
    """Whether a capacity leaves the tiles of a GEMM of the fp32 FFN to its rows."""
    return 2 * (cap // 16 + E_loc) * _up(N, 16) >= _f32_from(K) * cus


def f32_large(counts, K, N, cus):
    """Whether the rows of a GEMM of the fp32 FFN take the large tiles (if its capacity allows them)."""
    small, large = m_tiles(counts, 16) * _up(N, 16), m_tiles(counts, 64) * _up(N, 32)
    return 2 * small >= _f32_from(K) * cus and small >= 3 * large
