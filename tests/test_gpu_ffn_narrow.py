"""The bf16 expert FFN's narrow tiles (calls of few rows per expert) on the GPU: against the oracle at the edges of
their tiles, bit for bit against the wide tiles, and with the destination combine in the epilogue."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_05116_amd import capi
from tests import cases as C
from workloads import generator as gen

pytestmark = pytest.mark.gpu
CDT = capi.CAP_DTYPE_BF16


def _bf(g, *shape, std=1.0):
    return (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)


def _weights(g, E_loc, d, inter):
    return (_bf(g, E_loc, inter, d, std=d ** -0.5), _bf(g, E_loc, inter, d, std=d ** -0.5),
            _bf(g, E_loc, d, inter, std=1 / (12 * inter ** 0.5)))


def _ws(d, inter, cap):
    return torch.full((capi.cap_workspace_size(capi.CAP_OP_EXPERT_FFN, None, d, inter, cap, CDT),), 0xA5,
                      dtype=torch.uint8, device="cuda")


def _offs(counts):
    return torch.tensor(np.concatenate([[0], np.cumsum(counts)]) + 3, dtype=torch.int32, device="cuda")


def _f32(t):
    return t.float().cpu().numpy()


@pytest.mark.parametrize("d,inter,counts,cap", [
    (256, 128, [1], 1),                                  # two K stages in the down GEMM, one row
    (512, 384, [15, 16, 17, 0, 31, 33], 200),
    (1024, 256, [63, 64, 65, 0, 2, 129], 8192),          # the first launch of a call of the fused kernel's capacity
    (512, 256, [1] * 70 + [0] * 30, 70),                 # more tiles than workgroups in turn
])
@pytest.mark.parametrize("gathered", [False, True])
def test_narrow_ffn_against_oracle(d, inter, counts, cap, gathered):
    g = torch.Generator(device="cuda").manual_seed(len(counts) + d)
    E_loc, rows = len(counts), sum(counts)
    w = _weights(g, E_loc, d, inter)
    x = _bf(g, max(cap, rows) + 9, d)
    y = torch.zeros((cap, d), dtype=torch.bfloat16, device="cuda")
    if gathered:
        src = torch.randint(-2, x.shape[0] + 2, (cap,), generator=g, device="cuda", dtype=torch.int32)
        capi.cap_expert_ffn_gather(CDT, E_loc, d, inter, cap, x, x.shape[0], src, _offs(counts), *w, y, _ws(d, inter, cap))
        xs = x[src[:rows].long().clamp(0, x.shape[0] - 1)]
    else:
        capi.cap_expert_ffn(CDT, E_loc, d, inter, cap, x[:cap], _offs(counts), *w, y, _ws(d, inter, cap))
        xs = x[:rows]
    torch.cuda.synchronize()
    w1, w3, w2 = (_f32(t) for t in w)
    ref = oracle.expert_ffn(_f32(xs), np.concatenate([[0], np.cumsum(counts)]).astype(np.int32),
                            [(w1[l], w3[l], w2[l]) for l in range(E_loc)])
    got = _f32(y[:rows])
    ok, worst = C.within_tol(got, ref)           # bf16 H and Y over fp32 sums, as for the wide tiles
    assert ok, worst
    assert C.rel_fro(got, ref) <= 1e-2
    assert not y[rows:].any()


@pytest.mark.parametrize("cap", [2600, 8300])
def test_narrow_rows_equal_wide_rows(cap):
    """The same expert rows alone (narrow tiles) and beside an expert of more rows than narrow tiles take: same bits."""
    d, inter, few, many = 512, 256, [5, 64, 0, 130, 77], 2200
    g = torch.Generator(device="cuda").manual_seed(cap)
    w = _weights(g, len(few) + 1, d, inter)
    x = _bf(g, cap, d)
    n = sum(few)
    y1 = torch.zeros((cap, d), dtype=torch.bfloat16, device="cuda")
    y2 = torch.zeros_like(y1)
    capi.cap_expert_ffn(CDT, len(few), d, inter, cap, x, _offs(few), *(t[:-1].contiguous() for t in w), y1,
                        _ws(d, inter, cap))
    capi.cap_expert_ffn(CDT, len(few) + 1, d, inter, cap, x, _offs(few + [many]), *w, y2, _ws(d, inter, cap))
    torch.cuda.synchronize()
    assert torch.equal(y1[:n].view(torch.int16), y2[:n].view(torch.int16))
    # the combining call: the rows with a plan go, scaled, to parts; the others to y
    dst = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    dst[:n:2] = torch.randperm(cap, generator=g, device="cuda")[:len(dst[:n:2])].to(torch.int32)
    dst[1] = cap + 5                                     # past parts_rows: to y
    gate = torch.rand(cap, generator=g, device="cuda")
    src = torch.arange(cap, dtype=torch.int32, device="cuda")
    outs = []
    for E_loc, counts in ((len(few), few), (len(few) + 1, few + [many])):
        y = torch.zeros((cap, d), dtype=torch.bfloat16, device="cuda")
        parts = torch.zeros((cap, d), dtype=torch.bfloat16, device="cuda")
        capi.cap_expert_ffn_combine(CDT, E_loc, d, inter, cap, x, cap, src, _offs(counts),
                                    *(t[:E_loc].contiguous() for t in w), y, dst, gate, parts, cap, _ws(d, inter, cap))
        torch.cuda.synchronize()
        outs.append((y[:n].clone(), parts))
    for a, b in zip(outs[0], outs[1]):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert torch.equal(outs[0][0][1::2].view(torch.int16), y1[1:n:2].view(torch.int16))
    want = (gate[:n:2, None] * y1[:n:2].float()).to(torch.bfloat16)
    assert torch.equal(outs[0][1][dst[:n:2].long()].view(torch.int16), want.view(torch.int16))
