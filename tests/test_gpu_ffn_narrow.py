"""The bf16 expert FFN's narrow tiles (calls of few rows per expert) on the GPU: against the oracle at the edges of
their tiles, bit for bit against the wide tiles, and with the destination combine in the epilogue."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_05116_amd import capi
from tests import cases as C
from tests.ffn_forms import bf16_form, bf16_tiles
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


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


EDGES = [1, 65, 127, 128, 129, 0]


@pytest.mark.parametrize("d,inter,counts,cap,form", [
    (256, 128, [1], 1, 64),                              # two K stages in the down GEMM, one row
    (512, 384, [15, 16, 17, 0, 31, 33], 200, 64),
    (1024, 256, [63, 64, 65, 0, 2, 129], 8192, 64),      # the first launch of a call of the fused kernel's capacity
    (512, 256, [1] * 70 + [0] * 30, 70, 256),            # the forms cost the same: wide, a tile a workgroup
    (256, 384, [40] * 200 + [0], 8000, 64),              # tiles in turn, in both GEMMs
    (1024, 256, EDGES + [70] * 18, 1800, 128),           # 128-row tiles, a tile a workgroup in the gate/up GEMM
    (1024, 256, EDGES + [100] * 66, 7100, 128),          # and in turn in both, the row counts at the tiles' edges
    (1024, 256, EDGES + [100] * 66, 8300, 128),
])
@pytest.mark.parametrize("gathered", [False, True])
def test_narrow_ffn_against_oracle(d, inter, counts, cap, form, gathered):
    assert bf16_form(counts, d, inter, _cus()) == form
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


@pytest.mark.parametrize("d,inter,counts,form", [(256, 384, [40] * 200 + [0], 64),
                                                 (1024, 256, EDGES + [100] * 66, 128)])
@pytest.mark.parametrize("cap", [8000, 9000])
def test_narrow_tiles_in_turn_equal_wide_bits(d, inter, counts, form, cap):
    """Calls of more narrow tiles than workgroups in both GEMMs (the ring of stages runs on across a workgroup's tiles)
    give the wide tiles' bits: plain, gathered and with the destination combine.  A cap on the workgroups keeps a call
    on wide tiles."""
    n_cu, rows = _cus(), sum(counts)
    assert bf16_form(counts, d, inter, n_cu) == form and min(bf16_tiles(counts, form, d, inter)) > n_cu
    g = torch.Generator(device="cuda").manual_seed(form)
    E_loc, w, offs = len(counts), _weights(g, len(counts), d, inter), _offs(counts)
    x, ws = _bf(g, cap, d), _ws(d, inter, cap)
    src = torch.randint(0, cap, (cap,), generator=g, device="cuda", dtype=torch.int32)
    dst = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    dst[:rows:2] = torch.randperm(cap, generator=g, device="cuda")[:len(dst[:rows:2])].to(torch.int32)
    gate = torch.rand(cap, generator=g, device="cuda")
    outs = []
    for opt in (None, capi.make_ffn_options(max_workgroups=n_cu)):
        y = [torch.zeros((cap, d), dtype=torch.bfloat16, device="cuda") for _ in range(4)]
        capi.cap_expert_ffn_ex(CDT, E_loc, d, inter, cap, x, 0, None, offs, *w, y[0], ws, options=opt)
        capi.cap_expert_ffn_ex(CDT, E_loc, d, inter, cap, x, cap, src, offs, *w, y[1], ws, options=opt)
        capi.cap_expert_ffn_combine(CDT, E_loc, d, inter, cap, x, cap, src, offs, *w, y[2], dst, gate, y[3], cap, ws,
                                    options=opt)
        torch.cuda.synchronize()
        outs.append(y)
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert all(t.any() for t in outs[0])


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
