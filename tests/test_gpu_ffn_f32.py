"""The fp32 expert FFN at the edges of its matrix-instruction tiles, against the fp64 definition."""
import numpy as np
import pytest
import torch

from paper_2607_05116_amd import capi
from tests.ffn_forms import f32_large, f32_open

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,inter,counts,cap", [
    (4, 1, [1], 1),                                # one K step, mostly past K; one output column
    (128, 256, [33, 28, 0, 65, 43], 512),
    (20, 17, [15, 16, 17], 60),                    # rows of H and W2 not 16-byte aligned; partial column blocks
    (132, 64, [3, 0, 130], 140),                   # K one step past a batch
    (64, 2048, [700, 0, 900], 2000),               # large tiles in the gate/up GEMM, small ones in the down GEMM
    (2048, 63, [1500, 1], 1600),                   # large tiles, K not a multiple of four, in the down GEMM
    (256, 320, [9, 0, 3, 40], 4000),               # a capacity for large tiles, rows for small ones
    (64, 512, [16] * 160, 3000),                   # many small tiles, but three quarters of every large one empty
    (256, 768, [700, 33, 900], 1700),              # large tiles in the gate/up GEMM, remainders of 16 and of 64
    (1024, 128, [700, 33, 900], 1700),             # the same in the down GEMM
])
@pytest.mark.parametrize("gathered", [False, True])
def test_ffn_f32_tiles(d, inter, counts, cap, gathered):
    g = torch.Generator(device="cuda").manual_seed(d + inter)
    E_loc, rows = len(counts), sum(counts)
    rnd = lambda std, *shape: torch.randn(shape, generator=g, device="cuda") * std
    x = rnd(1.0, cap + 7, d)
    w1, w3, w2 = rnd(d ** -0.5, E_loc, inter, d), rnd(d ** -0.5, E_loc, inter, d), rnd(inter ** -0.5, E_loc, d, inter)
    offs = torch.tensor(np.concatenate([[0], np.cumsum(counts)]) + 5, dtype=torch.int32, device="cuda")
    y = torch.zeros((cap, d), device="cuda")
    ws = torch.empty(capi.cap_workspace_size(capi.CAP_OP_EXPERT_FFN, None, d, inter, cap, capi.CAP_DTYPE_F32),
                     dtype=torch.uint8, device="cuda")
    if gathered:
        src = torch.randint(-2, x.shape[0] + 2, (cap,), generator=g, device="cuda", dtype=torch.int32)
        capi.cap_expert_ffn_gather(capi.CAP_DTYPE_F32, E_loc, d, inter, cap, x, x.shape[0], src, offs, w1, w3, w2, y, ws)
        xs = x[src.long().clamp(0, x.shape[0] - 1)]
    else:
        capi.cap_expert_ffn(capi.CAP_DTYPE_F32, E_loc, d, inter, cap, x[:cap], offs, w1, w3, w2, y, ws)
        xs = x
    torch.cuda.synchronize()
    ref, at = torch.zeros((rows, d), dtype=torch.float64, device="cuda"), 0
    for l, n in enumerate(counts):
        r = xs[at:at + n].double()
        h = torch.nn.functional.silu(r @ w1[l].double().T) * (r @ w3[l].double().T)
        ref[at:at + n] = h @ w2[l].double().T
        at += n
    # Rounding the running sum of K independent terms K times, each to within u = 2^-24 of a partial sum whose rms
    # grows as sqrt(k / K), leaves an rms error of at most u * sqrt(K / 2) of the result's; the gate and the up sum
    # (K = d) both enter H, the down sum (K = inter) adds its own, and silu's hardware exp2 and reciprocal a few u.
    u = 2.0 ** -24
    bound = u * (2 * (d / 2) ** 0.5 + (inter / 2) ** 0.5 + 8)
    err = y[:rows].double() - ref
    assert float(err.norm() / ref.norm()) <= bound
    assert float(err.abs().max()) <= 6 * bound * float(ref.abs().max())
    assert not y[rows:].any()


def test_ffn_f32_forms_of_the_cases():
    """The capacity-bound cases above take the tiles their comments name, and their capacity leaves both open."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for d, inter, counts, cap, gu, dn in ((256, 320, [9, 0, 3, 40], 4000, False, False),
                                          (64, 512, [16] * 160, 3000, False, False),
                                          (256, 768, [700, 33, 900], 1700, True, False),
                                          (1024, 128, [700, 33, 900], 1700, False, True),
                                          (64, 2048, [700, 0, 900], 2000, True, False),
                                          (2048, 63, [1500, 1], 1600, False, True)):
        assert f32_large(counts, d, inter, cus) == gu and f32_large(counts, inter, d, cus) == dn, (d, inter)
        assert f32_open(cap, len(counts), d, inter, cus) or f32_open(cap, len(counts), inter, d, cus)


def test_ffn_f32_capacity_gives_the_same_bits():
    """The tiles follow the rows: a capacity many times the rows changes nothing."""
    d, inter, counts = 512, 512, [4, 60, 0, 17]
    g = torch.Generator(device="cuda").manual_seed(8)
    w = [torch.randn(s, generator=g, device="cuda") * 0.05 for s in ((4, inter, d), (4, inter, d), (4, d, inter))]
    offs = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    rows, outs = sum(counts), []
    x = torch.randn((8000, d), generator=g, device="cuda")
    for cap in (rows, 8000):
        y = torch.zeros((cap, d), device="cuda")
        ws = torch.empty(capi.cap_workspace_size(capi.CAP_OP_EXPERT_FFN, None, d, inter, cap, capi.CAP_DTYPE_F32),
                         dtype=torch.uint8, device="cuda")
        capi.cap_expert_ffn(capi.CAP_DTYPE_F32, 4, d, inter, cap, x[:cap], offs, *w, y, ws)
        outs.append(y[:rows])
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))
