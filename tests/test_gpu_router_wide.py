"""The fused router of more than 128 experts (eight waves, two rings of stages) at the edges of its tiles: one to
five K stages, token tails, expert counts that are no multiple of 64."""
import numpy as np
import pytest
import torch

from paper_2607_05116_amd import capi
from paper_2607_05116_amd.layer import DeviceLayer
from tests.test_gpu_parity import _check_router_route
from workloads import generator as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,R,d,p", [(8, 256, 8, 8, 64, 0.1), (136, 136, 2, 8, 192, 0.0), (128, 160, 6, 16, 256, 0.2),
                                         (400, 200, 8, 8, 320, 0.3), (1016, 256, 1, 8, 1088, 0.1)])
def test_router_wide_shapes(T, E, k, R, d, p):
    cfg = gen.Config("rw", T=T, d=d, E=E, k=k, inter=128, R=R, ranks_per_node=8, n_clusters=1, zipf_s=0.0, dtype="bf16")
    rng = np.random.default_rng(T + E)
    x = gen.f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32))
    wg = gen.f32_to_bf16_bits((rng.standard_normal((E, d)) / np.sqrt(d)).astype(np.float32))
    perm = rng.permutation(E)
    er, el = (perm // (E // R)).astype(np.int32), (perm % (E // R)).astype(np.int32)
    L = DeviceLayer(cfg, np.zeros((T, E), np.float32), x, er, el, p, 5.0, row_cap=8, recv_cap=8)
    _check_router_route(L, cfg, x, wg, er)


@pytest.mark.parametrize("E,k", [(256, 8), (136, 2)])
def test_router_rows_past_the_wide_kernel(E, k):
    """d = 2^23, the least that the four-wave kernel takes for more than 128 experts: its logits against 64-bit sums,
    its decisions against the logits-in kernel on them."""
    T, d, R = 8, 1 << 23, 8
    g = torch.Generator(device="cuda").manual_seed(E)
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    wg = torch.empty((E, d), dtype=torch.bfloat16, device="cuda")
    for e in range(E):
        wg[e] = torch.randn(d, generator=g, device="cuda") * d ** -0.5
    er = (torch.randperm(E, generator=g, device="cuda") // (E // R)).to(torch.int32)
    topo = capi.make_topology(E, R, R, T, k, er, torch.zeros_like(er), 5.0)
    out = [dict(idx=torch.zeros((T, k), dtype=torch.int32, device="cuda"), w=torch.zeros((T, k), device="cuda"),
                keep=torch.zeros((T, k), dtype=torch.uint8, device="cuda"),
                mask=torch.zeros(T, dtype=torch.int64, device="cuda")) for _ in range(2)]
    lg = torch.zeros((T, E), device="cuda")
    capi.cap_router_route_prune(topo, capi.CAP_DTYPE_BF16, d, x, wg, 0.1, *out[0].values(), lg)
    capi.cap_route_prune(topo, lg, 0.1, *out[1].values())
    torch.cuda.synchronize()
    for n in out[0]:
        assert torch.equal(out[0][n], out[1][n]), n
    ref = torch.zeros((T, E), dtype=torch.float64, device="cuda")
    for c in range(0, d, 1 << 18):
        ref += x[:, c:c + (1 << 18)].double() @ wg[:, c:c + (1 << 18)].double().T
    # at most d roundings of a running sum, each to within 2^-24 of a partial sum whose rms grows as sqrt(n / d)
    bound = 2.0 ** -24 * (d / 2) ** 0.5
    err = lg.double() - ref
    assert float(err.norm() / ref.norm()) <= bound
    assert float(err.abs().max()) <= 6 * bound * float(ref.abs().max())
