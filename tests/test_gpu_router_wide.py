"""The fused router of more than 128 experts (eight waves, two rings of stages) at the edges of its tiles: one to
five K stages, token tails, expert counts that are no multiple of 64."""
import numpy as np
import pytest

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
