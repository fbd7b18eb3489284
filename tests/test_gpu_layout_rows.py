"""Layout on the GPU against the oracle, at the edges of its scatter blocks:
one to three chunks of 256 tokens per source rank (each rank's first chunk
writes the rank's send counts), 1 to 64 ranks, and 1 to 8 slots per token.
Whole numbers: every array bit for bit, from both entry points."""
import numpy as np
import pytest

from workloads import generator as gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2607_05116_amd.layer import DeviceLayer  # noqa: E402

import oracle  # noqa: E402

NAMES = ("send_counts", "send_offsets", "recv_offsets", "expert_counts", "expert_offsets", "slot_pos", "copy_row",
         "vol", "totals")


@pytest.mark.parametrize("E,k,R,rpn,p,T_loc", [
    (64, 8, 64, 8, 0.3, 257), (256, 7, 64, 8, 0.0, 1), (20, 4, 1, 1, 0.2, 513), (34, 1, 2, 1, 0.1, 256),
    (256, 8, 32, 8, 0.0, 64), (9, 3, 3, 1, 0.3, 65)])
def test_layout_scatter_edges(E, k, R, rpn, p, T_loc):
    T = R * T_loc
    rng = np.random.default_rng(E + k + T_loc)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    perm = rng.permutation(E)
    er, el = (perm // (E // R)).astype(np.int32), (perm % (E // R)).astype(np.int32)
    cfg = gen.Config("edges", T=T, d=8, E=E, k=k, inter=128, R=R, ranks_per_node=rpn, n_clusters=1, zipf_s=0.0,
                     dtype="bf16")
    r = oracle.route_prune(logits, k, er, rpn, T_loc, 5.0, p)
    lay = oracle.dispatch_layout(r["idx"], r["keep"], r["mask"], er, el, R, rpn, T_loc, E)
    n_recv = int(lay["recv_offsets"][-1])
    L = DeviceLayer(cfg, logits, np.zeros((T, 8), np.uint16), er, el, p, 5.0, row_cap=8, recv_cap=8)
    for call in (lambda: L.route_layout(False), L.front):
        for n in NAMES:
            L.lay_t[n].fill_(-7) if n != "vol" else L.lay_t[n].fill_(99)
        L.lay_t["recv_token"].fill_(-7)
        call()
        torch.cuda.synchronize()
        for n in NAMES:
            assert np.array_equal(L.host(n), lay[n]), n
        tok = L.host("recv_token")
        assert np.array_equal(tok[:n_recv], lay["recv_token"])
        assert (tok[n_recv:] == -7).all()
