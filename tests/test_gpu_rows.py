"""The router's matrix-core kernels (few and many tokens, every number of 16-row blocks, ragged last
workgroup) and the t1 kernel's passes over the rank rows, against the oracle."""
import numpy as np
import pytest

import cmoe_inputs as ci
from oracle import cmoe_oracle as orc
from test_gpu_route_multi import _well_separated

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [257, 8192, 8193, 8250])
@pytest.mark.parametrize("G,K,k,d", [(2, 4, 1, 64), (4, 7, 2, 192), (5, 8, 3, 320), (8, 8, 2, 128), (8, 15, 8, 64)])
def test_router_rows(T, G, K, k, d):
    import torch

    import paper_2510_02345_amd as cm
    cfg = ci.small_config("rows", T=T, d=d, d_ff=64, G=G, K=K, r=4, k=k, q=8, seed=T + G)
    print(f"case {cfg}", flush=True)
    w = ci.generate(cfg)
    cid, eidx, gate, _, _ = orc.route(w["x"], w["router_cluster"], w["router_expert"], K, k, w["cluster_bias"])
    layer = cm.Layer(d, cfg.d_ff, G, K, cfg.r, k, cfg.q, w, T)
    c, e, g = layer.route(torch.from_numpy(w["x"]).to("cuda:0"))
    torch.cuda.synchronize()
    assert np.array_equal(c.cpu().numpy(), cid) and np.array_equal(e.cpu().numpy(), eidx)
    assert np.allclose(g.cpu().numpy(), gate, rtol=1e-5, atol=1e-6)
    # the variant of one cluster and temperature 1 is the same decision
    c2, e2, g2 = layer.route_multi(torch.from_numpy(w["x"]).to("cuda:0"))
    torch.cuda.synchronize()
    assert np.array_equal(c2.cpu().numpy()[:, 0], cid) and np.array_equal(e2.cpu().numpy()[:, 0], eidx)
    assert np.allclose(g2.cpu().numpy()[:, 0], gate, rtol=1e-5, atol=1e-6)
    layer.close()


# rank rows per cluster: 2, 4, 8 and more than 8 blocks of 16, one or two passes; tiles of 64 rows
# that hold one to 64 tokens
@pytest.mark.parametrize("T,K,r,k", [(257, 2, 16, 2), (600, 8, 8, 1), (900, 8, 16, 4), (1300, 16, 32, 3), (321, 32, 16, 8)])
def test_rank_rows_of_selected_experts(T, K, r, k):
    _check_rank_rows(T, 128, K, r, k)


# uneven shares of the contraction, rings that go round, and both sides of the line between the forms of 32 and
# of 64 tokens (256 workgroups of the former, three clusters)
@pytest.mark.parametrize("T,d,K,r,k", [(300, 832, 4, 16, 2), (300, 832, 32, 16, 8), (700, 2048, 8, 16, 2),
                                       (8096, 192, 8, 8, 2), (8097, 192, 8, 8, 2)])
def test_rank_rows_of_both_forms(T, d, K, r, k):
    _check_rank_rows(T, d, K, r, k)


# t1 in the permutation's launch: one and several sort blocks, a last tile of one row, experts whose rank rows are half a block
# of 16, one and two, more blocks of a cluster than one pass takes, several virtual tokens per row of x; and the calls
# on either side of a workgroup per CU
@pytest.mark.parametrize("T,d,G,K,r,k,top_g", [(257, 64, 2, 4, 8, 1, 1), (801, 128, 4, 8, 16, 2, 1), (1025, 192, 3, 4, 32, 1, 1),
                                               (2049, 64, 2, 16, 8, 2, 1), (321, 832, 5, 4, 16, 2, 1), (2688, 64, 3, 4, 8, 2, 1),
                                               (2689, 64, 3, 4, 8, 2, 1), (300, 128, 4, 4, 16, 2, 2), (400, 64, 4, 4, 8, 1, 4)])
def test_rank_rows_with_the_permutation(T, d, G, K, r, k, top_g):
    import torch

    import paper_2510_02345_amd as cm
    cfg = ci.small_config("t1 sort", T=T, d=d, d_ff=320, G=G, K=K, r=r, k=k, q=8, factor_std=0.2, seed=T + d)
    print(f"case {cfg} top_g {top_g}", flush=True)
    w = ci.generate(cfg)
    layer = cm.Layer(d, cfg.d_ff, G, K, r, k, cfg.q, w, T)
    x = torch.from_numpy(w["x"]).to("cuda:0")
    if top_g == 1:
        y, ref = layer.forward(x)["y"].cpu().numpy(), orc.forward_naive(w, w["x"], K, k, cfg.q)["y"]
    else:   # tokens whose choice of clusters or experts does not hinge on a near-tie
        rows = _well_separated(w, cfg, top_g)
        assert len(rows) >= 0.8 * T
        y, ref = layer.forward_multi(x, top_g)["y"].cpu().numpy()[rows], orc.forward_naive_multi(w, w["x"][rows], K, k, cfg.q, top_g)["y"]
    m = orc.error_metrics(y, ref)
    assert m["max_over_rms"] <= 1e-2 and m["mean_rel"] <= 2e-3, m
    layer.close()


def _check_rank_rows(T, d, K, r, k):
    import torch

    import paper_2510_02345_amd as cm
    cfg = ci.small_config("t1", T=T, d=d, d_ff=64, G=3, K=K, r=r, k=k, q=8, factor_std=0.2, seed=T)
    print(f"case {cfg}", flush=True)
    w = ci.generate(cfg)
    ref = orc.forward_naive(w, w["x"], K, k, cfg.q)
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, K, r, k, cfg.q, w, T)
    out = layer.forward(torch.from_numpy(w["x"]).to("cuda:0"))
    torch.cuda.synchronize()
    # factors ten times the usual size: the rank part is a large share of y (the layer's bars)
    m = orc.error_metrics(out["y"].cpu().numpy(), ref["y"])
    assert m["max_over_rms"] <= 1e-2 and m["mean_rel"] <= 2e-3, m
    layer.close()
