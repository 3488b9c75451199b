"""The permutation kernels on their own (exact) and, through the layer's output, the expert-pair
order inside the clusters: one, two and three launches, block edges, the most bins."""
import numpy as np
import pytest

import cmoe_inputs as ci
from oracle import cmoe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 63, 64, 65, 256, 257, 700, 1024, 1025, 4096, 4097, 131072, 131073, 150001])
@pytest.mark.parametrize("G", [1, 5, 64])
def test_permutation_is_the_stable_sort(T, G):
    import torch

    import paper_2510_02345_amd as cm
    print(f"case T={T} G={G}", flush=True)
    cfg = ci.small_config("sort", T=16, d=64, d_ff=64, G=G, K=2, r=4, k=1, q=8, seed=7)
    layer = cm.Layer(cfg.d, cfg.d_ff, G, cfg.K, cfg.r, cfg.k, cfg.q, ci.generate(cfg), T)
    # skewed ids, one bin empty where there are several
    ids = (np.random.default_rng(T + G).random(T) ** 2 * G).astype(np.int32)
    ids[ids == G // 2] = 0 if G > 1 else ids[ids == G // 2]
    ref = np.argsort(ids, kind="stable").astype(np.int32)
    for call in (layer.permute, layer.permute_static):
        perm, inv, off = call(torch.from_numpy(ids).to("cuda:0"))
        torch.cuda.synchronize()
        assert np.array_equal(perm.cpu().numpy(), ref)
        assert np.array_equal(inv.cpu().numpy()[ref], np.arange(T))
        assert np.array_equal(off.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(ids, minlength=G))]))
    layer.close()


# with 4096 bins two launches up to 16 blocks of 1024 tokens and three above; with 32 bins up to 128 and above
@pytest.mark.parametrize("T,G,K,k", [(300, 64, 8, 2), (5000, 64, 8, 2), (16384, 64, 8, 2), (16385, 64, 8, 2), (17409, 64, 8, 2),
                                     (4097, 3, 32, 1), (4500, 2, 4, 4), (131073, 2, 4, 2)])
def test_pair_order_leaves_the_output_in_place(T, G, K, k):
    import torch

    import paper_2510_02345_amd as cm
    print(f"case T={T} G={G} K={K} k={k}", flush=True)
    cfg = ci.small_config("pairs", T=T, d=64, d_ff=64, G=G, K=K, r=4, k=k, q=8, seed=T)
    w = ci.generate(cfg)
    ref = orc.forward_naive(w, w["x"], K, k, cfg.q)
    layer = cm.Layer(cfg.d, cfg.d_ff, G, K, cfg.r, k, cfg.q, w, T)
    out = layer.forward(torch.from_numpy(w["x"]).to("cuda:0"))
    torch.cuda.synchronize()
    for n in ("cluster_id", "expert_idx", "perm", "inv_perm", "offsets"):
        assert np.array_equal(out[n].cpu().numpy(), ref[n]), n
    m = orc.error_metrics(out["y"].cpu().numpy(), ref["y"])   # the layer's bars (FP16 operands and results)
    assert m["max_over_rms"] <= 1e-2 and m["mean_rel"] <= 2e-3, m
    layer.close()


# The pair sort of a permutation that the caller has: rows of one cluster up to, at and beyond what the
# workgroup keeps in registers (8 x 1024), one and two keys.
@pytest.mark.parametrize("T,G,k", [(257, 1, 2), (1025, 1, 2), (8192, 1, 1), (8193, 1, 2), (12000, 1, 2), (20000, 2, 2)])
def test_pair_order_of_a_given_permutation(T, G, k):
    import torch

    import paper_2510_02345_amd as cm
    print(f"case T={T} G={G} k={k}", flush=True)
    cfg = ci.small_config("pairs2", T=T, d=64, d_ff=64, G=G, K=4, r=4, k=k, q=8, seed=T)
    w = ci.generate(cfg)
    ref = orc.forward_naive(w, w["x"], cfg.K, k, cfg.q)
    layer = cm.Layer(cfg.d, cfg.d_ff, G, cfg.K, cfg.r, k, cfg.q, w, T)
    x = torch.from_numpy(w["x"]).to("cuda:0")
    c, e, g = layer.route(x)
    perm, inv, off = layer.permute(c)
    yb, s = layer.ffn_forward(x, perm, off, e, g)
    y = layer.combine(yb, s, perm, inv, off, e, g)
    torch.cuda.synchronize()
    m = orc.error_metrics(y.cpu().numpy(), ref["y"])   # the layer's bars (FP16 operands and results)
    assert m["max_over_rms"] <= 1e-2 and m["mean_rel"] <= 2e-3, m
    layer.close()
