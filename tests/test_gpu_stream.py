"""The weight streams for few tokens (16 and 32 tokens of a cluster per workgroup, slots found from the
offsets), over the rule's edge, single tokens, empty and overfull clusters, against the oracle."""
import numpy as np
import pytest

import cmoe_inputs as ci
from oracle import cmoe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,T", [(1, 1), (1, 12), (1, 16), (1, 17), (2, 24), (2, 25), (2, 256), (5, 60), (5, 61), (5, 177),
                                 (16, 256), (16, 193), (64, 3), (64, 255)])
@pytest.mark.parametrize("skew", [0.0, 100.0])
def test_weight_streams(G, T, skew):
    _check(ci.small_config("stream", T=T, d=192, d_ff=128, G=G, K=4, r=8, k=2, q=32, seed=T + G), skew)


# 32-token workgroups: more than 1024 workgroups of the 16-token form (64 row blocks of 2048 rows); the
# up-projection takes them from 13 expected tokens on, the down-projection from 12
@pytest.mark.parametrize("G,T", [(15, 180), (15, 181), (15, 195), (15, 196), (1, 255), (1, 256), (7, 144), (7, 160),
                                 (6, 255)])
@pytest.mark.parametrize("skew", [0.0, 100.0])
def test_wide_weight_streams(G, T, skew):
    _check(ci.small_config("wide", T=T, d=64, d_ff=2048, G=G, K=4, r=8, k=2, q=32, seed=T + G), skew)


def test_wide_weight_streams_beyond_the_caches():
    # bases above the size from which they are read without being kept
    _check(ci.small_config("far", T=200, d=2048, d_ff=2048, G=13, K=4, r=8, k=2, q=32, seed=213), 0.0)


# parts of the down-projection's contraction: 4, 2 and 1 of 32, 17 and 15 steps, uneven shares; as many parts as the
# scratch space holds to the byte (40 tokens), one token more; the largest launch that is split, the next one
@pytest.mark.parametrize("d,d_ff,G,T", [(256, 2048, 2, 1), (256, 1088, 2, 3), (256, 960, 2, 3), (512, 2048, 1, 40),
                                        (512, 2048, 1, 41), (192, 2112, 4, 7), (3072, 1024, 1, 1), (3136, 1024, 1, 1)])
def test_parts_of_the_contraction(d, d_ff, G, T):
    _check(ci.small_config("parts", T=T, d=d, d_ff=d_ff, G=G, K=4, r=8, k=2, q=32, seed=T + G), 0.0)


# residual terms: groups of experts whose rank rows fill 1 to 64 lanes; routers of 16 rows (all logits at once), of 17
@pytest.mark.parametrize("G,K,r,k", [(2, 8, 4, 1), (2, 8, 4, 3), (2, 8, 4, 8), (2, 8, 8, 1), (2, 8, 8, 5), (2, 8, 16, 1),
                                     (2, 8, 16, 3), (2, 8, 16, 8), (2, 8, 32, 1), (2, 8, 32, 3), (2, 7, 8, 2),
                                     (1, 16, 8, 2), (1, 15, 16, 8), (8, 1, 32, 1)])
def test_groups_of_experts(G, K, r, k):
    _check(ci.small_config("groups", T=5, d=128, d_ff=2112, G=G, K=K, r=r, k=k, q=32, seed=r + k), 0.0)


# V1 x beside the stream: one, two and four rank rows a wavefront, once and twice around, widths of part of a
# wavefront's chunks, of all of them and of one step more, for both numbers of chunks; factors that make up much of y
@pytest.mark.parametrize("r", [4, 8, 16, 32])
@pytest.mark.parametrize("d", [64, 1024, 1088, 2112])
def test_rank_rows_of_few_tokens(r, d):
    _check(ci.small_config("t1few", T=21, d=d, d_ff=64, G=2, K=4, r=r, k=2, q=32, factor_std=0.1, seed=r + d), 0.0)


def _check(cfg, skew):
    import torch

    import paper_2510_02345_amd as cm
    print(f"case {cfg} skew {skew}", flush=True)
    G, T = cfg.G, cfg.T
    w = ci.generate(cfg)
    if skew:   # every token in the last cluster
        w["cluster_bias"] = np.zeros(G, dtype=np.float32)
        w["cluster_bias"][-1] = skew
    ref = orc.forward_naive(w, w["x"], cfg.K, cfg.k, cfg.q)
    for pack in (True, False):
        layer = cm.Layer(cfg.d, cfg.d_ff, G, cfg.K, cfg.r, cfg.k, cfg.q, w, T, pack=pack)
        out = layer.forward(torch.from_numpy(w["x"]).to("cuda:0"))
        torch.cuda.synchronize()
        for n in ("cluster_id", "expert_idx", "perm", "offsets"):
            assert np.array_equal(out[n].cpu().numpy(), ref[n]), n
        inv = out["inv_perm"].cpu().numpy()
        assert np.array_equal(inv[ref["perm"]], np.arange(T)), "inv_perm"
        m = orc.error_metrics(out["y"].cpu().numpy(), ref["y"])   # the layer's bars (FP16 operands and results)
        assert m["max_over_rms"] <= 1e-2 and m["mean_rel"] <= 2e-3, m
        layer.close()


# The form of 64 tokens a pass (bases beyond the caches): a pass of up to 16, 32, 48 and 64 tokens, a second pass of a
# cluster, rows and blocks of the contraction that do not divide into workgroups and chunks; whole step and single calls,
# re-tiled and canonical bases.
@pytest.mark.parametrize("T,pack", [(58, True), (100, True), (200, True), (256, False)])
def test_sixty_four_token_passes(T, pack):
    import torch

    import paper_2510_02345_amd as cm
    cfg = ci.small_config("wide passes", T=T, d=2112, d_ff=8000, G=3, K=2, r=8, k=2, q=32, seed=T)
    print(f"case {cfg}", flush=True)
    w = ci.generate(cfg)
    ref = orc.forward_naive(w, w["x"], cfg.K, cfg.k, cfg.q)
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, T, pack=pack)
    x = torch.from_numpy(w["x"]).to("cuda:0")
    o = layer.forward(x)
    yb, s = layer.ffn_forward(x, o["perm"], o["offsets"], o["expert_idx"], o["gate"])
    y2 = layer.combine(yb, s, o["perm"], o["inv_perm"], o["offsets"], o["expert_idx"], o["gate"])
    torch.cuda.synchronize()
    for y in (o["y"], y2):
        m = orc.error_metrics(y.cpu().numpy(), ref["y"])
        assert m["max_over_rms"] <= 1e-2 and m["mean_rel"] <= 2e-3, m
    layer.close()
