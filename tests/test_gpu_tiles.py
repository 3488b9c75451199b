"""The grouped products' tile shapes: launches whose tiles per XCD (32 CUs) are below half a round,
between, and above, or full rounds plus each kind of leftover, with ragged row tiles; one and
several experts per token, rank panels in LDS and in memory."""
import numpy as np
import pytest

import cmoe_inputs as ci
from oracle import cmoe_oracle as orc

pytestmark = pytest.mark.gpu


# With d_ff = 2048 (8 column tiles) an XCD gets about T / 256 + G / 2 tiles of the up-projection.
@pytest.mark.parametrize("T", [1500, 3300, 5800, 8300, 10900, 13300])
@pytest.mark.parametrize("K,r,k", [(4, 8, 2), (2, 16, 1), (8, 32, 3)])
def test_up_projection_tiles(T, K, r, k):
    _check(ci.small_config("tiles", T=T, d=64, d_ff=2048, G=3, K=K, r=r, k=k, q=32, seed=T + K))


# factor panels and tokens that follow the operands through the stages: one to four portions of 32 rank rows behind
# contractions of two, four and more blocks, rows of t1 of 8 to 64 bytes that start at any multiple of them, a ragged last
# column tile; whole tiles, halves and quarters
@pytest.mark.parametrize("T", [301, 2999, 5801, 13301])
@pytest.mark.parametrize("d,K,r,k", [(64, 4, 4, 1), (128, 16, 4, 2), (64, 3, 32, 2), (192, 8, 16, 2), (256, 4, 32, 1)])
def test_up_projection_panels(T, d, K, r, k):
    _check(ci.small_config("panels", T=T, d=d, d_ff=1344, G=3, K=K, r=r, k=k, q=32, factor_std=0.2, seed=T + K))


# the same with panels too large for LDS, and one to three experts a token: whole tiles with and without groups of 16 rows that no token
# fills, halves, slabs, a ragged last column tile
@pytest.mark.parametrize("T", [301, 2999, 5801, 13301])
@pytest.mark.parametrize("d,K,r,k", [(64, 8, 32, 2), (128, 16, 16, 1), (64, 9, 16, 2), (64, 32, 8, 3)])
def test_up_projection_panels_in_memory(T, d, K, r, k):
    _check(ci.small_config("panels", T=T, d=d, d_ff=1344, G=3, K=K, r=r, k=k, q=32, factor_std=0.2, seed=T + K))


# the same for the down-projection: d = 1088 is four column tiles and a quarter of one
@pytest.mark.parametrize("T", [700, 2000, 4700, 9000, 14000])
def test_down_projection_tiles(T):
    _check(ci.small_config("tiles2", T=T, d=1088, d_ff=192, G=2, K=4, r=8, k=2, q=32, seed=T))


# parts of its contraction: one or two tiles per XCD in quarters of two, four and eight parts (50 to 96 blocks of it, parts
# of equal and of unequal length; small groups with four tiles on an XCD from 64 on), groups that fill only the upper quarters, up to four and more tiles per XCD, one
# after a full round; contractions that stay whole; and the same calls with a workspace that holds no parts
@pytest.mark.parametrize("T,G,d_ff", [(300, 2, 2112), (400, 4, 1024), (500, 4, 2112), (1000, 8, 1088), (1400, 2, 2112),
                                      (2000, 3, 1024), (13000, 1, 512), (400, 4, 1600), (400, 4, 1536), (300, 6, 1984), (300, 6, 2048), (1000, 8, 1856),
                                      (2000, 3, 1792), (13000, 1, 1792), (300, 2, 2560), (300, 1, 2496), (600, 2, 3072)])
def test_down_projection_parts(T, G, d_ff):
    cfg = ci.small_config("parts", T=T, d=1088, d_ff=d_ff, G=G, K=4, r=8, k=2, q=32, seed=T)
    _check(cfg)
    _check(cfg, drop=4 * 256 * 128 * 128 + 4 * 256)


# the residual of the second matrix as more blocks of that contraction: one, three and four blocks of rank rows, wider than
# the output, behind contractions of the fewest blocks and of an odd number, in whole tiles, halves, quarters and
# parts; factors ten times the usual size, so that it is a large share of y
@pytest.mark.parametrize("T,d,d_ff,G,K,r,k", [(300, 64, 192, 2, 4, 32, 2), (300, 64, 256, 2, 4, 32, 2), (700, 1088, 256, 2, 3, 32, 3),
                                              (2000, 1088, 288 + 32, 2, 8, 4, 2), (4700, 576, 320, 2, 8, 16, 2),
                                              (9000, 1088, 320, 2, 4, 8, 1), (500, 1088, 2112, 4, 8, 16, 2),
                                              (300, 1088, 2112, 2, 3, 32, 2)])
def test_down_projection_residual(T, d, d_ff, G, K, r, k):
    cfg = ci.small_config("residual", T=T, d=d, d_ff=d_ff, G=G, K=K, r=r, k=k, q=32, factor_std=0.2, seed=T + d)
    _check(cfg)
    _check(cfg, pack=False)


# A scale that is not finite: of the tokens that did not select its expert, only those in the same block of 16 rows
# can see it, and rows are ordered by expert: at most 15 on either side of the expert's rows in a cluster.
@pytest.mark.parametrize("bad", [np.inf, np.nan, 6e4])
@pytest.mark.parametrize("T,d_ff", [(500, 2112), (5000, 320)])
def test_down_projection_scale_not_finite(bad, T, d_ff):
    import torch

    import paper_2510_02345_amd as cm
    cfg = ci.small_config("bad scale", T=T, d=576, d_ff=d_ff, G=2, K=4, r=32, k=1, q=32, seed=T)
    print(f"case {cfg}", flush=True)
    w = ci.generate(cfg)
    ref = orc.forward_naive(w, w["x"], cfg.K, cfg.k, cfg.q)
    w["u2_s"] = w["u2_s"].copy()
    w["u2_s"][1] = bad
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, cfg.T)
    y = layer.forward(torch.from_numpy(w["x"]).to("cuda:0"))["y"].cpu().numpy()
    other = ref["expert_idx"][:, 0] != 1
    seen = other & ~np.isfinite(y).all(axis=1)
    assert not np.isfinite(y[~other]).all(axis=1).any() and seen.sum() <= 30
    m = orc.error_metrics(y[other & ~seen], ref["y"][other & ~seen])
    assert m["max_over_rms"] <= 1e-2 and m["mean_rel"] <= 2e-3, m
    layer.close()


def _check(cfg, drop=0, pack=True):
    import torch

    import paper_2510_02345_amd as cm
    print(f"case {cfg}", flush=True)
    w = ci.generate(cfg)
    ref = orc.forward_naive(w, w["x"], cfg.K, cfg.k, cfg.q)
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, cfg.T, pack=pack)
    layer.ws = layer.ws[:layer.ws.numel() - drop]
    out = layer.forward(torch.from_numpy(w["x"]).to("cuda:0"))
    torch.cuda.synchronize()
    m = orc.error_metrics(out["y"].cpu().numpy(), ref["y"])   # the layer's bars (FP16 operands and results)
    assert m["max_over_rms"] <= 1e-2 and m["mean_rel"] <= 2e-3, m
    layer.close()
