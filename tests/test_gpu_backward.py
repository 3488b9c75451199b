"""GPU parity of cmoe_backward (through the C ABI) against the FP64 oracle's dense chain rule.

The selection (expert_idx, gate) is the oracle's, frozen.  Bar per gradient tensor:
max|g - g_ref| <= 2e-2 * RMS(g_ref) (twice the forward bar: a weight gradient of a sparsely
hit expert is a sum over few rows, its RMS is taken over many zeros) and
sum|g - g_ref| / sum|g_ref| <= 2e-3 (the forward bar).
"""
import numpy as np
import pytest

import cmoe_inputs as ci
from oracle import cmoe_oracle as orc

pytestmark = pytest.mark.gpu

NAMES = ("dx", "d_router_expert", "dw1_base", "dw2_base", "du1", "dv1", "du2", "dv2")


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _run(cfg, w=None, dy_scale=1.0, pack=True, drop_canonical=False, selection=None):
    import torch
    import paper_2510_02345_amd as cm
    print(f"case {cfg}", flush=True)
    w = w if w is not None else ci.generate(cfg)
    rng = np.random.default_rng(cfg.seed + 7)
    dy = (dy_scale * rng.standard_normal((cfg.T, cfg.d))).astype(np.float16)
    cid, eidx, gate, _, _ = orc.route(w["x"], w["router_cluster"], w["router_expert"], cfg.K, cfg.k, w["cluster_bias"])
    if selection is not None:
        eidx, gate = selection(eidx, gate)
    ref = orc.backward_naive(w, w["x"], dy, eidx, gate, cfg.K, cfg.q)
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, cfg.T, pack=pack)
    if drop_canonical:
        layer.drop_canonical_bases()
    out = layer.backward(_dev(w["x"]), _dev(dy), _dev(eidx.astype(np.int32)), _dev(gate.astype(np.float32)))
    torch.cuda.synchronize()
    res = {}
    for n in NAMES + ("d_logits",):
        got = out[n].cpu().numpy().astype(np.float64)
        want = ref["dgate_logits" if n == "d_logits" else n]
        assert got.shape == want.shape, n
        assert np.all(np.isfinite(got)), n
        if want.size == 0:
            continue
        if not np.any(want):        # top_k = 1: the gate is constant, its gradient exactly zero
            assert np.abs(got).max() <= 1e-6, n
            continue
        m = orc.error_metrics(got, want)
        print(f"  {n}: max/rms={m['max_over_rms']:.3e} mean_rel={m['mean_rel']:.3e}", flush=True)
        res[n] = m
    for n, m in res.items():
        assert m["max_over_rms"] <= 2e-2, (n, m)
        assert m["mean_rel"] <= 2e-3, (n, m)
    layer.close()
    return out, ref


SMALL = [
    ci.small_config("bw_ragged", T=777, d=128, d_ff=384, G=3, K=4, r=8, k=2, q=32, seed=141),
    ci.small_config("bw_k1", T=300, d=64, d_ff=192, G=2, K=4, r=4, k=1, q=8, seed=142),
    ci.small_config("bw_flat_r32", T=130, d=192, d_ff=256, G=1, K=3, r=32, k=3, q=64, seed=143),
    ci.small_config("bw_sparse", T=19, d=64, d_ff=128, G=16, K=2, r=16, k=2, q=16, seed=144),
    ci.small_config("bw_k4", T=1500, d=128, d_ff=256, G=2, K=8, r=4, k=4, q=32, seed=145),
    ci.small_config("bw_one", T=1, d=64, d_ff=64, G=2, K=2, r=8, k=2, q=8, seed=146),
    # the largest top-k (8 of 32 experts per cluster) and the largest rank panel (K * r = 512)
    ci.small_config("bw_k8_of_32", T=400, d=64, d_ff=128, G=2, K=32, r=4, k=8, q=8, seed=153),
    ci.small_config("bw_max_rank", T=300, d=64, d_ff=128, G=1, K=16, r=32, k=2, q=8, seed=154),
    # the widest model dimension
    ci.small_config("bw_max_d", T=300, d=8192, d_ff=128, G=4, K=2, r=4, k=2, q=128, seed=155),
]


@pytest.mark.parametrize("cfg", SMALL, ids=[c.name for c in SMALL])
def test_backward_small(cfg):
    _run(cfg)


# Every run of an expert's rows holds several batches of 32 (the steady state of the factor-gradient
# kernel), the last one ragged: 16 runs for both widths, 8 for d_ff, 4 for d.
@pytest.mark.parametrize("r", [4, 8, 16, 32])
@pytest.mark.parametrize("T,G,K,d,f", [(2491, 1, 2, 64, 128), (4803, 4, 4, 64, 4096), (4501, 8, 4, 4160, 64)])
def test_backward_long_runs(r, T, G, K, d, f):
    _run(ci.small_config("bw_runs", T=T, d=d, d_ff=f, G=G, K=K, r=r, k=2, q=8, seed=160 + r))


# The middle kernel (top-k <= 2, K * r <= 128): every rank, one and two experts per token, panels of 32, 64, 96 and
# 128 rank rows, hidden widths that are and are not whole chunks of 128 units, clusters of one token, of whole
# and of ragged 32-token tiles, several runs of tiles; k = 3 and K * r = 160 are just beyond it.
@pytest.mark.parametrize("r,K,k", [(4, 32, 2), (4, 8, 1), (8, 12, 2), (8, 16, 1), (16, 8, 2), (16, 4, 2), (16, 8, 1),
                                   (32, 4, 2), (32, 3, 1), (32, 5, 2), (16, 8, 3)])
@pytest.mark.parametrize("T,G,d,f", [(33, 5, 64, 64), (1024, 1, 128, 320), (2113, 2, 64, 1984)])
def test_backward_middle(r, K, k, T, G, d, f):
    _run(ci.small_config("bw_mid", T=T, d=d, d_ff=f, G=G, K=K, r=r, k=k, q=8, seed=170 + r))


def test_backward_infinite_gradients_stay_with_their_expert():
    # one token's dy overflows the products of its own experts: the factor gradients of the other
    # experts, also of those that share its tiles and rank passes, stay finite
    import torch
    import paper_2510_02345_amd as cm
    cfg = ci.small_config("bw_inf", T=200, d=64, d_ff=128, G=1, K=8, r=8, k=2, q=8, seed=156)
    w = ci.generate(cfg)
    dy = np.random.default_rng(3).standard_normal((cfg.T, cfg.d)).astype(np.float16)
    dy[57] = np.float16(6e4)
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, cfg.T)
    x = _dev(w["x"])
    f = layer.forward(x)
    out = layer.backward(x, _dev(dy), f["expert_idx"], f["gate"])
    torch.cuda.synchronize()
    own = set(f["expert_idx"][57].tolist())
    bad = set()
    for n in ("du1", "dv1", "du2", "dv2"):
        bad |= set((~torch.isfinite(out[n])).flatten(1).any(1).nonzero()[:, 0].tolist())
    assert bad and bad <= own, (bad, own)
    layer.close()


@pytest.mark.parametrize("r,K", [(8, 4), (32, 5)])   # the middle kernel's path, and beyond it (K * r = 160)
def test_backward_of_a_token_that_names_an_expert_twice(r, K):
    # the selection is the caller's: both pairs of such a token count
    def selection(eidx, gate):
        eidx = eidx.copy()
        eidx[::2, 1] = eidx[::2, 0]
        return eidx, gate
    _run(ci.small_config("bw_twice", T=150, d=128, d_ff=256, G=2, K=K, r=r, k=2, q=32, factor_std=0.2, seed=158),
         selection=selection)


@pytest.mark.parametrize("factor", ["v1", "u1", "v2", "u2"])
@pytest.mark.parametrize("r,K", [(4, 8), (8, 8), (16, 8), (32, 4), (32, 5)])
def test_backward_factors_that_are_not_finite_stay_with_their_expert(r, K, factor):
    # one expert's scales hold infinities (0 * inf among its values): the tokens of the other experts, also those that
    # share its tiles and its block of 32 rank rows, get the gradients they get without it
    import torch
    import paper_2510_02345_amd as cm
    cfg = ci.small_config("bw_inf_factor", T=120, d=128, d_ff=192, G=2, K=K, r=r, k=2, q=32, seed=159)
    print(f"case {cfg} {factor}", flush=True)
    w = ci.generate(cfg)
    dy = np.random.default_rng(3).standard_normal((cfg.T, cfg.d)).astype(np.float16)
    _, eidx, gate, _, _ = orc.route(w["x"], w["router_cluster"], w["router_expert"], K, cfg.k, w["cluster_bias"])
    ref = orc.backward_naive(w, w["x"], dy, eidx, gate, K, cfg.q)
    e = int(eidx[0, 0])
    w[factor + "_s"] = w[factor + "_s"].copy()
    w[factor + "_s"][e, r // 2, :] = np.float16(np.inf)
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, K, r, cfg.k, cfg.q, w, cfg.T)
    out = layer.backward(_dev(w["x"]), _dev(dy), _dev(eidx.astype(np.int32)), _dev(gate.astype(np.float32)))
    torch.cuda.synchronize()
    own = (eidx == e).any(1)
    assert own.any() and not own.all()
    dx = out["dx"].cpu().numpy()
    assert not np.isfinite(dx[own]).all(1).any()
    m = orc.error_metrics(dx[~own].astype(np.float64), ref["dx"][~own])
    assert m["max_over_rms"] <= 2e-2 and m["mean_rel"] <= 2e-3, m
    # the experts that no token shares with this one
    far = np.setdiff1d(np.unique(eidx[~own]), np.unique(eidx[own]))
    for n in ("du1", "dv1", "du2", "dv2", "d_router_expert"):
        assert bool(torch.isfinite(out[n][far]).all()), n
    other = 1 - e // K
    for n in ("dw1_base", "dw2_base"):
        assert bool(torch.isfinite(out[n][other]).all()), n
    layer.close()


def test_backward_unused_experts_weights_never_used():
    # an expert without a token, in a cluster that has some: its stored factors may hold anything
    cfg = ci.small_config("bw_unused", T=40, d=64, d_ff=128, G=2, K=8, r=8, k=2, q=8, seed=157)
    w = ci.generate(cfg)
    _, eidx, _, _, _ = orc.route(w["x"], w["router_cluster"], w["router_expert"], cfg.K, cfg.k, w["cluster_bias"])
    used = np.unique(eidx)
    w["router_expert"] = w["router_expert"].copy()
    drop = int(used[0])   # an expert that tokens would choose: its routing vector turned away from them
    xm = w["x"].astype(np.float64)
    v = w["router_expert"][drop].astype(np.float64)
    w["x"] = (xm - np.outer(np.maximum(xm @ v, 0) / (v @ v) * 3.0, v)).astype(np.float16)
    cid, eidx, gate, _, _ = orc.route(w["x"], w["router_cluster"], w["router_expert"], cfg.K, cfg.k, w["cluster_bias"])
    unused = sorted(set(range(cfg.G * cfg.K)) - set(np.unique(eidx).tolist()))
    assert any(e // cfg.K in set(cid.tolist()) for e in unused)
    for e in unused:
        for n in ("v1", "u1", "v2", "u2"):
            w[n + "_s"][e] = np.float16(np.nan)
    out, _ = _run(cfg, w)
    for n in ("du1", "dv1", "du2", "dv2"):
        assert not out[n][unused].any()


@pytest.mark.parametrize("r", [4, 8, 32])
def test_backward_reads_no_codes_of_unused_experts(r):
    # their rows are in none of the panels that the call unpacks into its workspace, those of the used ones are
    import torch
    import paper_2510_02345_amd as cm
    cfg = ci.small_config("bw_unread", T=12, d=64, d_ff=128, G=2, K=4, r=r, k=2, q=32, seed=160)
    print(f"case {cfg}", flush=True)
    w = ci.generate(cfg)
    rng = np.random.default_rng(4)
    cid, _, _, _, _ = orc.route(w["x"], w["router_cluster"], w["router_expert"], cfg.K, cfg.k, w["cluster_bias"])
    eidx = (cid[:, None] * cfg.K + np.array([0, 2])).astype(np.int32)     # experts 1 and 3 of a cluster unused
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, cfg.T, pack=False)
    x, dy = _dev(w["x"]), _dev(rng.standard_normal((cfg.T, cfg.d)).astype(np.float16))
    gate = torch.full((cfg.T, 2), 0.5, device="cuda:0")
    layer.backward(x, dy, _dev(eidx), gate)     # sizes the workspace
    layer.bw_ws.zero_()
    layer.backward(x, dy, _dev(eidx), gate)
    torch.cuda.synchronize()
    ws = layer.bw_ws.cpu().numpy().tobytes()
    for n in ("v1", "u2", "v2", "u1"):
        vals = orc.dequant_int4(w[n + "_q"], w[n + "_s"], cfg.q).astype(np.float16)   # [E][r][L]
        for e in range(cfg.G * cfg.K):
            if e // cfg.K not in cid:
                continue
            # rank rows as they are, or the rank values of one element side by side
            row, col = vals[e, 1].tobytes(), np.concatenate([vals[e, :, i] for i in (5,)]).tobytes()
            found = row in ws or (n == "u1" and col in ws)
            assert found == (e % cfg.K in (0, 2)), (n, e)
    layer.close()


def test_backward_gelu_in_single_precision():
    # dL/d(logit) of two experts whose pre-activations are u and 0 at the one hidden unit that dy sees is g_0 g_1 GELU(u) in
    # FP32, g_0 = g_1 = 1/2 without a further rounding: the function over [-9, 9].  GELU'(u) reaches an output only through
    # FP16 (dx = g_0 GELU'(u), as the second expert's base and rank parts cancel).
    import math
    import torch
    import paper_2510_02345_amd as cm
    d, f, r, q = 64, 64, 4, 8
    u = np.concatenate([np.arange(-9, 9, 1 / 256), np.geomspace(1e-4, 9, 400), -np.geomspace(1e-4, 9, 400)]).astype(np.float16)
    T = len(u)
    w = dict(x=np.zeros((T, d), np.float16), router_cluster=np.zeros((1, d), np.float16),
             router_expert=np.zeros((2, d), np.float16), cluster_bias=None, w1_base=np.zeros((1, f, d), np.float16),
             w2_base=np.zeros((1, d, f), np.float16))
    w["x"][:, 0] = u
    w["w1_base"][0, 0, 0] = w["w2_base"][0, 0, 0] = 1
    for n, L in (("v1", d), ("u1", f), ("v2", f), ("u2", d)):
        w[n + "_q"] = np.zeros((2, r, L // 2), np.uint8)
        w[n + "_s"] = np.zeros((2, r, L // q), np.float16)
    w["v1_q"][1, 0, 0], w["v1_s"][1, 0, 0] = 1, 1          # t1 = u for the second expert,
    w["u1_q"][1, 0, 0], w["u1_s"][1, 0, 0] = 15, 1         # h = u - t1 = 0
    dy = np.zeros((T, d), np.float16)
    dy[:, 0] = 1
    layer = cm.Layer(d, f, 1, 2, r, 2, q, w, T)
    eidx = np.tile(np.array([0, 1], np.int32), (T, 1))
    out = layer.backward(_dev(w["x"]), _dev(dy), _dev(eidx), torch.full((T, 2), 0.5, device="cuda:0"))
    torch.cuda.synchronize()
    x = u.astype(np.float64)
    phi = np.array([0.5 * math.erfc(-v / math.sqrt(2)) for v in x])
    err = np.abs(4.0 * out["d_logits"][:, 0].cpu().numpy().astype(np.float64) - x * phi)
    print(f"  gelu: max error {err.max():.3e}", flush=True)
    # u Phi(u): Phi to 3.2e-7 and the product's rounding, at most 3.9e-7 together
    assert (err <= np.minimum(3.9e-7, 3.2e-7 * np.abs(x) + 2.0 ** -24 * np.abs(x * phi))).all()
    grad = phi + x * np.exp(-x * x / 2) / math.sqrt(2 * math.pi)
    got = 2.0 * out["dx"][:, 0].cpu().numpy().astype(np.float64)
    # the sum of dh in FP16, GELU'(u) / 2 + 1 / 4; q = -1 / 4
    assert (np.abs(got - grad) <= 2 * 2.0 ** -11 * (np.abs(grad) / 2 + 0.25) + 1e-6).all(), np.abs(got - grad).max()
    layer.close()


def test_backward_writes_nothing_behind_its_workspace():
    # exactly the stated bytes, and behind them what must stay as it is; a call of fewer tokens on the same buffer
    import torch
    import paper_2510_02345_amd as cm
    for K, r, k, T in ((4, 16, 2, 530), (4, 16, 1, 97), (5, 32, 2, 300), (8, 4, 4, 300)):
        cfg = ci.small_config("bw_guard", T=T, d=128, d_ff=1024, G=3, K=K, r=r, k=k, q=32, seed=161)
        print(f"case {cfg}", flush=True)
        w = ci.generate(cfg)
        layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, K, r, k, cfg.q, w, T)
        need = cm.lib().cmoe_backward_workspace_bytes(layer._h, T)
        buf = torch.full((need + (1 << 20),), 0x5a, dtype=torch.uint8, device="cuda:0")
        dy = _dev(np.random.default_rng(5).standard_normal((T, cfg.d)).astype(np.float16))
        x = _dev(w["x"])
        sel = layer.forward(x)
        for n in (T, T - 4, T // 2, 1):
            layer.bw_ws = buf[:need]
            out = layer.backward(x[:n], dy[:n], sel["expert_idx"][:n], sel["gate"][:n])
            torch.cuda.synchronize()
            assert layer.bw_ws.data_ptr() == buf.data_ptr() and layer.bw_ws.numel() == need
            assert bool((buf[need:] == 0x5a).all())
            assert all(bool(torch.isfinite(v).all()) for v in out.values())
        layer.close()


def test_backward_config1():
    _run(ci.config(1))


def test_backward_canonical_bases_without_the_packed_copy():
    _run(SMALL[0], pack=False)


@pytest.mark.parametrize("cfg", [SMALL[0], SMALL[8]], ids=lambda c: c.name)
def test_backward_packed_copy_as_the_only_resident_bases(cfg):
    # w1_base / w2_base freed and passed as NULL after packing: the transposed operands and the
    # forward base product of the backward pass are all built from the packed buffer
    _run(cfg, drop_canonical=True)


def test_backward_live_residual_and_gate_path():
    # factors ten times larger and a sharper router: the low-rank terms and the gate path are
    # far above the tolerance, so dropping either would fail
    cfg = ci.small_config("bw_bigres", T=500, d=128, d_ff=512, G=2, K=4, r=8, k=2, q=32, factor_std=0.2, seed=147)
    w = ci.generate(cfg)
    out, ref = _run(cfg, w)
    cid, eidx, gate, _, _ = orc.route(w["x"], w["router_cluster"], w["router_expert"], cfg.K, cfg.k, w["cluster_bias"])
    w0 = dict(w)
    for n in ("u1", "u2"):
        w0[n + "_s"] = np.zeros_like(w[n + "_s"])
    rng = np.random.default_rng(cfg.seed + 7)
    dy = rng.standard_normal((cfg.T, cfg.d)).astype(np.float16)
    ref0 = orc.backward_naive(w0, w["x"], dy, eidx, gate, cfg.K, cfg.q)
    assert orc.error_metrics(ref0["dx"], ref["dx"])["max_over_rms"] > 0.2
    assert np.sqrt((ref["dgate_logits"] ** 2).mean()) > 1e-2


def test_backward_empty_cluster_weights_never_read():
    cfg = ci.small_config("bw_onecluster", T=200, d=64, d_ff=128, G=2, K=4, r=8, k=2, q=8, seed=148)
    w = ci.generate(cfg)
    w["cluster_bias"] = np.array([-100.0, 100.0], dtype=np.float32)
    for n in ("w1_base", "w2_base"):
        w[n][0] = np.float16(np.nan)
    for n in ("v1", "u1", "v2", "u2"):
        w[n + "_s"][:cfg.K] = np.float16(np.nan)
    out, ref = _run(cfg, w)
    for n in ("dw1_base", "dw2_base"):
        assert not out[n][0].any()
    for n in ("du1", "dv1", "du2", "dv2", "d_router_expert"):
        assert not out[n][:cfg.K].any()


@pytest.mark.parametrize("G,K", [(2, 2), (20, 8)])
def test_backward_no_tokens_gives_zero_gradients(G, K):
    import torch
    import paper_2510_02345_amd as cm
    cfg = ci.small_config("bw_empty", T=0, d=64, d_ff=128, G=G, K=K, r=8, k=2, q=8, seed=149)
    w = ci.generate(cfg)
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, 16)
    e = torch.empty((0, cfg.k), dtype=torch.int32, device="cuda:0")
    out = layer.backward(torch.empty((0, cfg.d), dtype=torch.float16, device="cuda:0"),
                         torch.empty((0, cfg.d), dtype=torch.float16, device="cuda:0"), e, e.float())
    torch.cuda.synchronize()
    for n in NAMES[1:]:
        assert not out[n].any(), n
    layer.close()


def test_backward_is_deterministic():
    import torch
    import paper_2510_02345_amd as cm
    cfg = ci.small_config("bw_det", T=1500, d=128, d_ff=512, G=3, K=4, r=16, k=2, q=32, seed=150)
    w = ci.generate(cfg)
    rng = np.random.default_rng(5)
    dy = _dev(rng.standard_normal((cfg.T, cfg.d)).astype(np.float16))
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, cfg.T)
    x = _dev(w["x"])
    f = layer.forward(x)
    a = layer.backward(x, dy, f["expert_idx"], f["gate"])
    torch.cuda.synchronize()
    a = {n: v.clone() for n, v in a.items()}
    layer.bw_ws.fill_(0x7f)
    b = layer.backward(x, dy, f["expert_idx"], f["gate"])
    torch.cuda.synchronize()
    for n in a:
        assert torch.equal(a[n], b[n]), n
    layer.close()


def test_backward_more_than_64_experts():
    # 160 and 128 experts: rank products in slices of 64 experts
    _run(ci.small_config("bw_many", T=400, d=64, d_ff=128, G=20, K=8, r=4, k=2, q=8, seed=151))
    _run(ci.small_config("bw_many_clusters", T=3000, d=64, d_ff=128, G=64, K=2, r=8, k=2, q=16, seed=152))


def _sampled(cfg, clusters, n_tok, hidden, seed=0):
    """Full-size run; dx and d_logits checked on sampled tokens of a few clusters, the weight
    gradients on sampled hidden units (rows of dW1, columns of dW2) over every expert."""
    import torch
    import paper_2510_02345_amd as cm
    print(f"case {cfg}", flush=True)
    w = ci.generate(cfg)
    rng = np.random.default_rng(cfg.seed + 7)
    dy = rng.standard_normal((cfg.T, cfg.d)).astype(np.float16)
    cid, eidx, gate, _, _ = orc.route(w["x"], w["router_cluster"], w["router_expert"], cfg.K, cfg.k, w["cluster_bias"])
    pool = np.nonzero(np.isin(cid, clusters))[0]
    tokens = np.sort(np.random.default_rng(seed).choice(pool, size=min(n_tok, len(pool)), replace=False))
    hidden = np.asarray(hidden)
    ref = orc.backward_sampled(w, w["x"], dy, eidx, gate, cfg.K, cfg.q, tokens, hidden)
    print("oracle done", flush=True)
    layer = cm.Layer(cfg.d, cfg.d_ff, cfg.G, cfg.K, cfg.r, cfg.k, cfg.q, w, cfg.T)
    out = layer.backward(_dev(w["x"]), _dev(dy), _dev(eidx.astype(np.int32)), _dev(gate.astype(np.float32)))
    torch.cuda.synchronize()
    ti, hi = _dev(tokens), _dev(hidden)
    got = dict(dx=out["dx"][ti], dgate_logits=out["d_logits"][ti], dw1_base=out["dw1_base"][:, hi, :],
               dw2_base=out["dw2_base"][:, :, hi], du1=out["du1"][:, :, hi], dv2=out["dv2"][:, :, hi])
    for n in NAMES[1:]:
        assert bool(torch.isfinite(out[n]).all()), n
    for n, g in got.items():
        m = orc.error_metrics(g.cpu().numpy().astype(np.float64), ref[n])
        print(f"  {n}: max/rms={m['max_over_rms']:.3e} mean_rel={m['mean_rel']:.3e}", flush=True)
        assert m["max_over_rms"] <= 2e-2, (n, m)
        assert m["mean_rel"] <= 2e-3, (n, m)
    layer.close()


def test_backward_config2_zipf_loads_sampled():
    _sampled(ci.config(2), clusters=[0, 3], n_tok=64, hidden=[0, 1, 2047, 2048, 4095])


def test_backward_config3_sampled():
    _sampled(ci.config(3), clusters=[2, 7], n_tok=64, hidden=[0, 255, 256, 4097, 8191])


def test_backward_config4_weight_bound_sampled():
    # 64 tokens, every cluster hit, r = 32: tokens of one cluster, a few hidden units
    _sampled(ci.config(4), clusters=[5], n_tok=8, hidden=[0, 1023, 1024, 14335])
