"""What a user of the layer has it do, as cases to be timed.

A case is one use of the public entry points at one size:

  forward    one call of `Layer.forward` (route, permute, expert FFNs, combine): serving, from
             one decoded token to the prefill of a whole batch
  multi      one call of `Layer.forward_multi`: the routing variant with several clusters per
             token, a router temperature and cluster-probability scaling
  train      one training step of the layer: forward, backward for the selection it made, and
             the routing statistics (expert loads, centroid EMA, cluster activity)
  compress   construction of the stored form of one FFN matrix from dense experts

Sizes are the layer's configurations and what lies between them.  All inputs are drawn on
the GPU from the seed: x ~ N(0, 1), bases ~ N(0, 1 / fan_in), routers ~ N(0, 1 / d), factors
~ N(0, 0.02^2) in group-quantised INT4; tokens whose routing would hinge on a near-tie are
redrawn, so that index outputs are exact.
"""
import math

import torch

import paper_2510_02345_amd as cm

DEVICE = "cuda:0"
MARGIN = 1e-3      # smallest gap between logits whose order decides an index

# Layer geometries: the five configurations of the layer (without their token counts).
TINY = dict(d=128, d_ff=512, G=2, K=4, r=4, k=1, q=32)
BASE = dict(d=768, d_ff=3072, G=2, K=4, r=8, k=2, q=32)
MID = dict(d=1024, d_ff=4096, G=4, K=4, r=16, k=2, q=64)
LARGE = dict(d=2048, d_ff=8192, G=8, K=8, r=16, k=2, q=64)
WIDE = dict(d=4096, d_ff=14336, G=8, K=8, r=32, k=2, q=128)

# The largest amount of base-product work (tokens x d x d_ff) and of expert elements of a case.
MOST_PRODUCT = 32768 * 2048 * 8192
MOST_EXPERTS = 64 * 8192 * 2048


def listed():
    return [
        # one decoded token of one sequence: launches and latency
        dict(name="decode_1_base", kind="forward", T=1, router="uniform", **BASE),
        # a decode batch on the widest layer: every base matrix crosses HBM once
        dict(name="decode_64_wide", kind="forward", T=64, router="uniform", **WIDE),
        # a decode batch of continuous batching, odd count, several tokens per cluster
        dict(name="decode_203_large", kind="forward", T=203, router="uniform", **LARGE),
        # the smallest configuration, one expert per token
        dict(name="tiny_256", kind="forward", T=256, router="uniform", **TINY),
        # the prompt of one sequence, ragged
        dict(name="prefill_777_mid", kind="forward", T=777, router="uniform", **MID),
        # prefill of a batch of 8 x 512 tokens on the base width
        dict(name="prefill_4096_base", kind="forward", T=4096, router="uniform", **BASE),
        # 16 x 1024 tokens, cluster loads skewed as they are without load balancing
        dict(name="prefill_16384_zipf", kind="forward", T=16384, router="zipf", **MID),
        # 32 x 1024 tokens, the largest call
        dict(name="prefill_32768_large", kind="forward", T=32768, router="uniform", **LARGE),
        # two clusters per token, ragged token count
        dict(name="multi_2500_mid", kind="multi", T=2500, router="uniform", top_g=2, temperature=0.7, scale=True, **MID),
        # a training micro-batch on the base width
        dict(name="train_4096_base", kind="train", T=4096, router="uniform", **BASE),
        # the largest training step
        dict(name="train_32768_large", kind="train", T=32768, router="uniform", **LARGE),
        # first FFN matrix of the large layer from its 64 dense experts
        dict(name="compress_large", kind="compress", **LARGE),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("forward", "forward", "forward", "multi", "train", "compress"))
    g = dict(rng.choice((TINY, BASE, MID, LARGE) if kind == "train" else (BASE, MID, LARGE) if kind == "compress"
                        else (TINY, BASE, MID, LARGE, WIDE)))
    if rng.random() < 0.5:      # widths between the configurations (multiples of 64, not of 256)
        g["d"] = min(max(64 * rng.randint(g["d"] // 128, g["d"] // 64), 128), 4096)
        g["d_ff"] = 64 * rng.randint(2 * g["d"] // 64, min(4 * g["d"], 14336) // 64)
        g["q"] = min(g["q"], 64)
    if rng.random() < 0.3:      # ranks and numbers of experts per token of the other configurations
        g["r"] = rng.choice((4, 8, 16, 32))
        if g["K"] * g["r"] > 256:
            g["r"] = 256 // g["K"]
        g["k"] = rng.choice((1, 2, 4))
    c = dict(kind=kind, **g)
    if kind == "compress":
        c["G"] = rng.randint(1, max(1, min(g["G"], MOST_EXPERTS // (g["K"] * g["d"] * g["d_ff"]))))
        return c
    lo, hi = (128, 32768) if kind == "train" else (1, 32768)
    per = g["d"] * g["d_ff"]
    if kind == "multi":
        c.update(top_g=2, temperature=rng.choice((1.0, 0.7)), scale=rng.random() < 0.5)
        per *= 2
    c["T"] = _log_int(rng, lo, max(lo, min(hi, MOST_PRODUCT // per)))
    c["router"] = rng.choice(("uniform", "uniform", "zipf"))
    return c


# ---------------------------------------------------------------------------- inputs
def _randn(gen, shape, std, dtype=torch.float16):
    return (torch.randn(shape, device=DEVICE, generator=gen, dtype=torch.float32) * std).to(dtype)


def _int4(gen, E, r, L, q):
    """Factor ~ N(0, 0.02^2) as INT4 codes (even element in the low nibble) and FP16 scales."""
    w = _randn(gen, (E, r, L // q, q), 0.02, torch.float32)
    s = (w.abs().amax(-1) / 7.0).half()
    c = torch.round(w / s.float().clamp_min(1e-12)[..., None]).clamp_(-7, 7).to(torch.int32).view(E, r, L) & 15
    return (c[..., 0::2] | (c[..., 1::2] << 4)).to(torch.uint8), s


def _logits(x, w):
    return x.double() @ w.double().t()


def _gap(x, rc, re, bias, K, k, top_g):
    """Smallest gap between logits whose order decides an index of the token."""
    z = _logits(x, rc)
    if bias is not None:
        z = z + bias.double()
    G = z.shape[1]
    zs, zi = z.sort(dim=1, descending=True)
    gap = torch.full((x.shape[0],), math.inf, device=DEVICE, dtype=torch.float64)
    for a in range(min(top_g, G - 1)):
        gap = torch.minimum(gap, zs[:, a] - zs[:, a + 1])
    le = _logits(x, re).view(-1, G, K)
    for a in range(top_g):
        ls = le[torch.arange(x.shape[0], device=DEVICE), zi[:, a]].sort(dim=1, descending=True).values
        for b in range(min(k, K - 1)):
            gap = torch.minimum(gap, ls[:, b] - ls[:, b + 1])
    return gap


def _zipf_bias(x, rc, G):
    """Bias on the cluster logits with which the cluster loads follow Zipf(1)."""
    target = 1.0 / torch.arange(1, G + 1, device=DEVICE, dtype=torch.float64)
    target /= target.sum()
    z = _logits(x, rc)
    bias = torch.zeros(G, device=DEVICE, dtype=torch.float64)
    for _ in range(40):
        load = torch.bincount((z + bias).argmax(1), minlength=G).double() / z.shape[0]
        bias += 0.5 * torch.log(target / load.clamp_min(1e-4))
        bias -= bias.mean()
    return bias.float()


def _dense_experts(gen, c):
    """Experts of a cluster = common base + low-rank part of decaying spectrum + noise."""
    E, out_d, in_d, rank = c["G"] * c["K"], c["d_ff"], c["d"], c["r"] + 8
    W = torch.empty((E, out_d, in_d), dtype=torch.float16, device=DEVICE)
    decay = 0.8 ** torch.arange(rank, device=DEVICE, dtype=torch.float32)
    for g in range(c["G"]):
        B = _randn(gen, (out_d, in_d), in_d ** -0.5, torch.float32)
        for j in range(c["K"]):
            L = (_randn(gen, (out_d, rank), 1.0, torch.float32) * decay) @ _randn(gen, (rank, in_d), 1.0, torch.float32)
            N = _randn(gen, (out_d, in_d), 1.0, torch.float32)
            nb = B.norm()
            W[g * c["K"] + j] = (B + L * (0.2 * nb / L.norm()) + N * (0.002 * nb / N.norm())).half()
    return W


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    if c["kind"] == "compress":
        W = _dense_experts(gen, c)
        return dict(case=c, W=W, omega=_randn(gen, (min(c["r"] + 8, 48), c["d"]), 1.0))
    T, d, f, G, K, r, k, q = (c[n] for n in ("T", "d", "d_ff", "G", "K", "r", "k", "q"))
    E = G * K
    w = dict(router_cluster=_randn(gen, (G, d), d ** -0.5), router_expert=_randn(gen, (E, d), d ** -0.5),
             w1_base=_randn(gen, (G, f, d), d ** -0.5), w2_base=_randn(gen, (G, d, f), f ** -0.5))
    for n, L in (("v1", d), ("u1", f), ("v2", f), ("u2", d)):
        w[n + "_q"], w[n + "_s"] = _int4(gen, E, r, L, q)
    x = _randn(gen, (T, d), 1.0)
    bias = _zipf_bias(x, w["router_cluster"], G) if c["router"] == "zipf" else None
    for _ in range(40):
        bad = (_gap(x, w["router_cluster"], w["router_expert"], bias, K, k, c.get("top_g", 1)) < MARGIN).nonzero()[:, 0]
        if bad.numel() == 0:
            break
        x[bad] = _randn(gen, (bad.numel(), d), 1.0)
    w["cluster_bias"] = bias
    layer = cm.Layer(d, f, G, K, r, k, q, w, T, device=DEVICE)
    layer.drop_canonical_bases()
    s = dict(case=c, layer=layer, x=x)
    if c["kind"] == "multi":
        s["out"] = layer.forward_multi(x, c["top_g"], c["temperature"], c["scale"])   # its buffers, kept for reuse
    else:
        s["out"] = layer.forward_buffers(T)
    if c["kind"] == "train":
        s["dy"] = _randn(gen, (T, d), 1.0)
        s["mu"] = torch.zeros((E, d), dtype=torch.float32, device=DEVICE)
        s["act"] = torch.zeros((G,), dtype=torch.float32, device=DEVICE)
        s["idle"] = torch.zeros((G,), dtype=torch.int32, device=DEVICE)
    return s


# ---------------------------------------------------------------------------- one pass
_FORWARD = ("y", "cluster_id", "expert_idx", "gate", "perm", "inv_perm", "offsets")


def run(state):
    c = state["case"]
    if c["kind"] == "compress":
        o = cm.compress(state["W"], state["omega"], c["G"], c["K"], c["r"], c["q"], n_iter=2)
        return {n: o[n] for n in ("base", "u_q", "u_s", "v_q", "v_s", "report")}
    layer, x = state["layer"], state["x"]
    if c["kind"] == "multi":
        o = layer.forward_multi(x, c["top_g"], c["temperature"], c["scale"], out=state["out"])
        return {n: o[n] for n in _FORWARD}
    o = layer.forward(x, state["out"])
    res = {n: o[n] for n in _FORWARD}
    if c["kind"] == "train":
        res["grads"] = layer.backward(x, state["dy"], o["expert_idx"], o["gate"])
        res["stats"] = layer.route_stats(x, o["perm"], o["offsets"], o["expert_idx"], state["mu"], state["act"],
                                         state["idle"])
        res["mu"] = state["mu"]
    return res


# ---------------------------------------------------------------------------- work and tolerance
def work(case):
    """The method's own operations, and every input read and output written once."""
    c = case
    d, f, G, K, r, k, q = (c[n] for n in ("d", "d_ff", "G", "K", "r", "k", "q"))
    E = G * K
    if c["kind"] == "compress":
        me, sketch = E * f * d, min(r + 8, 48)
        # experts read; base, codes and scales written; six products of the residuals with the sketch
        return {"bytes": 2 * me + 2 * G * f * d + E * r * (f + d) * (0.5 + 2.0 / q), "flops": 6 * 2.0 * me * sketch}
    T = c["T"]
    Tv = T * c.get("top_g", 1)
    # clusters and experts that a uniform router hits
    hit_c = G * (1 - (1 - 1 / G) ** Tv) if G > 1 else 1
    hit_e = E * (1 - (1 - k / E) ** Tv)
    flops = Tv * (4.0 * d * f + k * 4.0 * r * (d + f)) + T * 2.0 * d * (G + K)
    byts = hit_c * 4.0 * d * f + hit_e * 2.0 * r * (d + f) * (0.5 + 2.0 / q) + 2.0 * (G + E) * d + 4.0 * T * d
    if c["kind"] == "train":
        M = T * k
        flops += 10.0 * T * d * f + 2.0 * M * r * (5 * d + 6 * f) + T * k * d
        # dy read, dx written; gradients of bases, factors and router rows written; centroids updated
        byts += 6.0 * T * d + 8.0 * G * d * f + 8.0 * E * r * (d + f) + 4.0 * E * d + 8.0 * E * d
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # FP16 operands and results, FP32 sums; about four times what was measured.  Against the
    # layer in FP64 on the same dequantised weights: y rel 3e-4 .. 4.6e-4, max 1.7e-3 on small
    # cases; gradients rel 3e-4 .. 4.9e-4, max 3.7e-3 (largest cases about twice that).
    if case["kind"] == "compress":
        # the same experts with rows and columns in another order (every sum in another order):
        # scales rel 2e-4, max 1.8e-3; 9e-4 of the code bytes differ (values next to a rounding
        # boundary)
        return {"rel": 1e-3, "max": 2e-2, "differ": 4e-3}
    if case["kind"] == "train":
        return {"rel": 2e-3, "max": 4e-2}
    return {"rel": 1.6e-3, "max": 2e-2}
