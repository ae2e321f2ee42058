"""The calls the library's speed is measured on: their sizes, their inputs, one
pass of each, the work a pass cannot do without, and their results in 64 bits.

A case is a dict of plain values:
  kind      "train" (sru.Stack, forward and backward), "infer" (sru.forward
            without the states and the projections) or "lowrank" (as "train",
            with Wcat = P Q^T)
  layers    layers of the stack (each after the first reads the one below)
  L, B      steps and sequences;  d_in, d  input and hidden width per direction
  dp        rank of the projection ("lowrank" only, else 0)
  direction "fwd", "rev" or "bi"
  dtype     product precision, "fp32" or "bf16"; inference with bf16 products
            holds its weights rounded
  masked    sequences of unequal length, with a padding mask
  linear    the recurrence without v * c in the gates
  reset_new, alpha  the gate variants
  carry     inference starts from the state of an earlier call (c0)
"""

import math

import torch

from paper_1709_02755_amd import sru

DIRECTION = {"fwd": sru.DIR_FWD, "rev": sru.DIR_REV, "bi": sru.DIR_BI}
DTYPE = {"fp32": sru.GEMM_FP32, "bf16": sru.GEMM_BF16}


def _case(name, kind, L, B, d_in, d, dtype, layers=1, dp=0, direction="fwd", masked=False,
          linear=False, reset_new=False, alpha=1.0, carry=False):
    c = dict(kind=kind, L=L, B=B, d_in=d_in, d=d, dtype=dtype, layers=layers, dp=dp,
             direction=direction, masked=masked, linear=linear, reset_new=reset_new, alpha=alpha,
             carry=carry)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small layer evaluated on a short batch: launches and latency
        _case("forward_f32_L32_B4_d128", "infer", 32, 4, 128, 128, "fp32"),
        # generation: one step of a few sequences, the state carried from the
        # step before, the weights held in bf16
        _case("decode_bf16_L1_B8_d1024", "infer", 1, 8, 1024, 1024, "bf16", carry=True),
        # sentence classification: two narrow layers, fp32
        _case("train2_f32_L64_B32_d256", "train", 64, 32, 256, 256, "fp32", layers=2),
        # question answering: an upper bidirectional layer (it reads both
        # directions of the one below), padded passages
        _case("train_f32_bi_masked_L400_B32_d256_128", "train", 400, 32, 256, 128, "fp32",
              direction="bi", masked=True),
        # the same model's first layer with the linear recurrence
        _case("train_f32_bi_linear_masked_L400_B32_d128", "train", 400, 32, 128, 128, "fp32",
              direction="bi", masked=True, linear=True),
        # a wide layer at the interface's default precision
        _case("train_f32_L256_B64_d1024", "train", 256, 64, 1024, 1024, "fp32"),
        # word embeddings of a width that is no multiple of 8, odd batch and
        # length, bidirectional, with the scaled highway and the reset gate
        # on the new state
        _case("train_bf16_bi_masked_L77_B13_d300_200", "train", 77, 13, 300, 200, "bf16",
              direction="bi", masked=True, reset_new=True, alpha=math.sqrt(3.0)),
        # language modelling: the benchmark's six-layer stack as one call
        _case("train6_bf16_L256_B64_d1024", "train", 256, 64, 1024, 1024, "bf16", layers=6),
        # its layer on one GPU's share of the batch under 8-way data parallelism
        _case("train_bf16_L256_B8_d1024", "train", 256, 8, 1024, 1024, "bf16"),
        # a wide layer on a large padded batch
        _case("train_bf16_masked_L128_B128_d2048", "train", 128, 128, 2048, 2048, "bf16",
              masked=True),
        # the benchmark's layer with the projection trick
        _case("lowrank_bf16_L256_B64_d1024_dp512", "lowrank", 256, 64, 1024, 1024, "bf16",
              dp=512),
        # translation: the layer that replaces a Transformer's feed-forward
        # layer, inference
        _case("infer_bf16_L64_B80_d512_2048", "infer", 64, 80, 512, 2048, "bf16"),
    ]


def _products(c):
    """Multiply-adds of the forward products of the whole stack."""
    total = 0
    for d_in, k in _layer_dims(c):
        m, n = c["L"] * c["B"], _ndir(c) * k * c["d"]
        total += m * c["dp"] * (d_in + n) if c["dp"] else m * n * d_in
    return total


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.99))))))


def draw(rng):
    """Any of the kinds, sizes over the whole range; no dearer than the listed
    ones of its precision (six 1024-wide bf16 layers, one fp32 layer)."""
    while True:
        kind = rng.choice(["train", "train", "train", "infer", "infer", "decode", "lowrank"])
        dtype = rng.choice(["fp32", "bf16"])
        if kind == "decode":
            L, B = rng.randint(1, 4), _log_int(rng, 1, 64)
        else:
            L, B = _log_int(rng, 5, 512), _log_int(rng, 1, 128)
        d = _log_int(rng, 48, 2048)
        # model widths are mostly multiples of 64 or of 4, and some are odd
        step = rng.choice([64, 64, 4, 1])
        d = max(step, d // step * step)
        d_in = d if rng.random() < 0.5 else max(4, _log_int(rng, 32, 1024) // step * step)
        dp = 0
        if kind == "lowrank":
            d, d_in = max(8, d // 8 * 8), max(8, d_in // 8 * 8)
            dp = max(8, min(d, d_in) // rng.choice([2, 4]) // 8 * 8)
        c = _case("", "infer" if kind == "decode" else kind, L, B, d_in, d, dtype,
                  layers=1 if kind in ("infer", "decode") else rng.choice([1, 1, 2, 3]), dp=dp,
                  direction=rng.choice(["fwd", "fwd", "rev", "bi"]), masked=rng.random() < 0.4,
                  linear=rng.random() < 0.2, reset_new=rng.random() < 0.3,
                  alpha=rng.choice([1.0, 1.0, math.sqrt(3.0)]),
                  carry=kind == "decode" or (kind == "infer" and rng.random() < 0.3))
        most = 256 * 64 * 3 * 1024 * 1024 * (1 if dtype == "fp32" else 6)
        if _products(c) <= most and L * B * _ndir(c) * d * c["layers"] <= 1 << 26:
            return c


def _ndir(c):
    return 2 if c["direction"] == "bi" else 1


def _layer_dims(c):
    """(d_in, k) of each layer."""
    out, d_in = [], c["d_in"]
    for _ in range(c["layers"]):
        out.append((d_in, 3 if d_in == c["d"] else 4))
        d_in = _ndir(c) * c["d"]
    return out


def _inputs(c, seed):
    """Inputs and parameters as the paper initialises them (weights of variance
    1 / width), on the GPU, from the seed alone."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    L, B, d, nd = c["L"], c["B"], c["d"], _ndir(c)

    def uniform(bound, *shape):
        return (torch.rand(shape, generator=gen, device=dev) * 2 - 1) * bound

    x = torch.randn((L, B, c["d_in"]), generator=gen, device=dev)
    layers = []
    for d_in, k in _layer_dims(c):
        if c["dp"]:
            p = dict(Q=uniform(math.sqrt(3 / d_in), d_in, c["dp"]),
                     P=uniform(math.sqrt(3 / c["dp"]), nd, k, d, c["dp"]))
        else:
            p = dict(W=uniform(math.sqrt(3 / d_in), nd, k, d, d_in))
        p.update(v_f=uniform(0.5, nd, d), v_r=uniform(0.5, nd, d), b_f=uniform(1.0, nd, d),
                 b_r=torch.zeros((nd, d), device=dev))
        layers.append(p)
    mask = None
    if c["masked"]:
        lengths = torch.randint((L + 1) // 2, L + 1, (B,), generator=gen, device=dev)
        lengths[0] = L
        mask = (torch.arange(L, device=dev)[:, None] >= lengths[None, :]).to(torch.uint8)
        mask = mask.contiguous()
    inp = dict(X=x, layers=layers, mask=mask)
    if c["kind"] == "infer":
        inp["c0"] = torch.randn((B, nd * d), generator=gen, device=dev) if c["carry"] else None
        if c["dtype"] == "bf16":
            layers[0]["W"] = layers[0]["W"].to(torch.bfloat16)
    else:
        inp["dH"] = torch.randn((L, B, nd * d), generator=gen, device=dev)
    return inp


def prepare(case, seed):
    c = case
    inp = _inputs(c, seed)
    inp["case"] = c
    inp["options"] = dict(highway_scale=c["alpha"], reset_new=c["reset_new"],
                          linear=c["linear"])
    if c["kind"] != "infer":
        inp["stack"] = sru.Stack(inp["layers"], c["L"], c["B"], c["d_in"], c["d"],
                                 DIRECTION[c["direction"]], DTYPE[c["dtype"]], inp["X"].device,
                                 **inp["options"])
    return inp


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "infer":
        p = s["layers"][0]
        out = sru.forward(s["X"], p["W"], p["v_f"], p["v_r"], p["b_f"], p["b_r"], c0=s["c0"],
                          direction=DIRECTION[c["direction"]], mask=s["mask"],
                          gemm_dtype=DTYPE[c["dtype"]], store_c=False, keep_u=False,
                          **s["options"])
        return {"H": out["H"], "c_last": out["c_last"]}
    st = s["stack"]
    H = st.forward(s["X"], s["mask"])
    dX = st.backward(s["X"], s["dH"], s["mask"])
    names = (("dQ", "dP") if c["dp"] else ("dW",)) + ("dv_f", "dv_r", "db_f", "db_r")
    return {"H": H, "dX": dX,
            "layers": [dict([(n, g[n]) for n in names], c_last=f["c_last"])
                       for f, g in zip(st.fw, st.bw)]}


def work(case):
    """Inputs and parameters read once, results written once, layer by layer;
    the products, and the recurrence's operations per state."""
    c = case
    m, nd, d = c["L"] * c["B"], _ndir(c), c["d"]
    infer = c["kind"] == "infer"
    nbytes = 0
    for d_in, k in _layer_dims(c):
        weights = d_in * c["dp"] + nd * k * d * c["dp"] if c["dp"] else nd * k * d * d_in
        vectors = 4 * (nd * d * 4 + c["B"] * nd * d)
        if infer:
            nbytes += (2 if c["dtype"] == "bf16" else 4) * weights
            nbytes += 4 * m * (d_in + nd * d) + vectors
        else:
            # X, W, dH in and H, dX, dW out
            nbytes += 4 * (2 * weights + 2 * m * (d_in + nd * d)) + 2 * vectors
        nbytes += m if c["masked"] else 0
    states = m * nd * d * c["layers"]
    flops = (2 if infer else 6) * _products(c) + (20 if infer else 60) * states
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """About four times the largest distance to the 64-bit results measured:
    fp32 1.0e-6; bf16 products 0.0031 (0.0044 low-rank) in one layer, 0.0049
    through six."""
    if case["dtype"] == "fp32":
        return {"rel": 4e-6}
    return {"rel": 1.2e-2 if case["layers"] == 1 and not case["dp"] else 2e-2}


def _layer64(c, x, p, mask, c0):
    """One layer step by step in 64 bits: H [L, B, ndir d] and c_last."""
    L, B, d, nd = c["L"], c["B"], c["d"], _ndir(c)
    w = (torch.einsum("ikdp,np->ikdn", p["P"], p["Q"]) if "P" in p else p["W"])
    k = w.shape[1]
    u = (x.reshape(L * B, -1) @ w.reshape(nd * k * d, -1).t()).reshape(L, B, nd, k, d)
    hs, last = [], []
    for i in range(nd):
        reverse = c["direction"] == "rev" or i == 1
        state = c0[:, i * d:(i + 1) * d] if c0 is not None else x.new_zeros((B, d))
        v_f, v_r = (0.0, 0.0) if c["linear"] else (p["v_f"][i], p["v_r"][i])
        h = [None] * L
        ui = [t.unbind(0) for t in u[:, :, i].unbind(2)]
        xi = x.unbind(0) if k == 3 else ui[3]
        for t in range(L - 1, -1, -1) if reverse else range(L):
            f = torch.sigmoid(ui[1][t] + v_f * state + p["b_f"][i])
            new = f * state + (1 - f) * ui[0][t]
            r = torch.sigmoid(ui[2][t] + v_r * (new if c["reset_new"] else state) + p["b_r"][i])
            h[t] = r * new + (1 - r) * c["alpha"] * xi[t]
            if mask is not None:
                pad = mask[t][:, None]
                h[t] = torch.where(pad, torch.zeros_like(h[t]), h[t])
                new = torch.where(pad, state, new)
            state = new
        hs.append(torch.stack(h))
        last.append(state)
    return torch.cat(hs, 2), torch.cat(last, 1)


def exact(case, seed):
    """The paper's equations step by step in 64 bits (gradients by autograd),
    nothing rounded to 16 bits but weights that are held so."""
    c = case
    inp = _inputs(c, seed)
    infer = c["kind"] == "infer"
    mask = None if inp["mask"] is None else inp["mask"].bool()
    x = inp["X"].double().requires_grad_(not infer)
    layers = [{n: t.double().requires_grad_(not infer) for n, t in p.items()}
              for p in inp["layers"]]
    if infer:
        c0 = None if inp["c0"] is None else inp["c0"].double()
        H, last = _layer64(c, x, layers[0], mask, c0)
        return {"H": H, "c_last": last}
    h, lasts = x, []
    for p in layers:
        h, last = _layer64(c, h, p, mask, None)
        lasts.append(last)
    h.backward(inp["dH"].double())
    names = (("Q", "P") if c["dp"] else ("W",)) + ("v_f", "v_r", "b_f", "b_r")
    return {"H": h.detach(), "dX": x.grad,
            "layers": [dict([("d" + n, None if c["linear"] and n[0] == "v" else p[n].grad)
                             for n in names], c_last=last.detach())
                       for p, last in zip(layers, lasts)]}
