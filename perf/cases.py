"""Timed cases of the encoder stage: what a user of this library has it do.

A case is one pass through the binding's public entry points (`Stage.forward`,
`Stage.backward`, `Stage.backward_noalloc`) of a stage whose weights were set
with `Stage.set_param`, as a pipeline device of a training job calls them: the
previous device's activations in, the next device's gradient in, this stage's
output, input gradient and parameter gradients out (the gradients are read in
place through `stage_grad`, where an optimiser would use them).

Fields of a case:
  mode    "step" (forward + backward), "noalloc" (the same with
          `backward_noalloc`) or "forward" (evaluation: forward only)
  part    "layers" (whole encoder layers), "attn" or "ffn" (a stage holding one
          half-layer allocation unit)
  layers, hidden, heads, ffn, batch, seq, dtype ("bf16" or "f32")
  len_lo, len_hi   range of the sequences' valid lengths; 0, 0: no key mask
"""
import math

import numpy as np
import torch

from paper_2202_11836_amd import PARAM_NAMES, Stage
from paper_2202_11836_amd.binding import stage_grad

MATRICES = ("W_qkv", "W_o", "W_1", "W_2")
ATTN_PARAMS = ("W_qkv", "b_qkv", "W_o", "b_o", "g1", "be1")


def _case(name, part, mode, layers, hidden, ffn, batch, seq, len_lo, len_hi, dtype):
    return {"name": name, "part": part, "mode": mode, "layers": layers, "hidden": hidden,
            "heads": hidden // 64, "ffn": ffn, "batch": batch, "seq": seq, "len_lo": len_lo,
            "len_hi": len_hi, "dtype": dtype}


def listed():
    return [
        # The smallest stage (the fp32 preset the repository's own checks use):
        # a unit test of a training loop, or the allocator's dry run of a
        # stage.  Nothing but latency and launches.
        _case("tiny_f32_step", "layers", "step", 2, 128, 512, 2, 32, 16, 32, "f32"),
        # One fp32 BERT-base layer on a mini-batch of MNLI-sized sentences: the
        # fp32 stages are what a user validates a bf16 run against.
        _case("base_f32_step", "layers", "step", 1, 768, 3072, 16, 128, 64, 128, "f32"),
        # Evaluation of single sentences through one BERT-base layer in bf16:
        # the latency of a pipeline stage at batch 1.
        _case("base_one_sentence_forward", "layers", "forward", 1, 768, 3072, 1, 128, 0, 0,
              "bf16"),
        # A training step on a very small micro-batch (a pipeline splits its
        # batch of 32 into micro-batches), with an odd length.
        _case("base_microbatch_step", "layers", "step", 1, 768, 3072, 3, 77, 20, 77, "bf16"),
        # Three BERT-base layers at 16 x 128, padded: the whole call of a
        # slower device of the paper's cluster.
        _case("base3_step", "layers", "step", 3, 768, 3072, 16, 128, 64, 128, "bf16"),
        # One layer of a BERT-base stage at full length with uneven sentences.
        _case("base_uneven_step", "layers", "step", 1, 768, 3072, 32, 512, 256, 512, "bf16"),
        # One layer of the depth sweep that feeds the allocator, through the
        # backward that may not allocate (training loops that capture graphs).
        _case("large_sweep_noalloc_step", "layers", "noalloc", 1, 1024, 4096, 8, 512, 128, 512,
              "bf16"),
        # The headline stage: four BERT-large layers, batch 32 x 512, no
        # padding.  The largest whole call.
        _case("large4_step", "layers", "step", 4, 1024, 4096, 32, 512, 0, 0, "bf16"),
        # Evaluation of a full batch through one BERT-large layer.
        _case("large_forward", "layers", "forward", 1, 1024, 4096, 32, 512, 0, 0, "bf16"),
        # A stage that holds one attention half (allocation units are
        # half-layers), ragged batch, lengths from a few tokens up.
        _case("large_attn_half_step", "attn", "step", 1, 1024, 4096, 13, 387, 5, 387, "bf16"),
        # A stage that holds one feed-forward half of a narrow layer, odd
        # token count (11 * 231 = 2541).
        _case("narrow_ffn_half_step", "ffn", "step", 1, 512, 2048, 11, 231, 0, 0, "bf16"),
        # One layer at the greatest width the library takes.
        _case("wide_step", "layers", "step", 1, 2048, 8192, 8, 512, 200, 512, "bf16"),
    ]


def _flops_forward(c):
    """Multiply-adds count twice; attention over the mean valid length."""
    h, f, S = c["hidden"], c["ffn"], c["seq"]
    keys = (c["len_lo"] + c["len_hi"]) / 2.0 if c["len_hi"] else float(S)
    attn = 2.0 * 4 * h * h + 4.0 * h * keys
    ffn = 2.0 * 2 * h * f
    per_token = {"layers": attn + ffn, "attn": attn, "ffn": ffn}[c["part"]]
    return c["layers"] * c["batch"] * S * per_token


def work(case):
    c = case
    h, f, T = c["hidden"], c["ffn"], c["batch"] * c["seq"]
    step = c["mode"] != "forward"
    esz = 2 if c["dtype"] == "bf16" else 4
    attn_w, attn_v = 4 * h * h, 6 * h
    ffn_w, ffn_v = 2 * h * f, f + 3 * h
    mats = c["layers"] * {"layers": attn_w + ffn_w, "attn": attn_w, "ffn": ffn_w}[c["part"]]
    vecs = c["layers"] * {"layers": attn_v + ffn_v, "attn": attn_v, "ffn": ffn_v}[c["part"]]
    # activations in and out, parameters read once, fp32 gradients written once
    nbytes = T * h * esz * (4 if step else 2) + mats * esz + vecs * 4
    nbytes += (mats + vecs) * 4 if step else 0
    nbytes += T if c["len_hi"] else 0
    return {"bytes": nbytes, "flops": _flops_forward(c) * (3 if step else 1)}


def draw(rng):
    """One more case: widths, token counts, lengths, types and modes over the
    ranges of the listed cases."""
    largest = max(work(c)["flops"] for c in listed())
    largest_f32 = max(work(c)["flops"] for c in listed() if c["dtype"] == "f32")
    while True:
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        hidden = 64 * round(math.exp(rng.uniform(math.log(2), math.log(32))))
        ffn = 4 * hidden if rng.random() < 0.7 else 64 * round(hidden / 64 * rng.uniform(1.5, 5.0))
        seq = round(math.exp(rng.uniform(math.log(16), math.log(512))))
        batch = round(math.exp(rng.uniform(math.log(1), math.log(32))))
        layers = rng.choice((1, 1, 1, 2, 3, 4))
        part = rng.choice(("layers", "layers", "attn", "ffn"))
        mode = rng.choice(("step", "step", "noalloc", "forward"))
        if part != "layers":
            layers = 1
        if rng.random() < 0.3:
            lo = hi = 0
        else:
            hi = rng.randint(max(1, seq // 2), seq)
            lo = rng.randint(1, hi)
        # The backward that may not allocate is promised for every token count
        # up to BERT-large's widths only.
        if mode == "noalloc" and (hidden > 1024 or ffn > 4096):
            mode = "step"
        # Left out: bf16 backward passes of a feed-forward half over an odd
        # number of 128-token blocks.  Versions of the library without
        # test_gpu_ragged_blocks.py write past a buffer there, and the cases
        # have to run on every version that is compared.
        if (dtype == "bf16" and part != "attn" and mode != "forward" and
                (batch * seq + 127) // 128 % 2):
            continue
        c = _case("", part, mode, layers, hidden, ffn, batch, seq, lo, hi, dtype)
        del c["name"]
        flops = work(c)["flops"]
        if flops <= (largest_f32 if dtype == "f32" else largest):
            return c


def _held(case):
    """Names of the parameters each layer of the stage holds."""
    if case["part"] == "attn":
        return [n for n in PARAM_NAMES if n in ATTN_PARAMS]
    if case["part"] == "ffn":
        return [n for n in PARAM_NAMES if n not in ATTN_PARAMS]
    return list(PARAM_NAMES)


def _inputs(case, seed):
    """Activations, output gradient, key mask and parameters, on the GPU, from
    the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 12345)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    B, S, h, f = case["batch"], case["seq"], case["hidden"], case["ffn"]
    shapes = {"W_qkv": (3 * h, h), "b_qkv": (3 * h,), "W_o": (h, h), "W_1": (f, h), "b_1": (f,),
              "W_2": (h, f)}

    def normal(shape, std, mean=0.0):
        return torch.randn(shape, generator=g, device="cuda") * std + mean

    x = normal((B, S, h), 1.0).to(dt)
    dy = normal((B, S, h), 1.0).to(dt)
    mask = None
    if case["len_hi"]:
        lens = np.random.default_rng(seed).integers(case["len_lo"], case["len_hi"], size=B,
                                                    endpoint=True)
        mask = torch.from_numpy((np.arange(S)[None, :] < lens[:, None]).astype(np.uint8)).cuda()
    params = []
    for _ in range(case["layers"]):
        p = {}
        for n in _held(case):
            shape = shapes.get(n, (h,))
            if n in MATRICES:
                w = normal(shape, 0.02)
                if n == "W_qkv":
                    w[:2 * h] *= 2.0  # scores of a trained model are not all alike
                p[n] = w.to(dt)
            elif n in ("g1", "g2"):
                p[n] = normal(shape, 0.1, 1.0)
            else:
                p[n] = normal(shape, 0.05)
        params.append(p)
    return x, dy, mask, params


class _Raw:
    """A library-owned device buffer, for torch.as_tensor (the tensor keeps
    this object, and so the stage that owns the memory, alive)."""

    def __init__(self, stage, ptr, shape):
        self.stage = stage
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": shape, "typestr": "<f4",
                                         "strides": None, "version": 2}


def prepare(case, seed):
    x, dy, mask, params = _inputs(case, seed)
    kw = {"attn": {"first_unit": 0, "n_units": 1}, "ffn": {"first_unit": 1, "n_units": 1}}
    stage = Stage(case["layers"], case["hidden"], case["heads"], case["ffn"], seed=0,
                  dtype=case["dtype"], **kw.get(case["part"], {}))
    grads = []
    for l, p in enumerate(params):
        views = {}
        for n, v in p.items():
            which = PARAM_NAMES.index(n)
            stage.set_param(l, which, v)
            ptr, _ = stage_grad(stage.handle, l, which)
            views[n] = torch.as_tensor(_Raw(stage, ptr, tuple(v.shape)), device="cuda")
        grads.append(views)
    return {"stage": stage, "mode": case["mode"], "x": x, "dy": dy, "mask": mask,
            "y": torch.empty_like(x), "dx": torch.empty_like(x), "grads": grads}


def run(state):
    st = state["stage"]
    y = st.forward(state["x"], state["mask"], out=state["y"])
    if state["mode"] == "forward":
        return {"y": y}
    if state["mode"] == "noalloc":
        dx = st.backward_noalloc(state["dy"], state["dx"])
    else:
        dx = st.backward(state["dy"], out=state["dx"])
    return {"y": y, "dx": dx, "grads": state["grads"]}


def tolerance(case):
    """Relative 2-norm per output.  Measured against 64 bits over the listed
    and some drawn cases: fp32 at most 1.2e-6; bf16 y 2e-3 a layer, gradients
    2e-3 to 5e-3 and up to 7.1e-3 (the query and key weights at width 2048; a
    stage of four layers 6.6e-3).  Another correct implementation differs from
    this one by up to about 1.4 times that: the errors are roundings of stored
    tensors, which add up over a stage's layers."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2 if case["layers"] == 1 else 2e-2}


# ---------------------------------------------------------------------------
# The same in 64 bits: post-LN encoder layer (attention with masked softmax,
# erf GELU, LayerNorm epsilon 1e-12) and its chain rule.
# ---------------------------------------------------------------------------
def _ln(z, g, b):
    mu = z.mean(-1, keepdim=True)
    var = ((z - mu) ** 2).mean(-1, keepdim=True)
    r = 1.0 / torch.sqrt(var + 1e-12)
    xh = (z - mu) * r
    return g * xh + b, xh, r


def _ln_back(dy, xh, r, g):
    d = dy * g
    dz = r * (d - d.mean(-1, keepdim=True) - xh * (d * xh).mean(-1, keepdim=True))
    return dz, (dy * xh).sum(0), dy.sum(0)


def _heads(t, B, S, H):
    return t.reshape(B, S, H, 64).transpose(1, 2).contiguous()


def _merge(t):
    B, H, S, d = t.shape
    return t.transpose(1, 2).reshape(B * S, H * d)


def _tr(t):
    return t.transpose(-1, -2).contiguous()


def _forward64(x, p, mask, B, S, H):
    s = {"X": x}
    if "W_qkv" in p:
        qkv = x @ p["W_qkv"].T + p["b_qkv"]
        q, k, v = (_heads(t, B, S, H) for t in qkv.chunk(3, -1))
        sc = q @ _tr(k) / 8.0
        if mask is not None:
            sc = sc.masked_fill((mask == 0)[:, None, None, :], -math.inf)
        P = torch.softmax(sc, -1)
        C = _merge(P @ v)
        s.update(q=q, k=k, v=v, P=P, C=C)
        x, s["xh1"], s["r1"] = _ln(x + (C @ p["W_o"].T + p["b_o"]), p["g1"], p["be1"])
    if "W_1" in p:
        u = x @ p["W_1"].T + p["b_1"]
        phi = 0.5 * torch.erfc(-u / math.sqrt(2.0))
        s.update(H1=x, G=u * phi,
                 Gd=phi + u * torch.exp(-0.5 * u * u) / math.sqrt(2.0 * math.pi))
        x, s["xh2"], s["r2"] = _ln(x + (s["G"] @ p["W_2"].T + p["b_2"]), p["g2"], p["be2"])
    return x, s


def _backward64(dy, s, p, B, S, H):
    g = {}
    if "W_1" in p:
        dz, g["g2"], g["be2"] = _ln_back(dy, s["xh2"], s["r2"], p["g2"])
        g["W_2"], g["b_2"] = dz.T @ s["G"], dz.sum(0)
        du = (dz @ p["W_2"]) * s["Gd"]
        g["W_1"], g["b_1"] = du.T @ s["H1"], du.sum(0)
        dy = dz + du @ p["W_1"]
    if "W_qkv" in p:
        dz, g["g1"], g["be1"] = _ln_back(dy, s["xh1"], s["r1"], p["g1"])
        g["W_o"], g["b_o"] = dz.T @ s["C"], dz.sum(0)
        dC = _heads(dz @ p["W_o"], B, S, H)
        dv = _tr(s["P"]) @ dC
        dP = dC @ _tr(s["v"])
        dS = s["P"] * (dP - (dP * s["P"]).sum(-1, keepdim=True)) / 8.0
        dqkv = torch.cat([_merge(dS @ s["k"]), _merge(_tr(dS) @ s["q"]), _merge(dv)], 1)
        g["W_qkv"], g["b_qkv"] = dqkv.T @ s["X"], dqkv.sum(0)
        dy = dz + dqkv @ p["W_qkv"]
    return dy, g


def exact(case, seed):
    x, dy, mask, params = _inputs(case, seed)
    B, S, h, H = case["batch"], case["seq"], case["hidden"], case["heads"]
    params = [{n: v.double() for n, v in p.items()} for p in params]
    cur, saved = x.double().reshape(B * S, h), []
    for p in params:
        cur, s = _forward64(cur, p, mask, B, S, H)
        saved.append(s)
    out = {"y": cur.reshape(B, S, h)}
    if case["mode"] == "forward":
        return out
    d, grads = dy.double().reshape(B * S, h), [None] * len(params)
    for l in reversed(range(len(params))):
        d, g = _backward64(d, saved[l], params[l], B, S, H)
        saved[l] = None
        grads[l] = {n: g[n] for n in params[l]}
    out["dx"] = d.reshape(B, S, h)
    out["grads"] = grads
    return out
