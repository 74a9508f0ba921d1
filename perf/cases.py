"""Performance cases of the GBLA library: what its users run, over the sizes they run it at.

Three entry points carry the use: ``gbla.forward`` (attention over projected
tensors, dense batches or packed ragged ones), ``gbla.backward`` (the training
step's gradients of the same pass) and ``gbla.layer_forward`` (the whole layer
from the embeddings).  The listed cases take the repository's own workloads
(``paper_2606_07317_amd/inputs.py``) and the neighbouring uses that its tests
cover: fp32 inputs, short histories packed together, small layers.  ``draw``
gives further cases of the same ranges: every head dim, both data types, conv
widths 1 to 4 and the ablation switches.

A case is a dict of plain values:
  kind      "forward", "backward" or "layer"
  layout    "dense" (batch x seqlen) or "ragged" (batch sequences whose lengths
            are lognormal(len_mu, len_sigma) within [len_min, len_max])
  heads, head_dim, conv_width, dtype ("bf16" / "f32"), flags (gbla.NO_*)
  d_model   layers only
  lengths_seed  ragged only: seeds the lengths, so that a case's size (and so
            its work) does not change with the seed of its inputs
"""
import math

import numpy as np
import torch

from paper_2606_07317_amd import gbla

EPS = 1e-6


def listed():
    return [
        # The smallest call: one short fp32 history, two heads (the parity
        # workload tiny_f32).  Launches and host time are all there is.
        _dense("fwd_f32_b1_n256_d32", "forward", 1, 256, 2, 32, dtype="f32"),
        # A serving batch of eight histories of ordinary length.
        _dense("fwd_bf16_b8_n2048_d64", "forward", 8, 2048, 8, 64),
        # One long history, the throughput workload.
        _dense("fwd_bf16_b1_n32768_d64", "forward", 1, 32768, 8, 64),
        # Full-precision inference on odd-length histories.
        _dense("fwd_f32_b2_n8191_d64", "forward", 2, 8191, 8, 64, dtype="f32"),
        # Packed histories of very different lengths, wide heads (the workload
        # ragged64_d128).
        _ragged("fwd_bf16_ragged64_d128", "forward", 64, 7.5, 1.0, 16, 32768, 8, 128),
        # Many short histories packed together, from a single item upwards.
        _ragged("fwd_bf16_ragged256_short_d64", "forward", 256, 4.5, 1.0, 1, 2048, 8, 64),
        # The training step's gradients on one long history.
        _dense("bwd_bf16_b1_n32768_d64", "backward", 1, 32768, 8, 64),
        # ... on a packed batch with wide heads.
        _ragged("bwd_bf16_ragged16_d128", "backward", 16, 7.5, 1.0, 16, 32768, 8, 128),
        # ... in full precision on a small batch of odd-length histories.
        _dense("bwd_f32_b4_n999_d32", "backward", 4, 999, 4, 32, dtype="f32"),
        # The whole layer of the paper's latency table at its shortest and its
        # longest history: batch 8, width 1024, 16 heads of 64.
        _dense("layer_b8_n2048_d1024", "layer", 8, 2048, 16, 64, d_model=1024),
        _dense("layer_b8_n32768_d1024", "layer", 8, 32768, 16, 64, d_model=1024),
        # A small layer on a packed batch of short and middling histories.
        _ragged("layer_ragged24_d256", "layer", 24, 5.5, 1.0, 1, 4096, 4, 64, d_model=256),
    ]


def draw(rng):
    # The kinds and layouts in the shares of the listed cases; sizes uniform in
    # their logarithm, from the smallest listed to no more work than the largest.
    kind = rng.choice(["forward"] * 6 + ["backward"] * 3 + ["layer"] * 3)
    d = rng.choice([32, 64, 64, 64, 128])
    heads = rng.choice([1, 2, 3, 4, 8, 8, 12, 16])
    dtype = "bf16" if kind == "layer" or rng.random() < 0.7 else "f32"
    width = rng.choice([4, 4, 4, 3, 2, 1])
    flags = 0
    if kind != "layer" and rng.random() < 0.25:
        flags = rng.choice([gbla.NO_GATE, gbla.NO_CONV, gbla.NO_NORM, gbla.BLA])
    d_model = rng.choice([128, 192, 256, 512, 768, 1024]) if kind == "layer" else 0
    # tokens x heads x head_dim of the pass (tokens x width for a layer)
    top = {"forward": 2.0 ** 26, "backward": 2.0 ** 24, "layer": 2.0 ** 26}[kind]
    per_token = max(heads * d, d_model)
    tokens = int(math.exp(rng.uniform(math.log(200.0), math.log(top / per_token))))
    if rng.random() < 0.4:
        batch = int(math.exp(rng.uniform(math.log(2.0), math.log(256.0))))
        mean = max(2.0, tokens / batch)
        sigma = rng.choice([0.5, 1.0])
        case = _ragged(None, kind, batch, math.log(mean) - sigma * sigma / 2, sigma, 1,
                       max(16, int(8 * mean)), heads, d, width, dtype, flags, d_model,
                       rng.randrange(1 << 20))
    else:
        batch = min(tokens, int(math.exp(rng.uniform(0.0, math.log(16.0)))))
        case = _dense(None, kind, batch, max(1, tokens // batch), heads, d, width, dtype, flags,
                      d_model)
    del case["name"]
    return case


def _dense(name, kind, batch, seqlen, heads, d, width=4, dtype="bf16", flags=0, d_model=0):
    return dict(name=name, kind=kind, layout="dense", batch=batch, seqlen=seqlen, heads=heads,
                head_dim=d, conv_width=width, dtype=dtype, flags=flags, d_model=d_model)


def _ragged(name, kind, batch, mu, sigma, lo, hi, heads, d, width=4, dtype="bf16", flags=0,
            d_model=0, lengths_seed=4):
    return dict(name=name, kind=kind, layout="ragged", batch=batch, len_mu=mu, len_sigma=sigma,
                len_min=lo, len_max=hi, heads=heads, head_dim=d, conv_width=width, dtype=dtype,
                flags=flags, d_model=d_model, lengths_seed=lengths_seed)


def _lengths(case):
    """Length of every sequence of the batch."""
    if case["layout"] == "dense":
        return [case["seqlen"]] * case["batch"]
    rng = np.random.Generator(np.random.PCG64(case["lengths_seed"]))
    raw = rng.lognormal(case["len_mu"], case["len_sigma"], case["batch"])
    return [int(x) for x in np.clip(np.rint(raw), case["len_min"], case["len_max"])]


def _inputs(case, seed):
    """Tensors of the case on the GPU, from the seed alone: standard-normal
    activations (rounded to bf16 for bf16 cases), taps near the identity conv,
    a norm weight near one."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def randn(*shape, dtype=torch.float32, scale=1.0):
        x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
        return x.mul_(scale).to(dtype)

    H, d, W, flags = case["heads"], case["head_dim"], case["conv_width"], case["flags"]
    lengths = _lengths(case)
    t = {"cu": None, "max_seqlen": None}
    if case["layout"] == "ragged":
        t["cu"] = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32,
                               device="cuda")
        t["max_seqlen"] = max(lengths)
    t["gamma"] = 1.0 + 0.1 * randn(H, d)
    if case["kind"] == "layer":
        m = case["d_model"]
        rows = (sum(lengths),) if t["cu"] is not None else (case["batch"], case["seqlen"])
        t["x"] = randn(*rows, m, dtype=dt)
        t["w_proj"] = randn(H * (4 * d + 1), m, dtype=dt, scale=m ** -0.5)
        t["conv_x"] = 0.1 * randn(m, W)
        t["conv_x"][:, W - 1] += 1.0
        return t
    rows = (H, sum(lengths)) if t["cu"] is not None else (case["batch"], H, case["seqlen"])
    for n in ("q", "k", "v"):
        t[n] = randn(*rows, d, dtype=dt)
    t["a"] = None if flags & gbla.NO_GATE else randn(*rows, dtype=dt)
    t["r"] = None if flags & gbla.NO_NORM else randn(*rows, d, dtype=dt)
    if flags & gbla.NO_NORM:
        t["gamma"] = None
    t["conv_w"] = None
    if not flags & gbla.NO_CONV:
        t["conv_w"] = 0.1 * randn(3, H, d, W)
        t["conv_w"][..., W - 1] += 1.0
    if case["kind"] == "backward":
        t["dy"] = randn(*rows, d)
    return t


_GRADS = ("dq", "dk", "dv", "da", "dr", "dconv_w", "dgamma")


def prepare(case, seed):
    """The inputs, and the scratch and output buffers that a serving loop or a
    training step keeps from call to call."""
    t = _inputs(case, seed)
    t["kind"], t["flags"] = case["kind"], case["flags"]
    if case["kind"] == "layer":
        shape = gbla.layer_shape(t["x"], t["conv_x"], case["heads"], case["head_dim"], EPS, t["cu"],
                                 t["max_seqlen"])
        nbytes = gbla.layer_workspace_bytes(shape)
        act = ((case["heads"], t["x"].shape[0]) if t["cu"] is not None
               else (case["batch"], case["heads"], case["seqlen"])) + (case["head_dim"],)
    else:
        shape = gbla.make_shape(t["q"], t["conv_w"], EPS, t["cu"], t["max_seqlen"], case["flags"])
        nbytes = (gbla.workspace_bytes(shape) if case["kind"] == "forward"
                  else gbla.backward_workspace_bytes(shape))
        act = t["q"].shape
    t["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    if case["kind"] == "backward":
        t["grads"] = {}
        like = {"dq": t["q"], "dk": t["k"], "dv": t["v"], "da": t["a"], "dr": t["r"],
                "dconv_w": t["conv_w"], "dgamma": t["gamma"]}
        for n in _GRADS:
            if like[n] is not None:
                t["grads"][n] = torch.empty(like[n].shape, dtype=torch.float32, device="cuda")
    else:
        t["out"] = torch.empty(act, dtype=torch.float32, device="cuda")
    return t


def run(state):
    t = state
    if t["kind"] == "layer":
        return gbla.layer_forward(t["x"], t["conv_x"], t["w_proj"], t["gamma"], EPS,
                                  cu_seqlens=t["cu"], max_seqlen=t["max_seqlen"],
                                  workspace=t["workspace"], out=t["out"])
    if t["kind"] == "forward":
        return gbla.forward(t["q"], t["k"], t["v"], t["a"], t["r"], t["conv_w"], t["gamma"], EPS,
                            cu_seqlens=t["cu"], max_seqlen=t["max_seqlen"],
                            workspace=t["workspace"], out=t["out"], flags=t["flags"])
    return gbla.backward(t["q"], t["k"], t["v"], t["a"], t["r"], t["conv_w"], t["gamma"], t["dy"],
                         EPS, cu_seqlens=t["cu"], max_seqlen=t["max_seqlen"],
                         workspace=t["workspace"], grads=t["grads"], flags=t["flags"])


def work(case):
    H, d, W, flags = case["heads"], case["head_dim"], case["conv_width"], case["flags"]
    tokens = sum(_lengths(case))
    e = 2 if case["dtype"] == "bf16" else 4
    th = tokens * H
    cu = 4 * (case["batch"] + 1) if case["layout"] == "ragged" else 0
    if case["kind"] == "layer":
        m, features = case["d_model"], H * (4 * d + 1)
        # x, the weights, taps and gamma once; y once.  The projections, the
        # state and the readout (2 d^2 each a token and head).
        return {"bytes": tokens * m * e + features * m * e + m * W * 4 + H * d * 4 + cu + th * d * 4,
                "flops": 2.0 * tokens * features * m + 2.0 * W * tokens * m + 4.0 * th * d * d}
    gates = 0 if flags & gbla.NO_GATE else 1
    norm = 0 if flags & gbla.NO_NORM else 1
    conv = 0 if flags & gbla.NO_CONV else 1
    params = 4 * (3 * H * d * W * conv + H * d * norm) + cu
    # q, k, v, the logits and the output gate once
    reads = th * ((3 + norm) * d + gates) * e + params
    if case["kind"] == "forward":
        return {"bytes": reads + th * d * 4,
                "flops": 4.0 * th * d * d + 6.0 * W * conv * th * d}
    # backward: dy too; a gradient of every input in fp32.  State, readout,
    # dQh, dS, t and dvt: six products of 2 d^2 a token and head; each conv
    # forward, its transpose and its tap sums.
    writes = th * ((3 + norm) * d + gates) * 4 + params - cu
    return {"bytes": reads + th * d * 4 + writes,
            "flops": 12.0 * th * d * d + 18.0 * W * conv * th * d}


# Four times the errors measured against ``exact`` on the listed cases and 24
# drawn ones ("max": the largest difference over the result's rms, or over the
# value itself where that is larger).  fp32 forward: rel 2.2e-7, max 4.4e-6.
# Gradients (fp32 arithmetic for both input types): rel 5.8e-7 (dq), max 3.5e-5
# (dk).  bf16 forward, whose MFMA operands are rounded to bf16: rel 6.5e-4, max
# 1.3e-2.  Layer, whose projections are stored in bf16: rel 5.5e-3, max 0.116.
def tolerance(case):
    if case["kind"] == "layer":
        return {"rel": 2.2e-2, "max": 0.46}
    if case["kind"] == "backward":
        return {"rel": 2.4e-6, "max": 1.4e-4}
    if case["dtype"] == "bf16":
        return {"rel": 2.6e-3, "max": 5.2e-2}
    return {"rel": 9e-7, "max": 1.8e-5}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by torch operators on whole sequences.
# ---------------------------------------------------------------------------
def _conv(x, w):
    """Causal depthwise conv of x [..., n, c] along n with taps w [..., c, W];
    tap W - 1 multiplies the current token."""
    n, W = x.shape[-2], w.shape[-1]
    y = x * w[..., None, :, W - 1]
    for s in range(1, min(W, n)):
        y = torch.cat([y[..., :s, :], y[..., s:, :] + x[..., :n - s, :] * w[..., None, :, W - 1 - s]],
                      dim=-2)
    return y


def _phi(u):
    return torch.where(u > 0, u + 1.0, torch.exp(torch.clamp(u, max=0.0)))


def _attend(q, k, v, a, r, conv_w, gamma):
    """One sequence, all heads: q, k, v, r [H, n, d], a [H, n]."""
    if conv_w is not None:
        q, k, v = (_conv(x, conv_w[i]) for i, x in enumerate((q, k, v)))
    n = q.shape[-2]
    g = torch.softmax(a, dim=-1) if a is not None else torch.full_like(q[..., 0], 1.0 / n)
    kg = _phi(k) * g[..., None]
    S = torch.matmul(kg.transpose(-1, -2), v)
    z = kg.sum(dim=-2)
    fq = _phi(q)
    o = torch.matmul(fq, S) / torch.matmul(fq, z[..., None])
    if gamma is None:
        return o
    oh = o * torch.rsqrt((o * o).mean(dim=-1, keepdim=True) + EPS)
    return oh * gamma[:, None, :] * (r * torch.sigmoid(r))


def _pieces(case):
    """Index of each sequence in the batch: (b,) slices of dense tensors, token
    ranges of ragged ones."""
    lengths = _lengths(case)
    if case["layout"] == "dense":
        return list(range(case["batch"]))
    ends = np.cumsum(lengths)
    return [slice(int(e) - n, int(e)) for e, n in zip(ends, lengths)]


def _take(x, case, at, token_dim):
    if x is None:
        return None
    if case["layout"] == "dense":
        return x[at]
    return x.narrow(token_dim, at.start, at.stop - at.start)


def exact(case, seed):
    t = _inputs(case, seed)
    wide = {n: x.double() if torch.is_tensor(x) and x.is_floating_point() and n not in ("x", "w_proj")
            else x for n, x in t.items()}
    H, d = case["heads"], case["head_dim"]
    if case["kind"] == "layer":
        w = t["w_proj"].double()
        ys = []
        for at in _pieces(case):
            xt = _conv(_take(t["x"], case, at, 0).double(), wide["conv_x"])
            p = torch.matmul(xt, w.t())
            n = xt.shape[0]
            q, k, v, r = (p[:, i * H * d:(i + 1) * H * d].reshape(n, H, d).transpose(0, 1)
                          for i in range(4))
            ys.append(_attend(q, k, v, p[:, 4 * H * d:].t(), r, None, wide["gamma"]))
        return torch.stack(ys) if case["layout"] == "dense" else torch.cat(ys, dim=1)
    acts = [wide[n] for n in ("q", "k", "v", "a", "r")]
    conv_w, gamma = wide["conv_w"], wide["gamma"]
    if case["kind"] == "forward":
        ys = [_attend(*[_take(x, case, at, 1) for x in acts], conv_w, gamma)
              for at in _pieces(case)]
        return torch.stack(ys) if case["layout"] == "dense" else torch.cat(ys, dim=1)
    params = [p.requires_grad_() if p is not None else None for p in (conv_w, gamma)]
    leaves = [x.requires_grad_() if x is not None else None for x in acts]
    for at in _pieces(case):
        y = _attend(*[_take(x, case, at, 1) for x in leaves], *params)
        (y * _take(wide["dy"], case, at, 1)).sum().backward()
    out = {}
    for n, x in zip(_GRADS, leaves + params):
        if x is not None:
            out[n] = x.grad
    return out

