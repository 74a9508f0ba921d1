"""The channel-layout kernels at the edges of their tiles: 16 tokens a wave in
the fp32 forward, 32 in the backward's split products, units of 64 to 512 (the
backward) or 2048 tokens (the forward) chosen by the batch's size; the one-launch
forward; the layer's conv and gate pass.  Against the fp64 oracles, with the tolerances of test_parity_gpu.py,
test_backward_gpu.py and test_layer_gpu.py.
"""
import numpy as np
import pytest
import torch

from paper_2606_07317_amd import inputs
from tests import test_layer_gpu
from tests.test_backward_gpu import NAMES, TOL, close_scaled, run_backward
from tests.test_parity_gpu import close, say, small

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def G():
    from paper_2606_07317_amd import gbla
    gbla.load_library()
    return gbla


# lengths about the tile (16), the wave's quarter and the unit (64, 128, 256,
# 512), and what a conv window of three earlier tokens sees across each
EDGES = [2, 3, 4, 15, 16, 17, 63, 64, 65, 66, 67, 128, 131, 255, 257, 511, 512, 515]
DIMS = [(32, inputs.F32, 4), (32, inputs.BF16, 3), (64, inputs.F32, 2), (64, inputs.BF16, 4),
        (128, inputs.F32, 4), (128, inputs.BF16, 4)]


def _case(d, dtype, width, seed, **kw):
    return small("ragged64_d128", head_dim=d, dtype=dtype, conv_width=width, seed=seed, **kw)


def backward_unit(work, d):
    """Tokens of the backward's units for `work` tokens x heads: 1024 waves, d / 16
    to a workgroup."""
    unit = 512
    while unit > 64 and work < unit * (1024 // (d // 16)):
        unit //= 2
    return unit


def fp32_state_unit(lengths, heads, d):
    """Tokens of the fp32 forward's state units: about 256 workgroups' share, up to
    d = 64 about 512 workgroups' where the records fit the fixed scratch (d = 64:
    16,896 bytes a record, 20,480 of operands a pair; d = 32: 4352, 6144)."""
    pow2 = lambda x: 1 << max(0, (x - 1).bit_length())
    work = sum(lengths) * heads
    coarse = min(max(256, pow2((work + 255) // 256)), 2048)
    fine = max(64, pow2((work + 511) // 512))
    if d == 128 or fine >= coarse:
        return coarse
    rec, ops = {64: (16896, 20480), 32: (4352, 6144)}[d]
    size = heads * ((sum(lengths) // fine + len(lengths)) * rec + len(lengths) * ops)
    return fine if size <= 16 << 20 else coarse


@pytest.mark.parametrize("unit", [64, 512])
@pytest.mark.parametrize("d,dtype,width", DIMS)
def test_backward_edges(G, dev, d, dtype, width, unit):
    from oracle import gbla_backward
    heads = 1 if unit == 64 else {32: 98, 64: 49, 128: 25}[d]
    assert backward_unit(sum(EDGES) * heads, d) == unit
    say("backward edges", d, dtype, width, heads)
    inp = inputs.make_inputs(_case(d, dtype, width, 51, heads=heads), lengths=EDGES)
    dy = inputs.make_cotangent(inp)
    got = run_backward(G, inp, dy, dev)
    ref = gbla_backward.backward_inputs(inp, dy)
    for n in NAMES:
        close_scaled(got[n], ref[n], TOL[dtype], n)


@pytest.mark.parametrize("d,dtype", [(32, inputs.F32), (64, inputs.BF16), (128, inputs.F32)])
def test_backward_square_overflow(G, dev, d, dtype):
    """Outputs whose squares overflow fp32 have the norm factor 0, and so have all
    the gradients."""
    say("backward, |o|^2 overflows", d, dtype)
    inp = inputs.make_inputs(_case(d, dtype, 4, 57, heads=2), lengths=[40, 3, 130])
    t = inputs.device_tensors(inp, dev)
    dy = torch.from_numpy(inputs.make_cotangent(inp)).to(dev)
    got = G.backward(t["q"], t["k"], t["v"] * 1e25, t["a"], t["r"], t["conv_w"], t["gamma"], dy, eps=inp.eps,
                     cu_seqlens=t["cu_seqlens"], max_seqlen=t["max_seqlen"])
    torch.cuda.synchronize()
    for n in NAMES:
        assert bool((got[n] == 0).all()), n


def test_backward_infinite_inputs_stay_in_their_sequence(G, dev):
    """An infinite value or gradient spoils its own sequence and head only."""
    say("backward, infinite inputs")
    inp = inputs.make_inputs(_case(64, inputs.F32, 4, 62, heads=2), lengths=[40, 33, 70])
    t = inputs.device_tensors(inp, dev)
    dy = torch.from_numpy(inputs.make_cotangent(inp)).to(dev)
    v2, dy2 = t["v"].clone(), dy.clone()
    v2[0, 45, 3] = float("inf")    # second sequence, first head
    dy2[1, 100, 60] = float("inf")  # third sequence, second head
    a, b = (G.backward(t["q"], t["k"], v, t["a"], t["r"], t["conv_w"], t["gamma"], g, eps=inp.eps,
                       cu_seqlens=t["cu_seqlens"], max_seqlen=t["max_seqlen"])
            for v, g in ((t["v"], dy), (v2, dy2)))
    torch.cuda.synchronize()
    for n in ("dq", "dk", "dv", "da", "dr"):
        same = torch.ones(2, 143, dtype=torch.bool, device=dev)
        same[0, 40:73] = same[1, 73:] = False
        assert bool((a[n][same] == b[n][same]).all()), n
        assert not bool(b[n][0, 40:73].isfinite().all()), n


@pytest.mark.parametrize("name", ["q", "k"])
@pytest.mark.parametrize("d,W", [(32, 4), (64, 3), (128, 4)])
def test_backward_infinite_last_token(G, dev, d, W, name):
    """phi of -inf is 0, so a -inf in a sequence's last token leaves finite gradients
    (but the tap's that multiplies it): the tile's tokens past the sequence, whose
    windows hold it too, take no part."""
    from oracle import gbla_backward
    say("backward, infinite last token", d, W, name)
    lengths = [40, 33, 70, 128, 5]
    inp = inputs.make_inputs(_case(d, inputs.F32, W, 63, heads=2), lengths=lengths)
    getattr(inp, name)[0, np.cumsum(lengths) - 1, 3] = -np.inf
    dy = inputs.make_cotangent(inp)
    got = run_backward(G, inp, dy, dev)
    with np.errstate(invalid="ignore"):
        ref = gbla_backward.backward_inputs(inp, dy)
    for n in NAMES:
        nan = np.zeros(ref[n].shape, bool)
        if n == "dconv_w":
            nan["qkv".index(name), 0, 3, W - 1] = True  # 0 * inf
        assert (np.isnan(got[n]) == nan).all() and (np.isnan(ref[n]) == nan).all(), n
        close_scaled(np.where(nan, 0, got[n]), np.where(nan, 0, ref[n]), TOL[inputs.F32], n)


def norm_of_infinite(y):
    """The output where channel 3 of o is infinite: the norm factor is 0."""
    other = [c for c in range(y.shape[-1]) if c != 3]
    assert bool(y[:, 3].isnan().all()) and bool((y[:, other] == 0).all())


@pytest.mark.parametrize("d,dtype", [(32, inputs.F32), (64, inputs.F32), (32, inputs.BF16), (64, inputs.BF16)])
def test_short_forward_infinite_value(G, dev, d, dtype):
    say("short forward, infinite value", d, dtype)
    inp = inputs.make_inputs(_case(d, dtype, 4, 60, heads=1), lengths=[40, 100])
    t = inputs.device_tensors(inp, dev)
    t["v"][0, 45, 3] = float("inf")
    y = G.forward(t["q"], t["k"], t["v"], t["a"], t["r"], t["conv_w"].abs(), t["gamma"], eps=inp.eps,
                  cu_seqlens=t["cu_seqlens"], max_seqlen=100)
    torch.cuda.synchronize()
    assert bool(y[0, :40].isfinite().all())
    norm_of_infinite(y[0, 40:])


@pytest.mark.parametrize("dtype", [inputs.F32, inputs.BF16])
def test_infinite_sums_stay_infinite(G, dev, dtype):
    """A state sum that is infinite in one unit is infinite, not NaN, over several:
    an infinite value leaves the other channels of the norm's output zero, an
    infinite key (z infinite: dnum = dy / den = 0) the other tokens' dv zero."""
    say("infinite sums", dtype)
    inp = inputs.make_inputs(_case(64, dtype, 4, 58, heads=1), lengths=[2600])  # several units, forward and backward
    t = inputs.device_tensors(inp, dev)
    conv_w = t["conv_w"].abs()  # every infinite term of one sign
    rest = dict(eps=inp.eps, cu_seqlens=t["cu_seqlens"], max_seqlen=t["max_seqlen"])
    v = t["v"].clone()
    v[0, 5, 3] = float("inf")
    y = G.forward(t["q"], t["k"], v, t["a"], t["r"], conv_w, t["gamma"], **rest)
    dy = torch.from_numpy(inputs.make_cotangent(inp)).to(dev)
    k = t["k"].clone()
    k[0, 5, 3] = float("inf")
    g = G.backward(t["q"], k, t["v"], t["a"], None, conv_w, None, dy, flags=G.NO_NORM, **rest)
    torch.cuda.synchronize()
    norm_of_infinite(y[0])
    assert bool((g["dv"][0, 16:] == 0).all())


def check_fp32_forward(G, dev, orc, d, width, heads, lengths, seed):
    inp = inputs.make_inputs(_case(d, inputs.F32, width, seed, heads=heads), lengths=lengths)
    t = inputs.device_tensors(inp, dev)
    y = G.forward(t["q"], t["k"], t["v"], t["a"], t["r"], t["conv_w"], t["gamma"], eps=inp.eps,
                  cu_seqlens=t["cu_seqlens"], max_seqlen=t["max_seqlen"])
    torch.cuda.synchronize()
    close(y.cpu().numpy(), orc.forward_inputs(inp)["y"], 1e-5, "y")


@pytest.mark.parametrize("d,width,heads,unit", [(32, 4, 1, 64), (32, 4, 13, 128), (64, 3, 1, 64), (64, 3, 13, 128),
                                                (128, 4, 1, 256), (128, 4, 24, 256)])
def test_fp32_forward_edges(G, dev, orc, d, width, heads, unit):
    say("fp32 forward edges", d, width, heads)
    assert fp32_state_unit(EDGES, heads, d) == unit
    check_fp32_forward(G, dev, orc, d, width, heads, EDGES, 52)


# lengths about the longer units
UNIT_EDGES = [2047, 2048, 2049, 2051, 4099, 1, 1023, 1025, 511, 513, 255, 257, 700]


@pytest.mark.parametrize("d,width,heads,unit", [(32, 4, 5, 256), (64, 3, 5, 256), (64, 4, 10, 512), (32, 2, 20, 1024),
                                                (32, 4, 34, 2048), (64, 4, 34, 2048)])
def test_fp32_forward_long_units(G, dev, orc, d, width, heads, unit):
    say("fp32 forward, units of", unit, d, width)
    assert fp32_state_unit(UNIT_EDGES, heads, d) == unit
    check_fp32_forward(G, dev, orc, d, width, heads, UNIT_EDGES, 61)


# One-launch forward: lengths about its tiles (16 tokens fp32, 32 bf16, four
# waves), every length class of the longest-first order (over 4, 2, 1 times the
# mean, the rest), empty sequences, more sequences than a workgroup has threads.
SHORT_LENGTHS = {
    "edges": [0, 1, 2, 3, 31, 32, 33, 63, 64, 65, 127, 128, 0],
    "classes": [500, 1, 40, 90, 3, 300, 7, 100, 0, 5, 8, 60, 2, 4, 9, 20],
    "many": [int(x) for x in (list(range(1, 41)) * 14)[:513]],
}


SHORT_DIMS = [(32, inputs.F32, 4), (64, inputs.F32, 2), (32, inputs.BF16, 3), (64, inputs.BF16, 4)]


def check_forms(G, dev, orc, d, dtype, width, lengths, bounds, flags=0):
    """The forward with each max_seqlen of `bounds` against the oracle; the bits
    differ where one takes one launch and the other three (bf16 without the norm:
    hardly, as all its roundings are the same)."""
    inp = inputs.make_inputs(_case(d, dtype, width, 53, heads=2), lengths=lengths)
    t = inputs.device_tensors(inp, dev)
    a = None if flags & G.NO_GATE else t["a"]
    cw = None if flags & G.NO_CONV else t["conv_w"]
    r, gm = (None, None) if flags & G.NO_NORM else (t["r"], t["gamma"])
    tol = 1e-5 if dtype == inputs.F32 else 2e-2
    ref = orc.forward_inputs(inp, gate=not flags & G.NO_GATE, conv=not flags & G.NO_CONV,
                             norm=not flags & G.NO_NORM)["y"]
    ys = []
    for m in bounds:
        y = G.forward(t["q"], t["k"], t["v"], a, r, cw, gm, eps=inp.eps, cu_seqlens=t["cu_seqlens"], max_seqlen=m,
                      flags=flags)
        torch.cuda.synchronize()
        ys.append(y.cpu().numpy())
        close(ys[-1], ref, tol, "y, max_seqlen %d" % m)
    if dtype == inputs.F32 or not flags & G.NO_NORM:
        assert (ys[0] != ys[1]).any(), "one form gave both"


@pytest.mark.parametrize("lens", list(SHORT_LENGTHS))
@pytest.mark.parametrize("d,dtype,width", SHORT_DIMS)
def test_short_forward(G, dev, orc, d, dtype, width, lens):
    """The one-launch forward (max_seqlen given) and the three launches that a
    loose max_seqlen takes."""
    say("short forward", d, dtype, width, lens)
    lengths = SHORT_LENGTHS[lens]
    if dtype == inputs.F32:  # fp32 takes one launch up to 128 (d = 64) or 256 tokens
        lengths = [min(n, 128 if d == 64 else 256) for n in lengths]
    check_forms(G, dev, orc, d, dtype, width, lengths, (max(lengths), 1 << 20))


@pytest.mark.parametrize("flags", ["NO_GATE", "NO_CONV", "NO_NORM", "BLA"])
@pytest.mark.parametrize("d,dtype,width", SHORT_DIMS)
def test_short_forward_switches(G, dev, orc, d, dtype, width, flags):
    say("short forward", d, dtype, width, flags)
    check_forms(G, dev, orc, d, dtype, width, SHORT_LENGTHS["edges"], (128, 1 << 20), getattr(G, flags))


@pytest.mark.parametrize("d,dtype,width", SHORT_DIMS)
def test_understated_bound_only_chooses(G, dev, orc, d, dtype, width):
    """Sequences for which the true max_seqlen takes three launches (more than 512
    tokens, few pairs) come out the same, to rounding, in one."""
    say("understated max_seqlen", d, dtype, width)
    check_forms(G, dev, orc, d, dtype, width, [1100, 3, 600, 0, 40], (1, 1100))


def test_short_forward_rounds_as_three_launches(G, dev):
    """Both forms of the bf16 forward at d = 64 round the same gated keys and the
    same normalised S (sequences of one state unit; at d = 32 the state kernel's
    gate maxima are per wave), so they differ where sums an ulp apart round to
    neighbouring values: a share of about 2^-14, each by 2^-8, so 2^-8 / 2^7 =
    3e-5 of the output.  Roundings of their own of S would be 4e-4 apart."""
    say("short forward, rounding")
    lengths = [0, 1, 2, 31, 33, 64, 65, 127, 128, 200, 255, 256, 90, 100, 7]
    inp = inputs.make_inputs(_case(64, inputs.BF16, 4, 56, heads=2), lengths=lengths)
    t = inputs.device_tensors(inp, dev)
    y = [G.forward(t["q"], t["k"], t["v"], t["a"], t["r"], t["conv_w"], t["gamma"], eps=inp.eps,
                   cu_seqlens=t["cu_seqlens"], max_seqlen=m).double() for m in (max(lengths), 1 << 20)]
    torch.cuda.synchronize()
    rel = float((y[0] - y[1]).norm() / y[1].norm())
    say("  one launch against three: rel %.2g" % rel)
    assert 0 < rel < 1e-4  # 0 would mean that one form gave both


def test_short_forward_without_norm_rounds_as_three_launches(G, dev):
    """Without the norm the denominator stays in o: z and phi(q) enter it rounded to
    bf16 in both forms.  With either in fp32 they are 2e-4 and more apart."""
    say("short forward, rounding without the norm")
    lengths = [0, 1, 2, 31, 33, 64, 65, 127, 128, 200, 255, 256, 90, 100, 7]
    inp = inputs.make_inputs(_case(64, inputs.BF16, 4, 64, heads=2), lengths=lengths)
    t = inputs.device_tensors(inp, dev)
    y = [G.forward(t["q"], t["k"], t["v"], t["a"], None, t["conv_w"], None, eps=inp.eps, cu_seqlens=t["cu_seqlens"],
                   max_seqlen=m, flags=G.NO_NORM).double() for m in (max(lengths), 1 << 20)]
    torch.cuda.synchronize()
    rel = float((y[0] - y[1]).norm() / y[1].norm())
    say("  one launch against three: rel %.2g" % rel)
    assert rel < 1e-4


@pytest.mark.parametrize("d,dtype", [(64, inputs.BF16), (32, inputs.F32)])
def test_short_forward_dense(G, dev, orc, d, dtype):
    say("short forward, dense", d, dtype)
    for n in (1, 33, 200):
        inp = inputs.make_inputs(small("b8_n2048_d64", batch=3, heads=2, seqlen=n, head_dim=d, dtype=dtype,
                                       seed=54))
        t = inputs.device_tensors(inp, dev)
        y = G.forward(t["q"], t["k"], t["v"], t["a"], t["r"], t["conv_w"], t["gamma"], eps=inp.eps)
        torch.cuda.synchronize()
        close(y.cpu().numpy(), orc.forward_inputs(inp)["y"], 1e-5 if dtype == inputs.F32 else 2e-2, "y")


@pytest.mark.parametrize("d,dtype,n,tol", [
    (32, inputs.F32, 2048, 2.0e-7), (64, inputs.F32, 2048, 2.0e-7), (32, inputs.BF16, 8192, 7e-4),
    (64, inputs.BF16, 8192, 5e-4), (32, inputs.F32, 16384, 2.3e-7), (64, inputs.F32, 16384, 2.3e-7)])
def test_error_does_not_grow_with_length(G, dev, orc, d, dtype, n, tol):
    """Many pairs of long sequences: the longest that one launch takes, and those
    past it.  Measured, 2-norm of the error over that of the result: fp32 1.67e-7
    at n = 2048, 1.9e-7 at 16384 (uncompensated sums over the sequence: 3.2e-7 and
    2.6e-7); bf16 6.3e-4 (d = 32) and 4.5e-4, the rounding of S."""
    say("long sequences, many pairs", d, dtype, n)
    inp = inputs.make_inputs(small("b8_n2048_d64", batch=1, heads=8, seqlen=n, head_dim=d, dtype=dtype, seed=59))
    ref = orc.forward_inputs(inp)["y"][0]
    t = inputs.device_tensors(inp, dev)
    B = 70 if dtype == inputs.BF16 else 33  # 560 or 264 pairs, all sequences alike
    q, k, v, a, r = (t[x].expand(B, *t[x].shape[1:]).contiguous() for x in ("q", "k", "v", "a", "r"))
    y = G.forward(q, k, v, a, r, t["conv_w"], t["gamma"], eps=inp.eps)
    torch.cuda.synchronize()
    for b in (0, B - 1):
        err = np.linalg.norm(y[b].cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
        say("  rel %.3g" % err)
        assert err < tol


# The layer's conv and gate logits in one pass: token tiles of 64 (32768 to
# 65535 tokens; test_layer_gpu.py has tiles of 32 and 128), sequences ending in
# and on a tile's runs, a half-empty last channel step, and gates past the 32nd,
# which a kernel of their own forms.
LAYER_CASES = {
    "tile64": dict(lens=[1, 32767, 3, 0, 60, 129, 2, 5], d_model=192, heads=2, head_dim=32, conv_width=3),
    "tile64_full_width": dict(lens=[32764, 4, 1], d_model=256, heads=1, head_dim=64, conv_width=4),
    "gates40": dict(lens=[33, 95, 7], d_model=64, heads=40, head_dim=32, conv_width=4),
    # taps of four steps through two buffers, one tap each
    "one_tap": dict(lens=[70, 33, 1], d_model=448, heads=3, head_dim=32, conv_width=1),
    # projections on 128 x 128 tiles: one full tile and one feature tile, one K
    # step; a last tile of one token; and, past them, deferred stores over 32 K
    # steps (17 x 16 tiles of 256)
    "small_tile": dict(lens=[100, 28], d_model=64, heads=1, head_dim=32, conv_width=2),
    "small_tile_rest": dict(lens=[257], d_model=320, heads=3, head_dim=128, conv_width=4),
    "deferred_long": dict(lens=[4099, 2], d_model=2048, heads=8, head_dim=128, conv_width=3),
}


@pytest.mark.parametrize("name", list(LAYER_CASES))
def test_layer_conv_gate(G, dev, monkeypatch, name):
    kw = dict(LAYER_CASES[name])
    lens = kw.pop("lens")
    w = inputs.LayerWorkload("conv gate " + name, batch=len(lens), seqlen=0, seed=55, ragged=True, **kw)
    monkeypatch.setitem(test_layer_gpu.CASES, name, (w, lens))
    test_layer_gpu.test_layer_project_parity(G, dev, name)
