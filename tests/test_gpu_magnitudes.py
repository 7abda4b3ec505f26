"""Magnitudes that differ widely inside one call: float32 keeps 24 bits of
every value whatever stands beside it, so a call's results must not depend on
how unequal its hidden units, channels or samples are.

Two kinds of case.  Rescaling: unit c of a layer is multiplied by a power of
two (its weights and bias) and the next layer's weights on it are divided by
the same, which leaves Q and, up to those factors, every gradient exactly as
they were; the factors cover 2^-24 .. 2^24 within each layer.  Unequal states:
states whose activations are 2^-30 of the others', or overflow to infinity,
in one batch with ordinary ones."""
import numpy as np
import pytest

import dqn_inputs as di
import oracle
import paper_1508_04186_amd as dq
from gpu_util import MARGIN_MIN, assert_close, assert_grad_close, dev_tensor, host, say
from test_gpu_parity import NETS, _run_td, _td_inputs

pytestmark = pytest.mark.gpu

F32 = np.float32
# Float32 sums of up to 1e5 products, relative to their norm: roundings of
# 2^-24 each, random in sign, on sums that cancel to about a tenth of their
# terms.  (A value kept to 2^-40 of a neighbour 2^30 larger is off by 1e-3.)
TOL = 1e-5


def _span(shape, name):
    off, shp = shape.slices()[name]
    return slice(off, off + int(np.prod(shp))), shp


def _rescaling(shape, layer, seed):
    """Float64 factors (powers of two) of the flat parameters: units of
    `layer` ("conv1", ..., "fc1") times 2^e, the next layer's weights on them
    divided by it."""
    names = [f"conv{i + 1}" for i in range(len(shape.conv))] + ["fc1", "fc2"]
    nxt = names[names.index(layer) + 1]
    f = np.ones(shape.param_count())
    sl, shp = _span(shape, layer + ".W")
    e = np.random.default_rng(seed).integers(-24, 25, shp[0])
    c = np.exp2(e.astype(np.float64))
    f[sl] = np.repeat(c, int(np.prod(shp[1:])))
    f[_span(shape, layer + ".b")[0]] = c
    sl, shp = _span(shape, nxt + ".W")
    per = int(np.prod(shp[1:])) // c.size     # weights on one unit: taps, or the pixels of a map
    f[sl] = np.tile(np.repeat(1.0 / c, per), shp[0])
    return f


def _quiet_theta(shape, seed, exp=-30):
    """Zero-bias parameters whose first layer's lower half of the channels
    sees the newest frame only and its upper half the oldest only, with
    weights of 2^exp of the others': a state that shows just the oldest frame
    has all its activations 2^exp of the ordinary ones."""
    th = di.xavier_theta(shape, seed)
    sl, shp = _span(shape, "conv1.W")
    w = th[sl].reshape(shp)
    half = shp[0] // 2
    w[:half, :3] = 0
    w[half:, 1:] = 0
    w[half:] *= F32(2.0) ** exp
    return th


def _forward(dev, net, th, s):
    import torch
    q = torch.empty((s.shape[0], net.n_actions), dtype=torch.float32, device=dev)
    dq.dqn_forward(net, dev_tensor(th), dev_tensor(s), q_out=q)
    torch.cuda.synchronize()
    return host(q)


# Both sides of the sizes at which the fc1 gradients change kernels (large 128,
# small 256); 301: runs of samples in the conv kernels.
@pytest.mark.parametrize("name,B,layer", [("large", B, layer) for layer in ("fc1", "conv3", "conv2", "conv1")
                                          for B in (40, 130, 301)] +
                         [("small", B, layer) for layer in ("fc1", "conv2", "conv1") for B in (90, 257)])
def test_td_gradient_under_unit_rescaling(dev, name, B, layer):
    net, shape = NETS[name]
    th = di.xavier_theta(shape, 500 + B, bias_scale=0.05)
    f = _rescaling(shape, layer, B)
    big = (th * f).astype(F32)
    assert np.array_equal(big / f, th.astype(np.float64))
    s, sn, a, r, t = _td_inputs(shape, B, 501 + B, theta=th)
    say(f"[magnitudes] net={name} batch={B} rescaled units of {layer}")
    g, loss, q, y = _run_td(dev, net, big, None, s, sn, a, r, t, 0.99)
    ref = oracle.td_gradient(shape, th, None, s, sn, a, r, t, float(F32(0.99)))
    assert_close(q, ref["q"], TOL, "q")
    assert_close(y, ref["y"], TOL, "y")
    assert abs(loss - ref["loss"]) <= TOL * abs(ref["loss"])
    assert_grad_close(shape, g * f, ref["grad"], TOL)


# The input gradients: what reaches the layers below the rescaled one, as the
# gradient of their weights.  A sample a workgroup, and runs of them (301).
@pytest.mark.parametrize("name,layer,B", [("large", "conv3", 40), ("large", "conv3", 301), ("large", "conv2", 40),
                                          ("large", "conv2", 301), ("small", "conv2", 90), ("small", "conv2", 300)])
def test_input_gradients_under_unit_rescaling(dev, name, layer, B):
    net, shape = NETS[name]
    th = di.xavier_theta(shape, 900 + B, bias_scale=0.05)
    f = _rescaling(shape, layer, 2 + B)
    s, sn, a, r, t = _td_inputs(shape, B, 901 + B, theta=th)
    say(f"[magnitudes] input gradients net={name} batch={B} rescaled units of {layer}")
    g, _, _, _ = _run_td(dev, net, (th * f).astype(F32), None, s, sn, a, r, t, 0.99)
    ref = oracle.td_gradient(shape, th, None, s, sn, a, r, t, float(F32(0.99)))["grad"]
    for below in ("conv1.W", "conv1.b", "conv2.W", "conv2.b"):
        if below[:5] < layer:
            sl, _ = _span(shape, below)
            assert_close(g[sl], ref[sl], TOL, below)


def _two_networks(shape, seed):
    """Parameters of two networks side by side, their first halves of the
    channels seeing the oldest frame only and their second halves the newest
    only, with negative biases (a half that sees black is silent); the output
    rows of the lower actions are 2^-16 of the others.  Returns them and the
    mask of the first network's parameters."""
    th = di.xavier_theta(shape, seed)
    mine = np.zeros(th.size, bool)
    rng = np.random.default_rng(seed + 1)
    names = [f"conv{i + 1}" for i in range(len(shape.conv))] + ["fc1"]
    for name in names:
        sl, shp = _span(shape, name + ".W")
        w, m = th[sl].reshape(shp), mine[sl].reshape(shp)
        ho, hi = shp[0] // 2, shp[1] // 2
        if name == "conv1":
            w[:, 1:3] = 0
            hi = 1
        w[:ho, hi:] = 0
        w[ho:, :(3 if name == "conv1" else hi)] = 0
        m[:ho, :hi] = True
        sl, _ = _span(shape, name + ".b")
        th[sl] = rng.uniform(-0.01, -0.001, shp[0]).astype(F32)
        mine[sl][:ho] = True
    sl, shp = _span(shape, "fc2.W")
    th[sl].reshape(shp)[:shp[0] // 2] *= F32(2.0) ** -16
    return th, mine


# Slots and tiles that hold samples of both kinds: half of the samples show
# only the oldest frame and have TD errors and output weights of 2^-16 of the
# others', so the first network's gradient is theirs alone, 2^-32 beside the
# second's.
@pytest.mark.parametrize("name,B", [("large", 301), ("large", 600), ("small", 300)])
def test_gradient_of_quiet_samples_among_ordinary_ones(dev, name, B):
    net, shape = NETS[name]
    th, mine = _two_networks(shape, 1000 + B)
    cand = di.random_states(2 * B, 1001 + B)
    quiet = np.arange(2 * B) % 2 == 1
    cand[quiet, 1:] = 0
    cand[~quiet, :3] = 0
    keep = np.nonzero(oracle.relu_margins(shape, th, cand) >= MARGIN_MIN)[0][:B]
    assert keep.size == B
    s, quiet = cand[keep], quiet[keep]
    a, r, t = di.random_transitions(B, shape.n_actions // 2, 1002 + B)
    a[~quiet] += shape.n_actions // 2
    r = (r + F32(0.5)) * np.where(quiet, F32(2.0) ** -16, F32(1.0))
    t[quiet] = 1
    sn = di.random_states(B, 1003 + B)
    say(f"[magnitudes] gradient net={name} batch={B} quiet samples")
    g, _, _, _ = _run_td(dev, net, th, None, s, sn, a, r.astype(F32), t, 0.99)
    ref = oracle.td_gradient(shape, th, None, s, sn, a, r.astype(F32), t, float(F32(0.99)))["grad"]
    for part in shape.slices():
        if part.startswith("fc2"):
            continue
        sl, _ = _span(shape, part)
        assert_close(g[sl][mine[sl]], ref[sl][mine[sl]], TOL, part)
        assert_close(g[sl][~mine[sl]], ref[sl][~mine[sl]], TOL, part + " of the others")


# The conv kernels: large to 64 states (a workgroup per tile) and above (runs
# of samples, the last short at 301), small from 100.
@pytest.mark.parametrize("name,layer,B", [("large", layer, B) for layer in ("conv1", "conv2", "conv3")
                                          for B in (20, 65, 301)] +
                         [("small", layer, B) for layer in ("conv1", "conv2") for B in (150, 600)])
def test_forward_under_unit_rescaling(dev, name, layer, B):
    net, shape = NETS[name]
    th = di.xavier_theta(shape, 800 + B, bias_scale=0.05)
    f = _rescaling(shape, layer, 1 + B)
    s = di.random_states(B, 801 + B)
    say(f"[magnitudes] forward net={name} batch={B} rescaled units of {layer}")
    q = _forward(dev, net, (th * f).astype(F32), s)
    rows = np.unique(np.linspace(0, B - 1, 30).astype(int))
    assert_close(q[rows], oracle.forward_q(shape, th, s[rows]), TOL, "q")


@pytest.mark.parametrize("name,B", [("large", 150), ("large", 1100), ("small", 300)])
def test_forward_of_quiet_states_among_ordinary_ones(dev, name, B):
    net, shape = NETS[name]
    th = _quiet_theta(shape, 600 + B)
    s = di.random_states(B, 601 + B)
    quiet = np.arange(B) % 3 == 1
    s[quiet, 1:] = 0
    say(f"[magnitudes] net={name} batch={B} quiet states")
    q = _forward(dev, net, th, s)
    rows = np.concatenate([np.nonzero(quiet)[0][:40], np.nonzero(~quiet)[0][:20]])
    ref = oracle.forward_q(shape, th, s[rows])
    err = np.linalg.norm(q[rows] - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= TOL, f"largest error of a state {err.max():.2e} (state {rows[err.argmax()]})"


@pytest.mark.parametrize("name,B", [("large", 3), ("large", 300), ("small", 150), ("small", 600)])
def test_forward_of_states_on_small_weights(dev, name, B):
    """Every unit of the first layer weighs the oldest frame by 2^-30 of the
    others; some states show only that frame."""
    net, shape = NETS[name]
    th = di.xavier_theta(shape, 1100 + B)
    sl, shp = _span(shape, "conv1.W")
    th[sl].reshape(shp)[:, 0] *= F32(2.0) ** -30
    s = di.random_states(B, 1101 + B)
    quiet = np.arange(B) % 3 == 1
    s[quiet, 1:] = 0
    say(f"[magnitudes] net={name} batch={B} states on small weights")
    rows = np.nonzero(quiet)[0][:40]
    q = _forward(dev, net, th, s)[rows]
    ref = oracle.forward_q(shape, th, s[rows])
    err = np.linalg.norm(q - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= TOL, f"largest error of a state {err.max():.2e} (state {rows[err.argmax()]})"


@pytest.mark.parametrize("name,B", [("large", 150), ("large", 1100), ("small", 300)])
def test_forward_with_overflowing_states(dev, name, B):
    """The newest frame's top left corner drives the last conv layer to
    infinity.  States where it is dark: the same bits beside overflowing
    states as beside none."""
    net, shape = NETS[name]
    th = di.xavier_theta(shape, 700 + B, bias_scale=0.02)
    for i in range(len(shape.conv)):
        sl, shp = _span(shape, f"conv{i + 1}.W")
        w = th[sl].reshape(shp)
        w[0] = 0
        if i == 0:
            w[0, 3, :4, :4] = F32(2.0) ** 70
        else:
            w[:, 0] = 0
            w[0, 0, 0, 0] = F32(2.0) ** (70 if i == len(shape.conv) - 1 else 0)
        th[_span(shape, f"conv{i + 1}.b")[0]][0] = 0
    s = di.random_states(B, 701 + B)
    s[:, 3] = 0
    hot = s.copy()
    loud = np.arange(B) % 50 == 7
    hot[loud, 3, :4, :4] = 255
    say(f"[magnitudes] net={name} batch={B} overflowing states")
    q, qh = _forward(dev, net, th, s), _forward(dev, net, th, hot)
    assert np.isfinite(q).all()
    assert np.array_equal(q[~loud], qh[~loud])
    rows = np.nonzero(~loud)[0][:40]
    assert_close(q[rows], oracle.forward_q(shape, th, s[rows]), TOL, "q")
