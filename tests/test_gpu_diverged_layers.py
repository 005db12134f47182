"""4-series LSTM layers with operands that are infinite or large: gates and weight gradients are those of plain fp32 products, so that
whoever tests a loss or a gradient for finiteness sees that a run has diverged."""
import numpy as np
import pytest

from oracle import oracle
from paper_1907_03329_amd import binding, synth
from paper_1907_03329_amd.synth import Config
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu

# (hidden, input window): first layers of every padded hidden size, later ones behind them
SHAPES = [(8, 4), (30, 6), (40, 4), (40, 23), (50, 12), (64, 64)]


def setting(hidden, window, blocks=((1,), (2,)), B=21, positions=6, H=3):
    cfg = Config("diverged", B=B, T=window + H + positions - 1, n_seas=1, m1=4, m2=0, I=window, H=H, hidden=hidden, blocks=blocks)
    inp = synth.make_inputs(cfg, seed=hidden + window)
    at = {name: inp["weights"][off:off + int(np.prod(shape))].reshape(shape) for name, off, shape in synth.weight_layout(cfg)}
    return cfg, inp, at


def check_gates(cfg, step, at):
    """Every gate against float64 products of the layer's own inputs and states; where those are infinite or NaN, exactly."""
    below, dilations = step.buffer("X").cpu().numpy(), [d for block in cfg.blocks for d in block]
    for layer, d in enumerate(dilations):
        gates, hid = (step.buffer(name, layer).cpu().numpy() for name in ("gates", "hid"))
        before = np.concatenate([np.zeros_like(hid[:d]), hid[:-d]])[:len(hid)]
        rows = np.concatenate([below, before], axis=-1).astype(np.float64)
        with np.errstate(all="ignore"):
            pre = (rows[:, :, None] * at[f"W{layer}"].astype(np.float64)).sum(-1) + at[f"b{layer}"]
            pre = pre.reshape(rows.shape[:2] + (4, cfg.hidden)).transpose(0, 1, 3, 2)
            want = 1.0 / (1.0 + np.exp(-pre))
            want[..., 2] = np.tanh(pre[..., 2])
        np.testing.assert_allclose(gates, want, rtol=0, atol=5e-6, equal_nan=True, err_msg=f"layer {layer}")
        below = hid


@pytest.mark.parametrize("together", ["0", "256"])
@pytest.mark.parametrize("hidden,window", SHAPES)
def test_gates_of_infinite_and_large_operands(hidden, window, together, monkeypatch):
    monkeypatch.setenv("ESRNN_NARROW_BELOW", "100000")
    monkeypatch.setenv("ESRNN_TOGETHER", together)
    # infinite weights of opposite signs in one row of either layer; a row whose largest weights count in proportion
    for a, b in ((np.inf, -np.inf), (np.inf, 1.0), (8.0 * 2.0 ** 101, -2.0 ** 101)):
        cfg, inp, at = setting(hidden, window)
        for layer, unit in (("W0", hidden - 1), ("W1", 1)):
            at[layer][unit, 0], at[layer][unit, 2] = a, b
        step = gc.run_gpu(cfg, inp, backward=False)
        check_gates(cfg, step, at)
        step.close()


@pytest.mark.parametrize("hidden,window", SHAPES)
def test_gates_of_infinite_inputs(hidden, window, monkeypatch):
    monkeypatch.setenv("ESRNN_NARROW_BELOW", "100000")
    cfg, inp, at = setting(hidden, window)
    inp["y"][1, 2:6] = inp["y"][1:3, 6:9] = 0.0       # one or two observations of zero in a window: their logarithms
    step = gc.run_gpu(cfg, inp, backward=False)
    assert np.isinf(step.buffer("X").cpu().numpy()).any()
    check_gates(cfg, step, at)
    step.close()


def weight_gradients(cfg, inp):
    """The first layer's, of the kernels and of the oracle: [gate, unit, column of x and h]."""
    step = gc.run_gpu(cfg, inp)
    with np.errstate(all="ignore"):
        f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
        g = oracle.backward(cfg, f, want_adjoints=False)
    off, shape = next((off, shape) for name, off, shape in synth.weight_layout(cfg) if name == "W0")
    out = [np.asarray(v[off:off + shape[0] * shape[1]]).reshape(4, cfg.hidden, -1) for v in (step.grad_weights.cpu().numpy(), g.grad_weights)]
    step.close()
    return out


@pytest.mark.parametrize("hidden,window", SHAPES)
def test_weight_gradient_of_infinite_inputs(hidden, window, monkeypatch):
    """The columns that the logarithm of an observation of zero reaches are NaN, the gradient of a saturated gate times infinity; the
    others are as they would be."""
    monkeypatch.setenv("ESRNN_NARROW_BELOW", "100000")
    cfg, inp, at = setting(hidden, window, positions=2)
    inp["y"][1, 4] = 0.0
    got, want = weight_gradients(cfg, inp)
    assert np.isnan(got[:, :, :2]).all() and np.array_equal(np.isfinite(got), np.isfinite(want))
    finite = np.isfinite(want)
    np.testing.assert_allclose(got[finite], want[finite], rtol=0, atol=1e-5 * np.abs(want[finite]).max())


@pytest.mark.parametrize("hidden,window", SHAPES)
def test_weight_gradient_of_gradients_past_the_largest_float(hidden, window, monkeypatch):
    """One window of one series.  Weights of the output stage of 3.3e38 and 3 make the gradient of one state, some half their product,
    larger than floats are; those of the other states stay below them."""
    monkeypatch.setenv("ESRNN_NARROW_BELOW", "100000")
    cfg, inp, at = setting(hidden, window, blocks=((1,),), B=1, positions=1, H=1)
    unit = hidden - 2
    at["Wo"][0, 2], at["Wa"][2] = 3.3e38, np.clip(at["Wa"][2], -0.5, 0.5)
    at["Wa"][2, unit] = 3.0
    got, want = (v[:, :, :window] for v in weight_gradients(cfg, inp))
    assert not np.isfinite(got[[0, 2, 3], unit]).any()      # input gate, candidate, output gate
    # (inputs of one window are logarithms of ratios, some 0.01 in size with an error of a few 2^-24)
    others = np.arange(hidden) != unit
    np.testing.assert_allclose(got[:, others], want[:, others], rtol=0, atol=1e-4 * np.abs(want[:, others]).max())
