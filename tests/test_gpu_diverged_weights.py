"""Output stage with weights that are infinite or close to the largest float: a training run that has diverged has to see it,
in the loss and in the gradients, as with plain fp32 products."""
import numpy as np
import pytest
import torch

from paper_1907_03329_amd import binding, synth
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu

SHAPES = [(8, 1), (8, 64), (32, 17), (40, 8), (40, 33), (52, 3), (50, 48), (64, 64)]


def setting(hidden, H, B=37, P=5):
    I = 8 if hidden == 8 else 20 if hidden == 64 else 12
    cfg = synth.CONFIGS["quarterly"].with_(B=B, T=I + H + P - 1, I=I, H=H, hidden=hidden, blocks=((1, 2),))
    inp = synth.make_inputs(cfg, seed=hidden + H)
    at = {name: (off, shape) for name, off, shape in synth.weight_layout(cfg)}
    return cfg, inp, at


def weight(inp, at, name):
    off, shape = at[name]
    return inp["weights"][off:off + int(np.prod(shape))].reshape(shape)


def tanh_layer(cfg, inp, at, step):
    r = step.buffer("block_out", len(cfg.blocks) - 1).cpu().numpy().astype(np.float64)
    with np.errstate(over="ignore"):
        return np.tanh(r @ weight(inp, at, "Wa").astype(np.float64).T + weight(inp, at, "ba"))


def gradients(cfg, at, step):
    g = step.grad_weights.cpu().numpy()
    return {name: g[off:off + int(np.prod(shape))].reshape(shape) for name, (off, shape) in at.items()}


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("hidden,H", SHAPES)
def test_infinite_weight_of_the_linear_layer(hidden, H, sign):
    cfg, inp, at = setting(hidden, H)
    plain = gc.run_gpu(cfg, inp)
    before = {n: t.cpu().numpy() for n, t in (("O", plain.buffer("O")), ("forecasts", plain.forecasts))}
    plain.close()
    row, unit = H - 1, hidden // 2
    weight(inp, at, "Wo")[row, unit] = sign * np.inf
    step = gc.run_gpu(cfg, inp)
    o, others = step.buffer("O").cpu().numpy(), np.arange(H) != row
    want = sign * np.inf * np.sign(tanh_layer(cfg, inp, at, step)[..., unit])
    assert np.array_equal(o[..., row], want) and np.array_equal(o[..., others], before["O"][..., others])
    assert step.loss.item() == np.inf
    fc = step.forecasts.cpu().numpy()
    assert np.array_equal(fc[..., row], np.where(want > 0, np.inf, 0.0)) and np.array_equal(fc[..., others], before["forecasts"][..., others])
    # infinite times a gradient, and infinite minus infinite: every gradient that the unit's has a part in
    g = gradients(cfg, at, step)
    assert not np.isfinite(g["Wa"][unit]).any() and not np.isfinite(g["ba"][unit])
    assert not np.isfinite(step.buffer("grad_top").cpu().numpy()).any()
    assert not any(np.isfinite(g[n]).any() for n in g if n[1:].isdigit())
    assert not np.isfinite(step.grad_es_params.cpu().numpy()).any()
    assert np.isfinite(g["Wo"]).all() and np.isfinite(g["bo"]).all()

    # without a reverse pass, and at the end of the series
    dev = gc.to_device(inp)
    args = [dev[k] for k in ("y", "lengths", "es_params", "weights")]
    binding.esrnn_set_forward_only(step.handle, True)
    step.forward(*args)
    assert step.loss.item() == np.inf and np.array_equal(step.forecasts.cpu().numpy(), fc)
    args[1] = args[1] - H
    last = step.predict(*args).cpu().numpy()
    assert np.array_equal(last[:, row], np.where(want[-1] > 0, np.inf, 0.0)) and np.isfinite(last[:, others]).all()
    # the next weights are looked at again
    weight(inp, at, "Wo")[row, unit] = 0.0
    args[1], args[3] = dev["lengths"], torch.from_numpy(inp["weights"]).cuda()
    step.forward(*args)
    assert np.isfinite(step.loss.item())
    step.close()


@pytest.mark.parametrize("hidden,H", SHAPES)
def test_infinite_weight_of_the_tanh_layer(hidden, H):
    cfg, inp, at = setting(hidden, H)
    weight(inp, at, "Wa")[hidden - 1, 1] = -np.inf
    step = gc.run_gpu(cfg, inp)
    # the unit saturates, and its gradient vanishes; infinite times nothing is what goes to the block output
    wo, bo = weight(inp, at, "Wo").astype(np.float64), weight(inp, at, "bo")
    assert gc.rel_err(step.buffer("O").cpu().numpy(), tanh_layer(cfg, inp, at, step) @ wo.T + bo) <= gc.TOL_FWD
    assert np.isfinite(step.loss.item())
    g = gradients(cfg, at, step)
    assert all(np.isfinite(g[n]).all() for n in ("Wa", "ba", "Wo", "bo")) and not g["Wa"][hidden - 1].any()
    assert not np.isfinite(step.buffer("grad_top").cpu().numpy()[..., 1]).any()
    assert not any(np.isfinite(g[n]).any() for n in g if n[1:].isdigit())
    assert not np.isfinite(step.grad_es_params.cpu().numpy()).any()
    step.close()


@pytest.mark.parametrize("size", [1e30, 1e35, 3.38e38])
@pytest.mark.parametrize("hidden,H", SHAPES)
def test_weights_near_the_largest_float(hidden, H, size):
    """Outputs are the weight times the tanh layer, which has an absolute error of a few units of 2^-24: those of its
    pre-activation and of 1 - 2 / (1 + exp(2 x)) near 1."""
    cfg, inp, at = setting(hidden, H)
    row, unit = H // 2, hidden - 1
    weight(inp, at, "Wo")[row, unit] = size
    step = gc.run_gpu(cfg, inp, backward=False)
    want = tanh_layer(cfg, inp, at, step)[..., unit] * size
    assert np.abs(step.buffer("O").cpu().numpy()[..., row] - want).max() <= 8 * 2.0 ** -24 * size
    step.close()
