"""Accuracy of the LSTM kernels whose products run on the bf16 matrix pipe as three-term sums: they have to be as
accurate as fp32 products, which the common bounds of 1e-4 / 1e-3 would not tell from products with a term missing.

Bound of a gate: a pre-activation is a sum of at most 128 products of |w| <= 1/sqrt(hidden) and inputs below 2 in size,
so the sum of their absolute values stays below 30, and rounding in fp32 accumulation over a layer stays below about
30 * 2^-24 * sqrt(128) / 4 = 5e-6 for the steepest gate (tanh; a sigmoid has a quarter of it).  Dropping the lo terms
would show as 2^-16 of a product, 1e-5 and more."""
import numpy as np
import pytest

from oracle import oracle
from paper_1907_03329_amd import synth
from paper_1907_03329_amd.synth import Config

pytestmark = pytest.mark.gpu

from tests import gpu_common as gc  # noqa: E402

# (hidden, input window): every way a contraction over pairs of unit tiles is cut (full groups of four pairs, rest of
# one, two, three pairs; a last pair with one tile), one and two tiles per wave, and the edges of the padded sizes
SHAPES = [(1, 4), (8, 8), (9, 8), (32, 6), (32, 30), (33, 3), (40, 12), (40, 23), (40, 30), (41, 11), (50, 18), (52, 52),
          (53, 64), (64, 64)]


@pytest.mark.parametrize("hidden,window", SHAPES)
def test_gates_are_as_accurate_as_fp32_products(hidden, window, monkeypatch):
    monkeypatch.setenv("ESRNN_NARROW_BELOW", "0")
    # chains of one, two, three and many positions; 17 series: a full tile and one with a single series
    cfg = Config("three_term", B=17, T=window + 3 + 12, n_seas=1, m1=4, m2=0, I=window, H=3, hidden=hidden,
                 blocks=((1, 5), (13,), (4,)))
    inp = synth.make_inputs(cfg, seed=hidden)
    f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
    step = gc.run_gpu(cfg, inp)
    worst = 0.0
    for layer in range(f.n_layers):
        got = step.buffer("gates", layer).cpu().numpy()
        worst = max(worst, float(np.abs(got - f.gates[layer].transpose(1, 0, 3, 2)).max()))
    print(f"  hidden {hidden} window {window}: gates within {worst:.2e}", flush=True)
    assert worst <= 5e-6
    gc.check_backward(cfg, inp, step, f)
    step.close()


def relative(got, want):
    got, want = np.asarray(got, dtype=np.float64).ravel(), np.asarray(want, dtype=np.float64).ravel()
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


# The 4-series kernels form fp32 products: the 16-series ones have to be as close to float64 on the same inputs, tensor by
# tensor.  A sum of products that lacks one of the small terms is off by 2.4e-6 to 3.5e-6 of its size (random factors,
# lengths 16 and 160); the errors here are 2e-7 to 6e-7 (4e-7 to 1.6e-6 for the first layer with long windows, most of it
# from its inputs), so half as much again and 3e-7 tell the two apart.  (The output stage is the same on both sides; what its
# products are held to is in test_output_stage_accuracy.py.)
@pytest.mark.parametrize("hidden,window", SHAPES)
def test_gradients_are_as_accurate_as_with_fp32_products(hidden, window, monkeypatch):
    cfg = Config("three_term", B=17, T=window + 3 + 40, n_seas=1, m1=4, m2=0, I=window, H=3, hidden=hidden,
                 blocks=((1, 5), (13,), (4,)))
    inp = synth.make_inputs(cfg, seed=hidden)
    f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
    wm = gc.valid_window_mask(cfg, inp["lengths"])
    errors = {}
    for narrow in ("0", "100000"):
        monkeypatch.setenv("ESRNN_NARROW_BELOW", narrow)
        step = gc.run_gpu(cfg, inp)
        near, side = gc.kink_sides(cfg, f, wm, step.buffer("grad_O").cpu().numpy())
        g = oracle.backward(cfg, f, want_adjoints=True, pin_side=side if near.any() else None)
        e = errors[narrow] = {"X": relative(step.buffer("grad_X").cpu().numpy(), g.gX.transpose(1, 0, 2))}
        gw = step.grad_weights.cpu().numpy()
        for name, off, shape in synth.weight_layout(cfg):
            n = int(np.prod(shape))
            e[name] = relative(gw[off:off + n], g.grad_weights[off:off + n])
        step.close()
    for name, fp32 in errors["100000"].items():
        print(f"  {name}: {errors['0'][name]:.1e} (fp32 products {fp32:.1e})", flush=True)
        assert errors["0"][name] <= 1.5 * fp32 + 3e-7, name


# The mean error of a unit's pre-activations does not average out in gradients.  Biases that the products are small
# beside: with every product rounded at the bias's size the mean is 1.35 to 1.9 times that of fp32 products, the bias added
# last gives 0.97 to 1.06; the noise of 2624 positions is 1 % of it.
@pytest.mark.parametrize("hidden,window", [(32, 6), (40, 4), (40, 30), (50, 12), (52, 52), (64, 64)])
def test_preactivations_have_no_systematic_error(hidden, window, monkeypatch):
    cfg = Config("three_term", B=64, T=window + 3 + 40, n_seas=1, m1=4, m2=0, I=window, H=3, hidden=hidden,
                 blocks=((1, 5), (13,), (4,)))
    inp = synth.make_inputs(cfg, seed=hidden)
    for name, off, shape in synth.weight_layout(cfg):
        if name[0] == "b" and name[1:].isdigit():
            b = inp["weights"][off:off + int(np.prod(shape))]
            b += 1.5 * np.sign(b)
    f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
    mean, rms = {}, {}
    for narrow in ("0", "100000"):
        monkeypatch.setenv("ESRNN_NARROW_BELOW", narrow)
        step = gc.run_gpu(cfg, inp, backward=False)
        m, r = [], []
        for layer in range(f.n_layers):
            want = f.gates[layer].transpose(1, 0, 3, 2)
            slope = np.where(np.arange(4) == 2, 1.0 - want * want, want * (1.0 - want))     # tanh, or sigmoid
            e = (step.buffer("gates", layer).cpu().numpy() - want) / slope
            m.append(np.sqrt((e.mean((0, 1)) ** 2).mean()))
            r.append(np.sqrt((e ** 2).mean()))
        mean[narrow], rms[narrow] = np.exp(np.mean(np.log(m))), np.exp(np.mean(np.log(r)))
        step.close()
    print(f"  mean {mean['0']:.1e} rms {rms['0']:.1e} (fp32 products {mean['100000']:.1e} {rms['100000']:.1e})", flush=True)
    assert mean["0"] <= 1.15 * mean["100000"] and rms["0"] <= rms["100000"]
