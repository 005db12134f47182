"""The 4-series kernels form the input half of the pre-activations and the weight gradient four positions at a time: chains of every
length modulo four, and every way columns and row tiles are dealt to the waves (all shared, some shared, none)."""
import numpy as np
import pytest

from oracle import oracle
from paper_1907_03329_amd import synth
from paper_1907_03329_amd.synth import Config
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


def relative(got, want):
    got, want = np.asarray(got, dtype=np.float64).ravel(), np.asarray(want, dtype=np.float64).ravel()
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


# Bound: rounding in fp32 accumulation stays below 5e-6 for the steepest gate (see test_gpu_three_term.py); a position's input half in
# the wrong place is 1e-2 and more.
@pytest.mark.parametrize("hidden,window", [(8, 4), (30, 6), (40, 4), (40, 23), (50, 18), (52, 52), (64, 64)])
@pytest.mark.parametrize("positions", [1, 2, 3, 4, 5, 7, 8, 9, 12, 13])
def test_gates_of_chains_of_every_length(hidden, window, positions, monkeypatch):
    monkeypatch.setenv("ESRNN_NARROW_BELOW", "100000")
    for together in ("0", "256"):
        monkeypatch.setenv("ESRNN_TOGETHER", together)
        cfg = Config("groups", B=21, T=window + 3 + positions - 1, n_seas=1, m1=4, m2=0, I=window, H=3, hidden=hidden,
                     blocks=((1,), (2,)) if positions > 1 else ((1,),))
        inp = synth.make_inputs(cfg, seed=positions)
        f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
        step = gc.run_gpu(cfg, inp)
        for layer in range(f.n_layers):
            got = step.buffer("gates", layer).cpu().numpy()
            assert float(np.abs(got - f.gates[layer].transpose(1, 0, 3, 2)).max()) <= 5e-6, (layer, together)
        step.close()


# Bound: a position that is missing or counted twice is 0.07 and more of a sum over 13 of them.  Inputs of later layers are states,
# whose fp32 errors reach the sum undiminished where it has few terms (2e-7 to 1.6e-6); without one of the six terms products are off
# by 2.4e-6 and more (random factors, lengths 16 and 160): 2.2e-6.  Inputs of the first layer are logarithms of ratios, some 0.05 in
# size with an error of a few 2^-24 from the ratio's rounding, 4e-6 of them: 1e-5.
@pytest.mark.parametrize("hidden,window", [(8, 4), (30, 6), (40, 4), (40, 23), (50, 18), (50, 12), (64, 64)])
@pytest.mark.parametrize("positions", [1, 2, 3, 4, 5, 6, 7, 8, 9, 13])
def test_weight_gradient_of_chains_of_every_length(hidden, window, positions, monkeypatch):
    monkeypatch.setenv("ESRNN_NARROW_BELOW", "100000")
    for together in ("0", "256"):
        monkeypatch.setenv("ESRNN_TOGETHER", together)
        cfg = Config("groups", B=21, T=window + 3 + positions - 1, n_seas=1, m1=4, m2=0, I=window, H=3, hidden=hidden,
                     blocks=((1,), (2,)) if positions > 1 else ((1,),))
        inp = synth.make_inputs(cfg, seed=positions)
        f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
        wm = gc.valid_window_mask(cfg, inp["lengths"])
        step = gc.run_gpu(cfg, inp)
        near, side = gc.kink_sides(cfg, f, wm, step.buffer("grad_O").cpu().numpy())
        g = oracle.backward(cfg, f, want_adjoints=True, pin_side=side if near.any() else None)
        gw = step.grad_weights.cpu().numpy()
        for name, off, shape in synth.weight_layout(cfg):
            n = int(np.prod(shape))
            if name.startswith("W") and name[1:].isdigit():
                assert relative(gw[off:off + n], g.grad_weights[off:off + n]) <= (1e-5 if name == "W0" else 2.2e-6), (name, together)
        step.close()
