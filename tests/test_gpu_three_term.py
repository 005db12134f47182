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
