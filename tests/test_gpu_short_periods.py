"""Smoothing recursions whose groups of steps are as short as the period allows: one step (period 1), two and four."""
import numpy as np
import pytest

from oracle import oracle
from paper_1907_03329_amd import synth
from paper_1907_03329_amd.synth import Config
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("logit", [False, True])
@pytest.mark.parametrize("m1,m2,B,T", [(1, 0, 65, 31), (1, 1, 40, 24), (1, 4, 130, 45), (4, 1, 33, 26), (1, 30, 64, 41), (2, 0, 40, 33),
                                       (2, 3, 70, 25), (5, 4, 40, 30)])
def test_short_periods(m1, m2, B, T, logit, ragged):
    cfg = Config("short", B=B, T=T, n_seas=2 if m2 else 1, m1=m1, m2=m2, I=6, H=5, hidden=8, blocks=((1,),), seas_sd1=0.1,
                 seas_sd2=0.1 if m2 else 0.0, noise_sd=0.05, param_space=synth.PARAMS_LOGIT if logit else synth.PARAMS_DIRECT)
    inp = synth.make_inputs(cfg, seed=m1 + B, ragged=ragged)
    f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
    step = gc.run_gpu(cfg, inp)
    gc.check_forward(cfg, inp, step, f)
    near, side = gc.kink_sides(cfg, f, gc.valid_window_mask(cfg, inp["lengths"]), step.buffer("grad_O").cpu().numpy())
    g = oracle.backward(cfg, f, want_adjoints=True, pin_side=side if near.any() else None)
    got = step.grad_es_params.cpu().numpy()
    live = np.arange(T)[:, None] < inp["lengths"][None, :]
    terms = np.where(live, np.abs(g.gu.T) + np.abs(g.gv.T), 0.0).sum(axis=0)
    for name, rows in synth.es_param_rows(cfg).items():
        if name.endswith("init") and rows.stop - rows.start == 1:
            # A factor that applies to every step scales the level and nothing else: its gradient vanishes.  What is left is
            # rounding, a few units (four) of 2^-24 in each of the T steps, of a sum of the adjoints of the logarithms.
            scale = 1.0 if logit else inp["es_params"][rows]
            assert np.all(np.abs(got[rows] * scale) <= 4 * T * 2.0 ** -24 * terms), name
        else:
            assert gc.rel_err(got[rows], g.grad_es_params[rows]) <= gc.TOL_GRAD, name
    step.close()
