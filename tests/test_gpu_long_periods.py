"""Smoothing recursions with long periods (three chunks of eight steps and more take a kernel of their own): periods at that
limit and past it, lengths that are no multiple of a chunk, rings that end inside a chunk, padded batches."""
import pytest

from paper_1907_03329_amd import synth
from paper_1907_03329_amd.synth import Config
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logit", [False, True])
@pytest.mark.parametrize("m1,m2,B,T", [(23, 0, 40, 70), (24, 0, 40, 71), (24, 0, 1100, 49), (29, 0, 70, 200), (40, 0, 17, 48),
                                       (24, 37, 64, 131), (25, 24, 65, 100), (24, 200, 33, 260), (24, 23, 33, 90)])
def test_long_periods(m1, m2, B, T, logit):
    cfg = Config("long", B=B, T=T, n_seas=2 if m2 else 1, m1=m1, m2=m2, I=6, H=5, hidden=8, blocks=((1,),), seas_sd1=0.1,
                 seas_sd2=0.1 if m2 else 0.0, noise_sd=0.05, param_space=synth.PARAMS_LOGIT if logit else synth.PARAMS_DIRECT)
    gc.run_and_check(cfg, seed=m1 + B)
    gc.run_and_check(cfg, seed=m2 + T, ragged=True)
