"""Output stage at the edges of its tilings: hidden sizes of every padded size, horizons at and past a 16-row tile, fewer
tiles than waves and more, tiles without any window, forward-only handles and forecasts at the end of the series."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_1907_03329_amd import binding, synth
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [1, 16, 17, 33, 64])
@pytest.mark.parametrize("hidden,B,P", [(8, 33, 1), (32, 16, 3), (40, 100, 40), (41, 50, 9), (52, 130, 30), (64, 47, 13)])
def test_every_tiling(hidden, B, P, H):
    I = 8 if hidden == 8 else 12 if hidden < 40 else 12 if hidden < 64 else 20
    cfg = synth.CONFIGS["quarterly"].with_(B=B, T=I + H + P - 1, I=I, H=H, hidden=hidden, blocks=((1, 2),))
    gc.run_and_check(cfg, seed=H, ragged=True)

    # the same loss and forecasts without a reverse pass, and the out-of-sample forecasts
    inp = synth.make_inputs(cfg, seed=H, ragged=True)
    dev = {k: torch.from_numpy(v).cuda() for k, v in inp.items()}
    args = [dev[k] for k in ("y", "lengths", "es_params", "weights")]
    both, alone = binding.TrainingStep(cfg), binding.TrainingStep(cfg)
    binding.esrnn_set_forward_only(alone.handle, True)
    both.forward(*args)
    alone.forward(*args)
    assert torch.equal(both.loss, alone.loss) and torch.equal(both.forecasts, alone.forecasts)
    lengths = np.clip(inp["lengths"] - H, 0, None).astype(np.int32)
    got = both.predict(dev["y"], torch.from_numpy(lengths).cuda(), dev["es_params"], dev["weights"]).cpu().numpy()
    want = oracle.predict(cfg, inp["y"], lengths, inp["es_params"], inp["weights"])
    live = lengths >= I
    assert np.all(got[~live] == 0.0)
    if live.any():
        assert np.abs(got[live] - want[live]).max() <= gc.TOL_FWD * np.abs(want[live]).max()
