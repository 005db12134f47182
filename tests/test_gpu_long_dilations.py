"""Dilations at and far past the number of window positions: every position is a chain of its own."""
import pytest

from paper_1907_03329_amd.synth import CONFIGS
from tests import gpu_common as gc
from tests.test_gpu_predict import run_case

pytestmark = pytest.mark.gpu


# T = 59: 48 positions; forecasts also find what a layer needs of the one below across such a dilation, either way round
@pytest.mark.parametrize("blocks", [((1, 1 << 30), (4,)), (((1 << 31) - 1,), (3, 48), (47, 2)), ((49, 6), (1 << 30, 50))])
@pytest.mark.parametrize("narrow", ["0", "100000"])
def test_dilations_past_the_last_position(blocks, narrow, monkeypatch):
    monkeypatch.setenv("ESRNN_NARROW_BELOW", narrow)
    cfg = CONFIGS["tiny_quarterly"].with_(B=21, T=59, hidden=33, blocks=blocks)
    assert cfg.P == 48
    gc.run_and_check(cfg, seed=41, ragged=True)
    run_case(cfg, seed=42)
