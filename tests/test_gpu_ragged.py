"""Ragged batches cost what they contain (Section 8.1): every kernel stops a 16-series tile at its longest
series.  What lies beyond is never computed, so it must never be read either: these tests fill the whole
workspace with NaN first, then run ragged batches - lengths sorted (most tiles far shorter than T), unsorted,
and with one tile of minimum-length series - and compare with the float64 oracle as usual."""
import numpy as np
import pytest

from oracle import oracle
from paper_1907_03329_amd import binding, synth
from paper_1907_03329_amd.synth import CONFIGS, Config

pytestmark = pytest.mark.gpu

from tests import gpu_common as gc  # noqa: E402


def run_poisoned(cfg, inp):
    import torch
    step = binding.TrainingStep(cfg)
    step.workspace.fill_(float("nan"))
    step.forecasts.fill_(float("nan"))
    dev = gc.to_device(inp)
    if "categories" in dev:
        step.set_categories(dev["categories"])
    step.forward(dev["y"], dev["lengths"], dev["es_params"], dev["weights"])
    step.backward(dev["y"], dev["lengths"], dev["es_params"], dev["weights"])
    torch.cuda.synchronize()
    return step


def check(cfg, inp, stages=True):
    f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"], categories=inp.get("categories"))
    step = run_poisoned(cfg, inp)
    errs = gc.check_forward(cfg, inp, step, f, stages)
    errs.update(gc.check_backward(cfg, inp, step, f, None, stages))
    assert np.all(np.isfinite(step.grad_weights.cpu().numpy())) and np.all(np.isfinite(step.grad_es_params.cpu().numpy()))
    step.close()
    return errs


def with_lengths(cfg, seed, order):
    inp = synth.make_inputs(cfg, seed=seed, ragged=True)
    lo = cfg.I + cfg.H + max(cfg.m1, cfg.m2, 2)
    rng = np.random.default_rng(seed)
    n = rng.integers(lo, cfg.T + 1, size=cfg.B).astype(np.int32)
    if order == "sorted":
        n = np.sort(n)[::-1].copy()
    elif order == "short_tile":
        n[16:32] = cfg.I + cfg.H                 # one tile with a single window per series
    inp["lengths"] = n
    inp["y"][np.arange(cfg.T)[:, None] >= n[None, :]] = 1.0
    return inp


@pytest.mark.parametrize("order", ["sorted", "unsorted", "short_tile"])
@pytest.mark.parametrize("kind", ["narrow", "wide"])
def test_ragged_batch_on_a_poisoned_workspace(order, kind):
    import os
    cfg = CONFIGS["quarterly"].with_(B=150, T=60)
    old = os.environ.get("ESRNN_NARROW_BELOW")
    os.environ["ESRNN_NARROW_BELOW"] = "0" if kind == "wide" else str(1 << 30)
    try:
        errs = check(cfg, with_lengths(cfg, 90, order))
    finally:
        if old is None:
            os.environ.pop("ESRNN_NARROW_BELOW", None)
        else:
            os.environ["ESRNN_NARROW_BELOW"] = old
    print(f"  {order} {kind}: worst {max(v for k, v in errs.items() if k != 'series_at_kink'):.2e}", flush=True)


def test_ragged_double_seasonality_three_blocks_categories_penalty():
    cfg = Config(name="ragged_mix", B=70, T=80, n_seas=2, m1=3, m2=7, seas_sd2=0.1, I=5, H=6, hidden=30,
                 blocks=((1, 3), (5,), (2,)), n_cat=6, lambda_c=0.5)
    inp = with_lengths(cfg, 91, "sorted")
    errs = check(cfg, inp)
    print(f"  worst {max(v for k, v in errs.items() if k != 'series_at_kink'):.2e}", flush=True)


def test_out_of_sample_forecasts_on_a_poisoned_workspace():
    import torch
    cfg = CONFIGS["quarterly"].with_(B=90, T=60)
    inp = with_lengths(cfg, 92, "sorted")
    inp["lengths"] = np.minimum(inp["lengths"], cfg.T - cfg.H).astype(np.int32)
    step = binding.TrainingStep(cfg, want_forecasts=False)
    step.workspace.fill_(float("nan"))
    dev = gc.to_device(inp)
    got = step.predict(dev["y"], dev["lengths"], dev["es_params"], dev["weights"]).cpu().numpy()
    want = oracle.predict(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
    rel = np.abs(got - want).max(axis=1) / np.abs(want).max(axis=1)
    assert rel.max() <= 1e-4, rel.max()
    step.close()


# Forecasts leave out what they do not depend on: it is NaN here and must not be read where it counts.  Six tiles: with
# a threshold of 20 workgroups the layers of dilation 1 to 3 run on the 4-series kernels, which compute every class, the
# others on the 16-series kernels, which skip classes; a layer with the penalty computes every class on either.
@pytest.mark.parametrize("narrow", ["0", "20", "100000"])
@pytest.mark.parametrize("blocks", [((1, 2), (4, 8)), ((8, 4), (2, 1)), ((3, 6), (9,), (2,)), ((12,), (1, 10), (5,))])
@pytest.mark.parametrize("penalty", [0.0, 1.0])
def test_forecasts_skip_classes_on_a_poisoned_workspace(narrow, blocks, penalty, monkeypatch):
    import torch
    monkeypatch.setenv("ESRNN_NARROW_BELOW", narrow)
    cfg = CONFIGS["quarterly"].with_(B=90, T=60, blocks=blocks, lambda_c=penalty)
    for order in ("unsorted", "short_tile", "alike"):
        inp = with_lengths(cfg, 93, order)
        inp["lengths"] = np.minimum(inp["lengths"], cfg.T - cfg.H).astype(np.int32)
        if order == "alike":
            inp["lengths"][:] = 41 - np.arange(cfg.B) // 16         # one class of most dilations in every tile
            inp["lengths"][5] = cfg.I - 1                           # a series that takes no part
        step = binding.TrainingStep(cfg, want_forecasts=False)
        step.workspace.fill_(float("nan"))
        dev = gc.to_device(inp)
        got = step.predict(dev["y"], dev["lengths"], dev["es_params"], dev["weights"]).cpu().numpy()
        ok = inp["lengths"] >= cfg.I
        want = oracle.predict(cfg, inp["y"], np.where(ok, inp["lengths"], cfg.T - cfg.H).astype(np.int32), inp["es_params"], inp["weights"])
        assert np.all(got[~ok] == 0.0)
        rel = (np.abs(got - want).max(axis=1) / np.abs(want).max(axis=1))[ok]
        assert rel.max() <= 1e-4, (order, rel.max())
        step.close()
