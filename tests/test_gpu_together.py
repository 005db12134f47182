"""Layers that follow each other in one launch against the same layers in launches of their own: every result is the same, bit
for bit, however the workgroups of the layers overtake each other."""
import re

import numpy as np
import pytest
import torch

from paper_1907_03329_amd import binding, synth

pytestmark = pytest.mark.gpu


# chains around a chunk of staged inputs, fewer positions than classes, tiles that end at different positions, hidden sizes of
# every instantiation, rising and falling dilations, layers that end a block or not, last layers of either kind; and how many
# layers share a launch, forward and reverse
CASES = {
    "serve": ((4, 4), dict(B=7)),
    "eight_tiles_and_more": ((2, 2), dict(B=145, blocks=((1,), (3,)))),
    "16_series_layer_last": ((2, 0), dict(B=512, blocks=((1, 4), (2, 8)))),
    "16_series_layer_ends_a_block": ((2, 0), dict(B=400, blocks=((1,), (5,), (2,)), hidden=50, I=12)),
    "several_narrow_layers_then_16_series": ((3, 2), dict(B=160, blocks=((1, 2), (8,)))),
    "falling_dilations": ((3, 3), dict(B=40, blocks=((4, 2), (1,)))),
    "one_position": ((2, 2), dict(B=20, T=24, H=20, blocks=((1,), (1,)))),
    "few_positions": ((4, 4), dict(B=33, T=32, H=24, blocks=((1, 2), (9, 3)))),
    "few_positions_whose_outputs_hold_fewer_words": ((2, 4), dict(B=33, T=16, blocks=((1, 2), (9, 3)))),
    "nine_positions": ((4, 4), dict(B=33, T=20, blocks=((1, 1), (1, 2)))),
    "many_layers": ((6, 6), dict(B=18, T=40, blocks=((1, 2, 1), (2, 1, 3)))),
    "more_layers_than_a_launch_has": ((8, 0), dict(B=18, T=40, blocks=((1, 2, 1), (2, 1, 3), (1, 2, 1)))),
    "hidden_50": ((4, 4), dict(B=21, hidden=50, I=12, blocks=((1, 3), (2, 6)))),
    "hidden_8": ((3, 2), dict(B=50, hidden=8, blocks=((1, 2), (3,)))),
    "hidden_30": ((3, 3), dict(B=100, hidden=30, I=6, blocks=((1, 2), (2, 6)))),
    "hidden_64": ((3, 3), dict(B=36, hidden=64, I=40, T=90, blocks=((1, 2), (4,)))),
    "hidden_64_16_series": ((2, 0), dict(B=300, hidden=64, I=40, T=90, blocks=((1, 4), (4,)))),
    "penalty": ((4, 4), dict(B=70, hidden=50, I=12, blocks=((1, 3), (2, 6)), lambda_c=0.3, n_cat=6)),
    "penalty_16_series_layer_starts_a_block": ((2, 0), dict(B=400, hidden=50, I=12, blocks=((1,), (5,)), lambda_c=0.3, n_cat=6)),
    "penalty_16_series": ((2, 0), dict(B=501, hidden=50, I=12, blocks=((1, 3), (2, 6)), lambda_c=0.3, n_cat=6)),
}


def shared(handle):
    """How many layers share a launch, forward and reverse."""
    n = dict(forward=0, backward=0)
    for name, _, _ in binding.esrnn_profile_read(handle):
        found = re.fullmatch(r"lstm_(forward|backward)_l0_to_l(\d+)", name)
        if found:
            n[found[1]] = int(found[2]) + 1
    return n["forward"], n["backward"]


def results(cfg, launches, monkeypatch, repeat):
    """Per pass: loss, forecasts, gradients, out-of-sample forecasts, and all arrays of the training step (its workspace, bit by bit).
    Every pass finds NaN wherever it has not written yet, and so does whoever reads there too early."""
    if launches == (0, 0):
        monkeypatch.setenv("ESRNN_TOGETHER", "0")
    else:
        monkeypatch.delenv("ESRNN_TOGETHER", raising=False)
    inp = synth.make_inputs(cfg, seed=3, ragged=True)
    dev = {k: torch.from_numpy(v).cuda() for k, v in inp.items()}
    step = binding.TrainingStep(cfg)
    assert shared(step.handle) == launches
    if cfg.n_cat:
        step.set_categories(dev["categories"])
    view = binding.esrnn_workspace_buffer(step.handle, "O", 0)
    outputs = slice(view.offset_bytes // 4, view.offset_bytes // 4 + int(np.prod([int(d) for d in view.dims[:3]])))
    ahead = torch.clamp(dev["lengths"] - cfg.H, min=cfg.I + max(cfg.m1, 2))
    out = []
    for _ in range(repeat):
        step.workspace.fill_(float("nan"))
        step.forward(dev["y"], dev["lengths"], dev["es_params"], dev["weights"])
        step.backward(dev["y"], dev["lengths"], dev["es_params"], dev["weights"])
        got = [step.loss, step.forecasts, step.grad_es_params, step.grad_weights]
        got = [t.cpu().numpy().copy() for t in got]
        arrays = step.workspace.view(torch.int32).clone()
        arrays[outputs] = 0     # (rows past a tile's last position hold whatever was there before)
        step.grad_weights.fill_(float("nan"))       # (a reverse pass may be run again)
        step.backward(dev["y"], dev["lengths"], dev["es_params"], dev["weights"])
        assert np.array_equal(step.grad_weights.cpu().numpy(), got[3])
        step.workspace.fill_(float("nan"))
        got.append(step.predict(dev["y"], ahead, dev["es_params"], dev["weights"]).cpu().numpy().copy())
        out.append((got, arrays))
    step.close()
    return out


@pytest.mark.parametrize("case", sorted(CASES))
def test_layers_of_one_launch_are_those_of_several(case, monkeypatch):
    launches, fields = CASES[case]
    cfg = synth.CONFIGS["quarterly"].with_(**fields)
    (want, want_arrays), = results(cfg, (0, 0), monkeypatch, 1)
    assert all(np.isfinite(w).all() for w in want)
    for got, arrays in results(cfg, launches, monkeypatch, 3):
        for name, g, w in zip(("loss", "forecasts", "grad_es", "grad_weights", "ahead"), got, want):
            assert np.array_equal(g, w), name
        # (the words of the reverse pass, cleared, lie where the output stage's operands were)
        assert int(((arrays != want_arrays) & (arrays != 0)).sum()) == 0


def test_profiling_times_the_launches_of_the_step():
    """The stages that are timed are those that a step runs, and timing them changes no result."""
    cfg = synth.CONFIGS["quarterly"].with_(B=16)
    inp = synth.make_inputs(cfg, seed=3, ragged=True)
    dev = {k: torch.from_numpy(v).cuda() for k, v in inp.items()}
    step = binding.TrainingStep(cfg)
    results = []
    for on in (False, True):
        binding.esrnn_profile_enable(step.handle, on)
        step.forward(dev["y"], dev["lengths"], dev["es_params"], dev["weights"])
        step.backward(dev["y"], dev["lengths"], dev["es_params"], dev["weights"])
        results.append([t.cpu().numpy().copy() for t in (step.loss, step.forecasts, step.grad_es_params, step.grad_weights)])
    binding.esrnn_profile_collect(step.handle)
    stages = {name: count for name, _, count in binding.esrnn_profile_read(step.handle) if count}
    assert stages == dict.fromkeys(["es_forward", "window_forward", "lstm_forward_l0_to_l3", "head_forward_backward", "forecasts",
                                    "lstm_backward_l0_to_l3", "window_backward", "es_backward"], 1)
    assert all(np.array_equal(a, b) for a, b in zip(*results))
    step.close()


def test_two_streams_at_once():
    """Launches of two handles that do not fit the chip together (240 and 192 workgroups of the reverse pass, one a compute unit):
    what a workgroup waits for runs, whichever of them the chip takes first."""
    steps, streams, want, got = [], [], [], []
    for seed, fields in ((5, dict(B=320, blocks=((1, 2),))), (6, dict(B=256, blocks=((2, 1),)))):
        cfg = synth.CONFIGS["quarterly"].with_(**fields)
        dev = {k: torch.from_numpy(v).cuda() for k, v in synth.make_inputs(cfg, seed=seed, ragged=True).items()}
        step = binding.TrainingStep(cfg)
        assert shared(step.handle) == (2, 2)
        steps.append((step, [dev[k] for k in ("y", "lengths", "es_params", "weights")]))
        streams.append(torch.cuda.Stream())

    def one(step, args):
        step.forward(*args)
        step.backward(*args)

    def copies(step):
        return [t.clone() for t in (step.loss, step.forecasts, step.grad_es_params, step.grad_weights)]

    for step, args in steps:
        one(step, args)
        want.append(copies(step))
    torch.cuda.synchronize()
    for _ in range(10):
        for (step, args), stream in zip(steps, streams):
            with torch.cuda.stream(stream):
                one(step, args)
    for (step, args), stream in zip(steps, streams):
        with torch.cuda.stream(stream):
            got.append(copies(step))
    torch.cuda.synchronize()
    for w, g in zip(want, got):
        assert all(torch.equal(a, b) for a, b in zip(w, g))
    for step, _ in steps:
        step.close()
