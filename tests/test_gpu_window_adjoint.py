"""GPU parity of the two window-adjoint kernels (the reverse of Eq. (6)'s windows: gradients of the
de-seasonalised log series and of the log level) against the float64 CPU oracle.

The library gathers per (time, series) at small batches and streams tile by tile at large ones; the
choice is made from the number of 16-series tiles when a handle is created (environment variable
ESRNN_WINDOW_STREAM_FROM: 0 = stream always, a large number = never), and windows of three row groups may
take a streaming kernel that requests a block ahead (ESRNN_WINDOW_AHEAD: 0 = never, 1 = wherever it streams).
Gather and streaming are forced onto every shape here, ragged lengths included, and compared on every series and time step (grad_u, grad_v) and in
what follows from them (gradients of the smoothing parameters)."""
import os

import pytest

from paper_1907_03329_amd.synth import CONFIGS, Config

pytestmark = pytest.mark.gpu

from tests import gpu_common as gc  # noqa: E402


class forced:
    def __init__(self, value):
        self.value = str(value)

    def __enter__(self):
        self.old = os.environ.get("ESRNN_WINDOW_STREAM_FROM")
        os.environ["ESRNN_WINDOW_STREAM_FROM"] = self.value

    def __exit__(self, *exc):
        if self.old is None:
            os.environ.pop("ESRNN_WINDOW_STREAM_FROM", None)
        else:
            os.environ["ESRNN_WINDOW_STREAM_FROM"] = self.old


def small(name, **kw):
    base = dict(name=name, B=37, T=40, n_seas=1, m1=4, m2=0, I=4, H=8, hidden=8, blocks=((1, 2), (4,)),
                tau=0.48, lambda_lv=50.0)
    base.update(kw)
    return Config(**base)


SHAPES = {
    "quarterly_70": lambda: CONFIGS["quarterly"].with_(B=70),
    "quarterly_categories_64": lambda: CONFIGS["quarterly"].with_(B=64, n_cat=6),
    "monthly_21": lambda: CONFIGS["monthly"].with_(B=21, T=90),
    "yearly_130": lambda: CONFIGS["yearly"].with_(B=130),
    "hourly_19": lambda: CONFIGS["hourly"].with_(B=19, T=300),
    "widest_windows": lambda: small("widest_windows", hidden=64, I=64, H=64, T=140, B=20, m1=12),
    "one_step_windows": lambda: small("one_step_windows", I=1, H=1, T=9, B=5, m1=2),
    "odd_widths": lambda: small("odd_widths", I=13, H=3, T=48, hidden=12),
    "no_level_penalty": lambda: small("no_level_penalty", lambda_lv=0.0, I=5, H=6),
    "single_series": lambda: small("single_series", B=1, I=3, H=5),
}


@pytest.mark.parametrize("kind", ["gather", "stream"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_each_window_adjoint_kernel_on_every_shape(shape, kind):
    cfg = SHAPES[shape]()
    with forced(0 if kind == "stream" else 1 << 30):
        errs = gc.run_and_check(cfg, seed=90, ragged=True, stages=True)
    print(f"  {shape} {kind}: grad_u {errs['grad_u']:.2e} grad_v {errs['grad_v']:.2e}", flush=True)


def test_default_choice_at_many_tiles_agrees_with_the_gather_kernel():
    """65536 quarterly series (4096 tiles) stream by default, a block requested ahead.  The oracle
    cannot run that size in the time of a test; both kernels are compared with it on every shape above,
    and here with each other on the full-size batch: the same sums in a different order."""
    import numpy as np
    import torch
    from paper_1907_03329_amd import synth
    cfg = CONFIGS["quarterly"].with_(B=65536)
    inp = synth.make_inputs(cfg, seed=91, ragged=True)
    got = {}
    for kind, value in (("default", None), ("gather", 1 << 30)):
        if value is None:
            assert "ESRNN_WINDOW_STREAM_FROM" not in os.environ
            step = gc.run_gpu(cfg, inp)
        else:
            with forced(value):
                step = gc.run_gpu(cfg, inp)
        got[kind] = {k: step.buffer(k).clone() for k in ("grad_u", "grad_v")}
        got[kind]["grad_es"] = step.grad_es_params.clone()
        step.close()
        torch.cuda.synchronize()
    live = torch.from_numpy(np.arange(cfg.T)[:, None] < inp["lengths"][None, :]).cuda()
    for k in ("grad_u", "grad_v"):
        a, b = got["default"][k], got["gather"][k]
        scale = b[live].abs().max().item()
        err = ((a - b).abs() * live).max().item() / scale
        print(f"  {k}: {err:.2e}", flush=True)
        assert err <= 2e-6, (k, err)
    a, b = got["default"]["grad_es"], got["gather"]["grad_es"]
    err = ((a - b).abs().amax(dim=1) / b.abs().amax(dim=1).clamp_min(1e-30)).max().item()
    print(f"  grad_es rows: {err:.2e}", flush=True)
    assert err <= 1e-5, err


# three row groups, and more than 3600 tiles: the kernel that requests a block ahead, on lengths that end in every place of a
# block and on tiles without a block, bit for bit what the other one (fewer series tiles) gives for the same series.  (Without the level
# penalty, whose normaliser counts all series; the comparison of the kernels at 65 536 series above has it.)
def test_blocks_requested_ahead_give_the_same_sums():
    import numpy as np
    import torch
    from paper_1907_03329_amd import binding, synth
    cfg = small("ahead", B=16 * 4096, T=40, lambda_lv=0.0)
    inp = synth.make_inputs(cfg.with_(B=4096), seed=5, ragged=True)
    rng = np.random.default_rng(6)
    lengths = np.repeat(rng.integers(cfg.I + cfg.H, cfg.T + 1, size=4096), 16).astype(np.int32)
    y = np.tile(inp["y"], (1, 16))
    es = np.tile(inp["es_params"], (1, 16))
    grads = torch.Generator(device="cuda").manual_seed(7)
    results = []
    X = O = None
    for B in (cfg.B, cfg.B - 16 * 512):
        c = cfg.with_(B=B)
        with forced(0):
            h = binding.esrnn_create(c)
        ws = torch.full((binding.esrnn_es_window_workspace_bytes(h) // 4,), float("nan"), dtype=torch.float32, device="cuda")
        dev = [torch.from_numpy(np.ascontiguousarray(v[..., :B])).cuda() for v in (y, lengths, es)]
        binding.esrnn_es_window_forward(h, *dev, ws)
        tiles = []
        for which in ("grad_X", "grad_O"):
            v = binding.esrnn_workspace_buffer(h, which)
            P, Bp, R, _ = (int(x) for x in v.dims)
            tiles.append(ws[v.offset_bytes // 4: v.offset_bytes // 4 + P * Bp * R].view(P, Bp // 16, R, 16))
        if X is None:
            X, O = (torch.randn(t.shape, generator=grads, device="cuda") for t in tiles)
        for t, g in zip(tiles, (X, O)):
            t.copy_(g[:, :B // 16])
        out = torch.empty((c.K, B), dtype=torch.float32, device="cuda")
        binding.esrnn_es_window_backward(h, *dev, ws, out)
        results.append(out.cpu().numpy())
        binding.esrnn_destroy(h)
    assert np.isfinite(results[1]).all()
    assert np.array_equal(results[0][:, :results[1].shape[1]], results[1])


# the same kernel on every way that three row groups are split and filled, on chains without a block, of one and of several, on every
# number of tiles modulo four (the last tile clears the columns that pad the batch to 64), against the other streaming kernel bit for bit
@pytest.mark.parametrize("I,H,n_cat", [(4, 8, 0), (3, 5, 0), (1, 7, 0), (6, 4, 0), (8, 1, 0), (5, 3, 6), (4, 8, 6)])
@pytest.mark.parametrize("B,positions", [(1, 3), (17, 4), (37, 5), (64, 8), (70, 13), (113, 26)])
def test_blocks_requested_ahead_on_every_shape_of_three_row_groups(I, H, n_cat, B, positions, monkeypatch):
    import numpy as np
    from paper_1907_03329_amd import binding, synth
    cfg = small("ahead", B=B, T=I + H + positions - 1, I=I, H=H, m1=2, hidden=30 if n_cat else 8, blocks=((1,),), n_cat=n_cat)
    inp = synth.make_inputs(cfg, seed=B, ragged=positions > 4)
    got = []
    for ahead in "01":
        monkeypatch.setenv("ESRNN_WINDOW_STREAM_FROM", "0")
        monkeypatch.setenv("ESRNN_WINDOW_AHEAD", ahead)
        step = gc.run_gpu(cfg, inp)
        views = [step.buffer(k).cpu().numpy() for k in ("grad_u", "grad_v")]
        v = binding.esrnn_workspace_buffer(step.handle, "grad_u", 0)
        padded = step.workspace[v.offset_bytes // 4: v.offset_bytes // 4 + int(v.dims[0]) * int(v.dims[1])].view(int(v.dims[0]), -1)
        got.append(views + [padded[:, 16 * -(-B // 16):].cpu().numpy(), step.grad_es_params.cpu().numpy()])
        step.close()
    assert all(np.isfinite(a).all() and np.array_equal(a, b) for a, b in zip(*got))
    assert not got[1][2].any()
