"""Accuracy of the output stage, whose products are three-term sums on the bf16 matrix pipe: every one of its six contractions
(tanh layer, linear layer, their transposes, two weight gradients) has to be as accurate as fp32 products, which the
common bounds of 1e-4 / 1e-3 would not tell from products with a term missing.

Yardstick: the stage in float64, from its own inputs (block output, loss gradient), errors relative to what sums of that
many products of that size are without cancellation.  The inputs are made so that a term shows: no biases beside the sums,
pre-activations where tanh passes most of a relative error on, and for the weight gradients one window of one series, as
sums over many would average the error away.  A contraction that lacks any one of its six terms is off by 7.8e-7 or more in
the 2-norm then (3e-6 at the median), which the last test shows without a GPU against BOUND; the kernels' own errors are the
roundings of fp32 sums, of tanh and of 1 - tanh^2: 6e-8 each of their values, 3.1e-7 at most together as measured."""
import numpy as np
import pytest

from oracle import oracle
from paper_1907_03329_amd import synth

BOUND = 6e-7
# every padded hidden size; one to four 16-row tiles of the horizon
SHAPES = [(hidden, H) for hidden in (8, 32, 40, 52, 64) for H in (5, 18, 40, 60)]
BATCHES = [(1, 1), (33, 6)]     # series, window positions


def setting(hidden, H, B, P):
    I = 8 if hidden == 8 else 20 if hidden == 64 else 12
    cfg = synth.CONFIGS["quarterly"].with_(B=B, T=I + H + P - 1, I=I, H=H, hidden=hidden, blocks=((1, 2),), tau=0.43)
    inp = synth.make_inputs(cfg, seed=hidden + H)
    w = {name: inp["weights"][off:off + int(np.prod(shape))].reshape(shape) for name, off, shape in synth.weight_layout(cfg)}
    f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
    w["ba"][:] = w["bo"][:] = 0.0
    w["Wa"] *= 0.6 / np.sqrt(np.mean((f.blk[-1] @ w["Wa"].T) ** 2))
    return cfg, inp, w


def stage(r, go, w, product):
    """Outputs and gradients; product(i, a, b): a @ b, the i-th of the six contractions."""
    a = np.tanh(product(0, r, w["Wa"].T))
    dp = product(2, go, w["Wo"]) * (1.0 - a * a)
    return {"O": product(1, a, w["Wo"].T), "top": product(3, dp, w["Wa"]), "Wo": product(4, go.T, a), "Wa": product(5, dp.T, r)}


def float64(r, go, w):
    return stage(r, go, w, lambda i, a, b: a.astype(np.float64) @ b.astype(np.float64))


def sizes(r, go, w):
    """The root of the sum of squared products in the place of every sum: what terms cancel to does not matter."""
    r, go, wa, wo = (x.astype(np.float64) for x in (r, go, w["Wa"], w["Wo"]))
    a = np.tanh(r @ wa.T)
    dp = np.sqrt(go ** 2 @ wo ** 2) * (1.0 - a * a)
    return {"O": np.sqrt(a ** 2 @ wo.T ** 2), "top": np.sqrt(dp ** 2 @ wa ** 2), "Wo": np.sqrt((go ** 2).T @ a ** 2),
            "Wa": np.sqrt((dp ** 2).T @ r ** 2)}


def error(got, want, size):
    return float(np.linalg.norm(got - want) / np.linalg.norm(size))


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,H", SHAPES)
def test_products_are_as_accurate_as_fp32_products(hidden, H):
    from tests import gpu_common as gc
    for B, P in BATCHES:
        cfg, inp, w = setting(hidden, H, B, P)
        step = gc.run_gpu(cfg, inp)
        rows = lambda name, *index: step.buffer(name, *index).cpu().numpy().reshape(P * B, -1)
        inputs = rows("block_out", 0), rows("grad_O"), w
        want, size = float64(*inputs), sizes(*inputs)
        errors = {"O": error(rows("O"), want["O"], size["O"]), "top": error(rows("grad_top"), want["top"], size["top"])}
        if B == 1:
            g = step.grad_weights.cpu().numpy()
            for name, off, shape in synth.weight_layout(cfg):
                if name in ("Wa", "Wo"):
                    errors[name] = error(g[off:off + int(np.prod(shape))].reshape(shape), want[name], size[name])
        # at the end of the series
        dev = gc.to_device(inp)
        step.predict(dev["y"], dev["lengths"] - H, dev["es_params"], dev["weights"])
        inputs = rows("block_out", 0)[-B:], rows("grad_O")[-B:], w
        errors["predict"] = error(rows("O")[-B:], float64(*inputs)["O"], sizes(*inputs)["O"])
        step.close()
        print(f"  hidden {hidden} H {H} B {B}: " + ", ".join(f"{k} {v:.1e}" for k, v in errors.items()), flush=True)
        assert max(errors.values()) <= BOUND


TERMS = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]


def bf16_parts(x):
    import torch
    parts, rest = [], torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32))
    for _ in range(3):
        p = rest.to(torch.bfloat16).to(torch.float32)
        parts.append(p.numpy().astype(np.float64))
        rest = rest - p
    return parts


@pytest.mark.parametrize("hidden,H", SHAPES)
def test_the_bound_tells_a_missing_term(hidden, H):
    def product_without(contraction, term):
        def product(i, a, b):
            a, b = bf16_parts(a), bf16_parts(b)
            return sum(a[p] @ b[q] for p, q in TERMS if i != contraction or (p, q) != term)
        return product

    for B, P in BATCHES:
        cfg, inp, w = setting(hidden, H, B, P)
        f = oracle.forward(cfg, inp["y"], inp["lengths"], inp["es_params"], inp["weights"])
        g = oracle.backward(cfg, f, want_adjoints=True)
        r, go = f.blk[-1].reshape(-1, hidden).astype(np.float32), g.gO.reshape(-1, H).astype(np.float32)
        want, size, all_six = float64(r, go, w), sizes(r, go, w), stage(r, go, w, product_without(None, None))
        assert max(error(all_six[k], want[k], size[k]) for k in want) <= BOUND / 4
        for contraction, shows_in in enumerate(["O", "O", "top", "top"] + (["Wo", "Wa"] if B == 1 else [])):
            for term in TERMS:
                without = stage(r, go, w, product_without(contraction, term))
                assert error(without[shows_in], want[shows_in], size[shows_in]) > BOUND, (B, contraction, term)
