"""Weight gradients of the proposer where the samples end in a part of the long products' work:
a last block of 16 samples, or the blocks past the last full round of the 16 wavefronts.  The
samples there carry half of the loss's weight, so that a gradient without them is far off in every
layer (checked on the CPU with the oracle's gradient), and every layer is compared by itself."""
import numpy as np
import pytest

PARTS = {"W1": slice(0, 192 * 64), "W2": slice(192 * 64 + 64, 192 * 64 + 64 + 64 * 64),
         "W3": slice(192 * 64 + 64 + 64 * 64 + 64, 192 * 64 + 64 + 64 * 64 + 64 + 64 * 3)}
# (samples, first of the heavy ones): the last block, or the last part round of blocks
CASES = [(241, 240), (256, 240), (273, 272), (273, 256), (500, 256), (4097, 4096), (4000, 3840)]
# Both sides round the same operands to bfloat16; FP32 sums differ from FP64's by ~1e-6, which
# turns a rounding of 2^-9 in one operand of 4000: 6e-5 of the norm, and three layers of it.
TOL = 2e-3


def _data(rows, heavy):
    rng = np.random.default_rng([rows, heavy])
    X = rng.normal(0, 1, (rows, 192)).astype(np.float32)
    y = rng.integers(0, 2, rows).astype(np.int32)
    y[heavy:] = 2
    cw = np.array([1.0, 1.0, heavy / (rows - heavy)], dtype=np.float32)
    lim = [np.sqrt(6.0 / f) for f in (192, 64, 64)]
    p = np.concatenate([np.concatenate([rng.uniform(-lm, lm, fi * fo), np.zeros(fo)])
                        for lm, (fi, fo) in zip(lim, ((192, 64), (64, 64), (64, 3)))]).astype(np.float32)
    return X, y, cw, p


def _oracle(orc, p, X, y, cw):
    return orc.mlp_loss_grad(p.astype(np.float64), X.astype(np.float64), y, tuple(float(c) for c in cw), bf16=True)[1]


def _off(a, b, part):
    return np.linalg.norm(a[PARTS[part]] - b[PARTS[part]]) / np.linalg.norm(b[PARTS[part]])


@pytest.mark.parametrize("rows,heavy", CASES)
def test_a_lost_remainder_shows(orc, rows, heavy):
    X, y, cw, p = _data(rows, heavy)
    ref = _oracle(orc, p, X, y, cw)
    w = cw[y].astype(np.float64)
    lost = _oracle(orc, p, X[:heavy], y[:heavy], cw) * (w[:heavy].sum() / w.sum())
    for part in PARTS:
        assert _off(lost, ref, part) > 100 * TOL, part


@pytest.mark.gpu
@pytest.mark.parametrize("rows,heavy", CASES)
def test_gradient_with_a_heavy_remainder(orc, rows, heavy):
    import torch
    from paper_2012_04385_amd.mrfv import MLP
    X, y, cw, p = _data(rows, heavy)
    net = MLP(rows)
    net.set_params(p)
    _, g = net.loss_grad(torch.as_tensor(X, device="cuda:0"), y, cw)
    ref = _oracle(orc, p, X, y, cw)
    for part in PARTS:
        off = _off(g, ref, part)
        print(f"{rows} samples, {part}: {off:.2e}", flush=True)
        assert off <= TOL, part
