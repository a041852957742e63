"""Weight gradients of the proposer: sums over the samples split over 16 wavefronts from 256
(padded) samples on, one wavefront below.  Sample counts around the switch and a block's
edge, against the gradient in FP64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [15, 240, 241, 256, 273, 4097])
def test_gradient_of_any_sample_count(rows):
    import torch
    from paper_2012_04385_amd.mrfv import MLP
    rng = np.random.default_rng(rows)
    net = MLP(rows)
    p = net.init_params(3)
    X = rng.normal(0, 1, (rows, 192)).astype(np.float32)
    y = rng.integers(0, 3, rows).astype(np.int32)
    _, g = net.loss_grad(torch.as_tensor(X, device="cuda:0"), y, np.ones(3, np.float32))
    ps, at = [], 0
    for fi, fo in ((192, 64), (64, 64), (64, 3)):
        for shape in ((fi, fo), (fo,)):
            n = int(np.prod(shape))
            ps.append(torch.tensor(p[at:at + n].astype(np.float64)).reshape(shape).requires_grad_())
            at += n
    h = torch.tensor(X.astype(np.float64))
    for k in range(3):
        h = h @ ps[2 * k] + ps[2 * k + 1]
        h = torch.relu(h) if k < 2 else h
    torch.nn.functional.cross_entropy(h, torch.tensor(y.astype(np.int64))).backward()
    ref = np.concatenate([q.grad.reshape(-1).numpy() for q in ps])
    # bfloat16 operands: 2^-9 relative each, three layers deep
    assert np.linalg.norm(g - ref) <= 3e-2 * np.linalg.norm(ref)
