"""Weight gradients of the proposer: sums over the samples split over 16 wavefronts from 256
(padded) samples on, one wavefront below.  Sample counts around the switch and a block's
edge, against the oracle with the same bfloat16 roundings (without them a ReLU near zero opens
in one and not in the other: 4 % of the gradient's norm at 240 samples)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [15, 240, 241, 256, 273, 4097])
def test_gradient_of_any_sample_count(orc, rows):
    import torch
    from paper_2012_04385_amd.mrfv import MLP
    rng = np.random.default_rng(rows)
    net = MLP(rows)
    p = net.init_params(3)
    X = rng.normal(0, 1, (rows, 192)).astype(np.float32)
    y = rng.integers(0, 3, rows).astype(np.int32)
    _, g = net.loss_grad(torch.as_tensor(X, device="cuda:0"), y, np.ones(3, np.float32))
    _, ref = orc.mlp_loss_grad(p.astype(np.float64), X.astype(np.float64), y, (1.0, 1.0, 1.0), bf16=True)
    # bfloat16 operands: 2^-9 relative each, three layers deep
    assert np.linalg.norm(g - ref) <= 3e-2 * np.linalg.norm(ref)
