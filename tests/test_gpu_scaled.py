"""The flux kernels in FP64 on states far from one: a tube with a jump between two gently varying
gases, whose density and energy are multiplied by a power of two (sound speeds keep their
values, so the right-hand side is that of the tube times the power, but for the
reconstructions' eps).  With 2^264 the WENO-AO indicators of candidates across the jump overflow
when they are squared: their weights vanish and the smooth candidates' value, which differs
from the cell's own by 1e-5, is the answer, as in the oracle."""
import numpy as np
import pytest

from gpu_helpers import make_pair, oracle_padded_to_gpu, slot_map
from paper_2012_04385_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [("hllc_wao53", 0), ("hllc_wao53", 100), ("hllc_wao53", 264), ("roe_weno5", 100), ("roe_teno5", -100),
         ("llf_weno5", -100)]


@pytest.mark.parametrize("scheme,power", CASES)
def test_rhs_of_a_scaled_tube(orc, scheme, power):
    import torch
    s = 2.0 ** power

    def tube(x, y, z):
        f = s * (1.0 + 2e-3 * np.sin(2 * np.pi * x)) * np.where(x < 0.5, 1.0, 0.125)
        return f, 0.0 * x, 0.0 * x, 0.0 * x, 0.8 * f

    pb = W.Problem(name="tube", kind="custom", custom=tube, lmax=0, n0=(2, 1, 1), dx0=1.0 / 32, bc=(1, 0, 0), noise=0.0,
                   scheme=scheme)
    o, g = make_pair(orc, pb, (), "f64", False)
    o.fill_halos()
    oracle_padded_to_gpu(o, g)
    ref = o.rhs()
    g.rhs_stage()
    torch.cuda.synchronize()
    got = g.L.cpu().numpy()
    gm = slot_map(g)
    for i, r in enumerate(o.blocks()):
        mine, scale = got[gm[tuple(int(v) for v in r[:4])]], np.abs(ref[i]).max()
        assert np.isfinite(mine).all() and np.isfinite(scale) and scale > 0
        assert np.abs(mine - ref[i]).max() <= 1e-10 * scale
