"""The fused kernel splits each leaf's planes over 1, 2, 4 or 8 workgroups by the number of
leaves in the launch.  Every face is evaluated by the same instruction sequence in every
split, so an instance's result must not depend on how many others share its launch."""
import numpy as np
import pytest

from paper_2012_04385_amd import workloads as W

pytestmark = pytest.mark.gpu


def _problem(kind):
    if kind == "sod":
        return W.sod_single_level()
    pb = W.blast_mr3()
    pb.n0, pb.lmax, pb.dx0 = (1, 1, 1), 1, 1.0 / 16
    return pb


@pytest.mark.parametrize("kind,batched", [("sod", 1), ("sod", 2), ("blast", 2)])
@pytest.mark.parametrize("copies", [13, 17, 30, 50])   # 104, 136, 240, 400 leaves: 4, 8, 2, 1 slabs
def test_result_independent_of_split(kind, batched, copies):
    from paper_2012_04385_amd.mrfv import Solver
    one = Solver([_problem(kind)], dtype="f32", batched=batched).init()
    many = Solver([_problem(kind)] * copies, dtype="f32", batched=batched).init()
    for s in (one, many):
        s.run(3)
        s.check()
    ref = one.leaf_states()
    assert len(ref) == 8
    for inst in (0, copies - 1):
        got = many.leaf_states(inst)
        assert set(got) == set(ref)
        for k in ref:
            assert np.array_equal(got[k], ref[k]), (inst, k)
    assert (many.dt == one.dt[0]).all()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("eos", ["stiffened", "tait"])
def test_stages_fused_and_through_l_agree(dtype, eos):
    """A step (fused stages, same-level neighbours read in place) against the same step put
    together from the public operators (own halos, right-hand side, update), on a tree with
    jumps, a few rounding units apart: the jump correction is added to the state in one and
    to the right-hand side in the other."""
    import torch
    from paper_2012_04385_amd.mrfv import Solver
    pb = W.sod_tait_mr3(eos=eos)
    pb.lmax = 2
    a = Solver([pb], dtype=dtype, batched=0, adapt=0).init()
    b = Solver([pb], dtype=dtype, batched=0, adapt=0).init()
    assert any(r[6] == 1 and r[2] < 2 for r in a.blocks())       # jumps
    a.step()
    b.cfl_dt()
    for stage in range(3):
        b.mr_project()
        b.fill_halos()
        b.rhs_stage()
        b.rk_update(stage)
    a.check()
    b.check()
    assert torch.equal(a.dt, b.dt)
    tol = (2e-6 if dtype == "f32" else 4e-15) * 2.5   # ~20 roundings of fields up to 2.5
    sa, sb = a.leaf_states(), b.leaf_states()
    assert set(sa) == set(sb)
    assert max(np.abs(sa[k] - sb[k]).max() for k in sa) <= tol


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("adapt", [0, 1])
def test_tait_keeps_the_energies_it_is_given(dtype, adapt):
    """Tait's equation evolves no energy; its stages pass the cells' powers of the density
    through a free energy component.  The caller's energies come back bit for bit, and the
    rest of the state is what it is with zero energies."""
    import torch
    from paper_2012_04385_amd.mrfv import Solver
    pb = W.sod_tait_mr3()
    pb.lmax, pb.eps = 2, 0.1 * pb.eps
    zero = Solver([pb], dtype=dtype, batched=0, adapt=adapt).init()
    some = Solver([pb], dtype=dtype, batched=0, adapt=adapt).init()
    some.U[:, 4] = 0.75                 # whole blocks: halos, parents and averages hold it too
    for _ in range(2):
        zero.step()
        some.step()
        some.check()
    sz, ss = zero.leaf_states(), some.leaf_states()
    assert set(sz) == set(ss)
    for k in sz:
        assert np.array_equal(sz[k][:4], ss[k][:4]), k
        assert (ss[k][4] == 0.75).all() and (sz[k][4] == 0).all(), k


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind", ["rti", "jumps"])
def test_viscous_stages_need_only_the_halos_they_fill(dtype, kind):
    """A viscous stage fills one layer of the halos beside same-level neighbours and no corner
    of a leaf.  From a state whose halos are all NaN a step gives bit for bit what the public
    operators give, which fill every halo and read no neighbour in place."""
    import torch
    from paper_2012_04385_amd.mrfv import HW, NI, Solver
    if kind == "rti":
        pb = W.rti(k=2.0, lmax=2, long_blocks=2)     # symmetry and fixed-value sides
    else:
        pb = W.sod_tait_mr3(eos="stiffened")         # zero-gradient and periodic sides
        pb.lmax, pb.mu = 2, 1e-3
    a = Solver([pb], dtype=dtype, batched=0, adapt=0).init()
    b = Solver([pb], dtype=dtype, batched=0, adapt=0).init()
    levels = {int(r[2]) for r in a.blocks() if r[6] == 1}
    assert len(levels) >= 2
    inner = a.U[:, :, HW:HW + NI, HW:HW + NI, HW:HW + NI].clone()
    a.U.fill_(float("nan"))
    a.U[:, :, HW:HW + NI, HW:HW + NI, HW:HW + NI] = inner
    a.step()
    b.cfl_dt()
    for stage in range(3):
        b.mr_project()
        b.fill_halos()
        b.rhs_stage()
        b.rk_update(stage)
    a.check()
    b.check()
    assert torch.equal(a.dt, b.dt)
    sa, sb = a.leaf_states(), b.leaf_states()
    assert set(sa) == set(sb)
    for k in sa:
        assert np.array_equal(sa[k], sb[k]), k
