"""The split of leaves over workgroups in the forms that a single-level FP32 batch does not reach:
FP64, whose rule counts one workgroup per CU (copies of a tube give 4, 2, 8 and 1 slabs per leaf),
Tait's system with its powers in the stage buffers, and a tree with jumps.  An instance's result
must not depend on how many others share its launch."""
import numpy as np
import pytest

from paper_2012_04385_amd import workloads as W

pytestmark = pytest.mark.gpu


def _tube(eos):
    if eos == "single":
        return W.sod_single_level()
    pb = W.sod_tait_mr3(eos=eos)      # 72 leaves on two levels
    pb.lmax = 2
    return pb


@pytest.mark.parametrize("dtype,eos,copies", [
    ("f64", "single", 5), ("f64", "single", 13), ("f64", "single", 17), ("f64", "single", 25),
    ("f64", "stiffened", 3), ("f64", "stiffened", 4), ("f64", "tait", 3), ("f64", "tait", 4),
    ("f32", "stiffened", 3), ("f32", "tait", 3), ("f32", "tait", 4)])
def test_result_independent_of_split(dtype, eos, copies):
    from paper_2012_04385_amd.mrfv import Solver
    one = Solver([_tube(eos)], dtype=dtype, batched=0, adapt=0).init()
    many = Solver([_tube(eos)] * copies, dtype=dtype, batched=0, adapt=0).init()
    assert eos == "single" or {int(r[2]) for r in one.blocks() if r[6] == 1} == {1, 2}
    for s in (one, many):
        s.run(2)
        s.check()
    ref = one.leaf_states()
    for inst in (0, copies - 1):
        got = many.leaf_states(inst)
        assert set(got) == set(ref)
        for k in ref:
            assert np.array_equal(got[k], ref[k]), (inst, k)
    assert (many.dt == one.dt[0]).all()
