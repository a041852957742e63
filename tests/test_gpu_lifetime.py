"""A solver that is dropped gives its device memory back at once, without a collection of
cycles: programs that make many solvers in a row live on that."""
import gc
import weakref

import pytest

from paper_2012_04385_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("own_ic", [False, True])
def test_dropped_solver_frees_its_memory(own_ic):
    import torch
    from paper_2012_04385_amd.mrfv import Solver
    pb = W.sod_single_level()
    gc.collect()
    gc.disable()
    try:
        g = Solver([pb], dtype="f64", batched=0)
        g.init((lambda inst, *key: pb.primitives(*key)) if own_ic else None)
        g.step()
        torch.cuda.synchronize()
        held, ref = torch.cuda.memory_allocated(), weakref.ref(g)
        del g
        assert ref() is None
        assert torch.cuda.memory_allocated() < held
    finally:
        gc.enable()
