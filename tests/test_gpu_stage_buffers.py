"""The two state buffers of the fused stages (W, W2) in contexts that do not get them when they
are created: who takes them, what runs where they cannot be had, and who gives them back.
Memory is read from the device; a filler tensor stands for a caller's other data."""
import gc

import numpy as np
import pytest

from gpu_helpers import N, make_pair, random_physical, same_tree, set_interiors
from paper_2012_04385_amd import workloads as W

pytestmark = pytest.mark.gpu

SLAB, FACE, CELLS_P = 3 * 16 * 16, 16 * 16, 24 ** 3


@pytest.fixture
def torch_mod():
    import torch
    assert torch.cuda.is_available()
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch


def _blast():
    from paper_2012_04385_amd.mrfv import Solver
    pb = W.blast_mr3()
    pb.n0, pb.lmax, pb.dx0 = (6, 6, 6), 1, 1.0 / 96
    return Solver([pb], dtype="f64", batched=0, adapt=0)


def _free(torch):
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _filler(torch, leave):
    """A tensor that leaves `leave` bytes of the card free."""
    return torch.empty(_free(torch) - int(leave), dtype=torch.uint8, device="cuda:0")


def test_only_a_global_step_takes_them(torch_mod):
    g = _blast()
    state = g.capacity * 5 * CELLS_P * 8
    lts = g.capacity * 5 * (CELLS_P + 6 * SLAB + 6 * FACE) * 8
    before = _free(torch_mod)
    g.init()
    g.mr_project()
    g.fill_halos()
    g.rhs_stage()
    g.cfl_dt()
    g.mr_flag()
    g.totals()
    assert before - _free(torch_mod) < state // 4
    g.step_lts()
    assert before - _free(torch_mod) < lts + state // 4
    g.step()
    g.check()
    assert before - _free(torch_mod) > lts + 1.5 * state


@pytest.mark.parametrize("room", [True, False])
def test_small_contexts_take_them_with_the_tree(torch_mod, room):
    from paper_2012_04385_amd.mrfv import Solver
    fill = None if room else _filler(torch_mod, 0.2 * torch_mod.cuda.mem_get_info()[1])
    pb = W.sod_single_level()
    pb.n0, pb.dx0 = (10, 10, 9), 1.0 / 160
    g = Solver([pb], dtype="f64", batched=0)
    state = g.capacity * 5 * CELLS_P * 8
    before = _free(torch_mod)
    g.init()
    taken = before - _free(torch_mod)
    assert taken > 1.5 * state if room else taken < state // 4
    del fill


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", [(0, 1, 0), (2, 1, 0)])
def test_refused_stages_match_the_oracle(orc, torch_mod, dtype, bc):
    """With less than a quarter of the card free the stages go through L and say so: one step on a
    tree with one- and two-level jumps, the bounds of the same step on the fused path."""
    from paper_2012_04385_amd.mrfv import lib
    fill = _filler(torch_mod, 0.2 * torch_mod.cuda.mem_get_info()[1])
    pb = W.uniform_flow(lmax=3, n0=(2, 2, 2))
    pb.bc = bc
    o, g = make_pair(orc, pb, [(1, 1, 1, 1), (1, 2, 1, 1), (2, 3, 2, 2), (1, 0, 3, 0)], dtype, False)
    rng = np.random.default_rng(5)
    set_interiors(o, g, lambda k: random_physical(rng, (N, N, N), rough=0.01))
    o.project()
    g.mr_project()
    before = _free(torch_mod)
    dt_o = o.step()
    g.step()
    g.check()
    assert before - _free(torch_mod) < g.capacity * 5 * CELLS_P * 4
    assert b"stage buffers" in lib().mrfv_last_error(g.h)
    del fill
    assert abs(float(g.dt.cpu()[0]) - dt_o) <= (1e-14 if dtype == "f64" else 1e-6) * dt_o
    ol, gl = o.leaf_states(), g.leaf_states()
    for k, v in ol.items():
        assert np.abs(gl[k] - v).max() / np.abs(v).max() < (1e-12 if dtype == "f64" else 2e-6), k


@pytest.mark.parametrize("eos", ["stiffened", "tait"])
def test_refused_adaptive_steps_match_the_oracle(orc, torch_mod, eos):
    fill = _filler(torch_mod, 0.2 * torch_mod.cuda.mem_get_info()[1])
    pb = W.sod_tait_mr3(eos=eos)
    pb.lmax = 2
    o, g = make_pair(orc, pb, (), "f64", adapt=1)
    for m in range(4):
        o.step()
        g.step()
        ok, ol, gl = same_tree(o, g)
        assert ok, (m, ol ^ gl)
    g.check()
    del fill
    ol, gl = o.leaf_states(), g.leaf_states()
    assert max(np.abs(gl[k] - v).max() / np.abs(v).max() for k, v in ol.items()) < 1e-11


def test_local_time_stepping_gets_their_memory(torch_mod):
    """A context that has taken the buffers still gets those of local time stepping on a card
    that has room for either: the results are those of a card with room for both."""
    ref = _blast().init()
    ref.step()
    ref.step_lts()
    want = ref.leaf_states()
    ref.close()
    del ref
    g = _blast().init()
    g.step()
    fill = _filler(torch_mod, 0.5e9)
    g.step_lts()
    g.check()
    got = g.leaf_states()
    g.step()                     # and global steps go on
    g.check()
    del fill
    assert set(got) == set(want)
    for k in want:
        assert np.array_equal(got[k], want[k]), k


def test_no_allocation_while_the_caller_captures(torch_mod):
    """The first step inside a caller's capture takes no memory; the step after it does and
    gives what it gives without the capture.  (The graph is only recorded.)"""
    torch = torch_mod
    ref = _blast().init()
    ref.step()
    want = ref.leaf_states()
    ref.close()
    del ref
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g = _blast().init()
        s.synchronize()
        gc.collect()
        torch.cuda.empty_cache()   # as entering a capture does
        before = _free(torch)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            g.step()
        assert before - _free(torch) < g.capacity * 5 * CELLS_P * 4
        del graph
        before = _free(torch)
        g.step()
        g.check()
        assert before - _free(torch) > 1.5 * g.capacity * 5 * CELLS_P * 8
        got = g.leaf_states()
    for k in want:
        assert np.array_equal(got[k], want[k]), k
