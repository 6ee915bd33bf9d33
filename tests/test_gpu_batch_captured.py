"""Steps of a batch inside the caller's own graph: a replay after new states
were set, with empty cells or without, takes those states' exchange term, as an
eager step does (the replay passes no host code that could look for empty cells)."""

import numpy as np
import pytest

import workloads
from tests.gpu_util import film, log, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 4e-9, 3e-9)


@pytest.mark.parametrize("meshes", [[(20, 12, 2)], [(20, 12, 2), (9, 6, 10)]], ids=["one", "two"])
def test_replay_after_new_states(meshes):
    import torch

    import paper_2107_06729_amd as llgx
    log(f"captured batch {meshes}")
    st = llgx.make_stepper("RK4", extrap=None, h=1e-14)
    full = [to_dev(workloads.random_m(n, 8e5, 40 + i), "f64") for i, n in enumerate(meshes)]
    holes = [to_dev(workloads.masked(workloads.random_m(n, 8e5, 50 + i), workloads.checkerboard_mask(n, 4)), "f64")
             for i, n in enumerate(meshes)]

    def batch():
        bt = llgx.Batch([film(n, CELL) for n in meshes], "f64", stream=torch.cuda.Stream())
        bt.precompute_demag()
        return bt

    def load(bt, states):
        for i, m in enumerate(states):
            bt.set_m(i, m)

    def states(bt):
        return [to_host(bt.get_m(i)) for i in range(len(meshes))]

    want = []
    ref = batch()
    for s in (full, holes):
        load(ref, s)
        ref.run_fixed(st, 1, use_graph=False)
        want.append(states(ref))

    bt = batch()
    load(bt, full)
    bt.run_fixed(st, 1, use_graph=False)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=bt._stream):
        bt.run_fixed(st, 1, use_graph=False)
    for k in (1, 0, 1, 1):  # empty cells come, go, come back and stay
        load(bt, (full, holes)[k])
        torch.cuda.synchronize()
        with torch.cuda.stream(bt._stream):
            g.replay()
        torch.cuda.synchronize()
        for got, w in zip(states(bt), want[k]):
            assert np.array_equal(got, w), k
    bt.close()
    ref.close()


def test_states_set_inside_the_graph():
    """The caller's graph sets the state from a buffer of its own; an eager step
    after a replay sees the empty cells that the buffer held then."""
    import torch

    import paper_2107_06729_amd as llgx
    n = (20, 12, 2)
    log(f"captured set_m {n}")
    st = llgx.make_stepper("RK4", extrap=None, h=1e-14)
    full = to_dev(workloads.random_m(n, 8e5, 60), "f64")
    holes = to_dev(workloads.masked(workloads.random_m(n, 8e5, 61), workloads.checkerboard_mask(n, 4)), "f64")

    def batch():
        bt = llgx.Batch([film(n, CELL)], "f64", stream=torch.cuda.Stream())
        bt.precompute_demag()
        return bt

    ref = batch()
    ref.set_m(0, holes)
    ref.run_fixed(st, 1, use_graph=False)
    want = to_host(ref.get_m(0))

    bt = batch()
    buf = full.clone()
    bt.set_m(0, full)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=bt._stream):
        bt.set_m(0, buf)
    bt.run_fixed(st, 1, use_graph=False)  # looks at the full state
    buf.copy_(holes)
    torch.cuda.synchronize()
    with torch.cuda.stream(bt._stream):
        g.replay()
    bt.run_fixed(st, 1, use_graph=False)
    assert np.array_equal(to_host(bt.get_m(0)), want)
    bt.close()
    ref.close()
