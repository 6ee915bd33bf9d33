"""Steps of a batch that are not replayed run each mesh group on a stream of its own,
joined back before anything else reads or writes the states: the same bits as the
groups one after another (job-table batches), copies enqueued right before and after."""

import numpy as np
import pytest

import workloads
from tests.gpu_util import film, log, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 4e-9, 3e-9)
MESHES = [(130, 70, 3), (21, 13, 1), (64, 32, 6)]


@pytest.mark.parametrize("method,extrap,graph,renormalize", [("RK4", 4, True, False), ("RK4", 3, False, True),
                                                             ("RK23", None, False, False), ("HEUN", 1, True, True)])
def test_forked_eager_steps_equal_serial(method, extrap, graph, renormalize):
    import torch

    import paper_2107_06729_amd as llgx
    log(f"forked {method} {extrap} {graph}")
    stream = torch.cuda.Stream()
    got = []
    for launch in ("jobs", "streams"):
        bt = llgx.Batch([film(n, CELL, Ha=(h, 1e3, 0.0)) for n in MESHES for h in (1e4, -2e4)], "f32", stream=stream)
        bt.set_launch(launch)
        bt.precompute_demag()
        outs = []
        for run in range(2):  # the second run overwrites states that the first one's streams used
            for i in range(6):
                bt.set_m(i, to_dev(workloads.random_m(MESHES[i // 2], 8e5, 60 + 10 * run + i), "f32"))
            bt.run_fixed(llgx.make_stepper(method, extrap=extrap, h=1e-14, renormalize=renormalize), 7, use_graph=graph)
            outs += [bt.get_m(i) for i in range(6)]
        got.append([to_host(o) for o in outs])
        bt.close()
    for a, b in zip(*got):
        assert np.isfinite(a).all() and np.array_equal(a, b)


def test_renormalised_steps_do_not_replay_plain_ones():
    """Graphs of steps with and without renormalisation are different ones."""
    import torch

    from tests.gpu_util import sim
    import paper_2107_06729_amd as llgx
    n = (40, 24, 2)
    s = sim(film(n, CELL), "f64", stream=torch.cuda.Stream())
    s.set_m(to_dev(workloads.random_m(n, 8e5, 70), "f64"))
    plain = llgx.make_stepper("HEUN", extrap=1, h=2e-13)
    renorm = llgx.make_stepper("HEUN", extrap=1, h=2e-13, renormalize=True)

    def drift():
        return float(np.abs(np.sqrt((to_host(s.get_m()) ** 2).sum(axis=0)) / 8e5 - 1.0).max())
    s.run_fixed(plain, 12)
    assert drift() > 1e-9
    s.run_fixed(renorm, 12)
    assert drift() < 1e-14
