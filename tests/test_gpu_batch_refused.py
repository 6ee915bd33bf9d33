"""A batch call that is refused changes no sample: every mesh group is checked
before any of them is stepped, so groups stay at one time."""

import numpy as np
import pytest

import workloads
from tests.gpu_util import film, log, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 4e-9, 3e-9)
MESHES = [(20, 12, 2), (9, 6, 10)]


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("launch", ["streams", "jobs"])
def test_a_group_without_magnetization_leaves_the_others(launch, graph):
    import torch

    import paper_2107_06729_amd as llgx
    log(f"refused batch {launch} {graph}")
    M = [workloads.random_m(n, 8e5, 30 + i) for i, n in enumerate(MESHES)]
    st = llgx.make_stepper("RK4", extrap=2, h=1e-14)

    def batch():
        bt = llgx.Batch([film(n, CELL) for n in MESHES], "f64", stream=torch.cuda.Stream())
        bt.set_launch(launch)
        bt.precompute_demag()
        bt.set_m(0, to_dev(M[0], "f64"))
        return bt

    bt = batch()
    with pytest.raises(llgx.LlgxError):
        bt.run_fixed(st, 6, use_graph=graph)
    assert bt.info()["t"] == 0.0
    assert np.array_equal(to_host(bt.get_m(0)), M[0])
    # after the missing call the batch steps as one that was never refused
    want = batch()
    for b in (bt, want):
        b.set_m(1, to_dev(M[1], "f64"))
        b.run_fixed(st, 6, use_graph=graph)
    assert bt.info()["t"] == want.info()["t"]
    for i in range(2):
        assert np.array_equal(to_host(bt.get_m(i)), to_host(want.get_m(i))), i
    bt.close()
    want.close()
