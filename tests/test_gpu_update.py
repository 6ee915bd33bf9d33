"""Steps with exact fields only: the last stage's x pass writes Eq. (3) itself;
job-table steps of a batch keep the update in a launch of its own, and the two must
agree bit for bit, with empty cells, rows that end inside a block and one x cell."""

import numpy as np
import pytest

import workloads
from tests.gpu_util import film, log, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 4e-9, 3e-9)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("method", ["RK4", "HEUN", "RKF45", "RK23"])
def test_update_in_the_x_pass_equals_separate(method, prec):
    import torch

    import paper_2107_06729_amd as llgx
    log(f"update {method} {prec}")
    meshes = [(21, 13, 3), (70, 9, 1), (1, 33, 6)]
    stream = torch.cuda.Stream()
    got = []
    for launch in ("jobs", "streams"):
        bt = llgx.Batch([film(n, CELL, K=2e4, Ha=(h, 1e3, 0.0)) for n in meshes for h in (1e4, -2e4)], prec, stream=stream)
        bt.set_launch(launch)
        bt.precompute_demag()
        with torch.cuda.stream(stream):
            for i in range(6):
                n = meshes[i // 2]
                M = workloads.random_m(n, 8e5, 80 + i)
                if i % 2:
                    M = workloads.masked(M, workloads.checkerboard_mask(n, 4))
                bt.set_m(i, to_dev(M, prec))
        bt.run_fixed(llgx.make_stepper(method, h=1e-14), 4, use_graph=True)
        if method != "RK23":  # a last stage that is the next step's first is not captured
            assert bt.info()["job_table"] == (launch == "jobs"), bt.last_error()
        got.append([to_host(bt.get_m(i)) for i in range(6)])
        bt.close()
    for a, b in zip(*got):
        assert np.isfinite(a).all() and np.array_equal(a, b)
