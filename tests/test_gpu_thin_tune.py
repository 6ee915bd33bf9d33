"""The autotuner on a thin mesh: its separate y passes are launched by job-table
steps alone, with tiles of their own, so there is nothing to choose for them; they
are still timed."""

import numpy as np
import pytest

import workloads
from tests.gpu_util import film, log, sim, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (5e-9, 5e-9, 3e-9)


@pytest.mark.parametrize("n,prec", [((40, 36, 3), "f64"), ((40, 36, 6), "f32")])
def test_y_variants_of_a_thin_mesh_are_left(n, prec):
    log(f"tune thin {n} {prec}")
    s = sim(film(n, CELL), prec)
    M = to_dev(workloads.random_m(n, 8e5, 54), prec)
    s.set_m(M)
    ref = to_host(s.demag(M))
    for v in (0, 1, 2):
        s.set_variants([0, v, 0, v, 0])
        us = s.autotune(3)
        assert [s.variants()[k] for k in (1, 3)] == [v, v]
        assert us["yfwd"] > 0 and us["yinv"] > 0
        t = s.time_passes(3)
        assert all(t[k] > 0 for k in t)
        assert np.array_equal(to_host(s.demag(M)), ref)
    s.close()
