"""The fused y/z/y pass of FP32 meshes of 5 to 8 layers (16-long z transforms in two
halves) against the separate passes, bit for bit as those of thinner meshes, and
against the oracle: every nz it takes, one-, two- and three-stage y lengths, mixed
ones, row counts that fill the padded length and that leave most of it empty.  FP32
tolerance as in the other length tests: 1e-5 Ms."""

import numpy as np
import pytest

import workloads
from oracle import demag, newell
from tests.gpu_util import f32_round, film, log, sim, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 3e-9, 2e-9)
MESHES = [(2, 2, 5), (9, 4, 8), (5, 7, 6), (33, 16, 7), (6, 33, 8), (7, 65, 5), (40, 12, 6), (31, 60, 8), (12, 129, 5),
          (5, 150, 8)]


@pytest.mark.parametrize("n", MESHES, ids=lambda n: "x".join(map(str, n)))
def test_equals_separate_passes(n):
    import torch

    import paper_2107_06729_amd as llgx
    log(f"thin8 {n}")
    stream = torch.cuda.Stream()
    got = []
    for launch in ("jobs", "streams"):
        bt = llgx.Batch([film(n, CELL, Ha=(h, 0.0, 0.0)) for h in (1e4, -2e4)], "f32", stream=stream)
        bt.set_launch(launch)
        bt.precompute_demag()
        with torch.cuda.stream(stream):
            for i in range(2):
                bt.set_m(i, to_dev(workloads.random_m(n, 8e5, 50 + i), "f32"))
        bt.run_fixed(llgx.make_stepper("RK4", h=1e-14), 4, use_graph=True)
        assert bt.info()["job_table"] == (launch == "jobs"), bt.last_error()
        got.append([to_host(bt.get_m(i)) for i in range(2)])
        bt.close()
    for i in range(2):
        assert np.array_equal(got[0][i], got[1][i]), i


@pytest.mark.parametrize("n", MESHES, ids=lambda n: "x".join(map(str, n)))
def test_against_oracle(n):
    import paper_2107_06729_amd as llgx
    log(f"thin8 oracle {n}")
    Nf = newell.tensor_full(n, CELL)
    M = f32_round(workloads.random_m(n, 8e5, 51))
    ref = demag.demag_fft(M, Nf)
    got = to_host(sim(film(n, CELL), "f32", tensor=Nf).demag(to_dev(M, "f32")))
    assert np.max(np.abs(got - ref)) <= 1e-5 * 8e5
