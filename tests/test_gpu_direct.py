"""Sub-steps that write the next stage input themselves, and form Eq. (6) inside
on small meshes, against the separate combination, Eq. (6) and stage launches:
job-table steps of a batch keep the separate ones, forked-stream steps take the
fused ones, and the two must agree bit for bit for every tableau, order and number
of terms, with empty cells, with rows that end inside a block and on both sides of
the mesh size up to which Eq. (6) is formed inside."""

import numpy as np
import pytest

import workloads
from tests.gpu_util import film, log, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 4e-9, 3e-9)


SMALL, LARGE = [(21, 13, 3), (70, 9, 1)], [(70, 64, 32), (21, 13, 3)]


@pytest.mark.parametrize("meshes,prec", [(SMALL, "f32"), (SMALL, "f64"), (LARGE, "f32")])
@pytest.mark.parametrize("method,p", [("RK23", 0), ("RK23", 3), ("RKF45", 1), ("RKCK45", 4), ("RKDP54", 5),
                                      ("RKF56", 2), ("HEUN", 2), ("RK4", 0), ("RK4", 4)])
def test_direct_equals_separate(method, p, meshes, prec):
    import torch

    import paper_2107_06729_amd as llgx
    log(f"direct {method} {p} {prec}")
    stream = torch.cuda.Stream()
    got = []
    for launch in ("jobs", "streams"):
        bt = llgx.Batch([film(n, CELL, K=2e4, Ha=(h, 1e3, 0.0)) for n in meshes for h in (1e4, -2e4)], prec, stream=stream)
        bt.set_launch(launch)
        bt.precompute_demag()
        with torch.cuda.stream(stream):
            for i in range(4):
                n = meshes[i // 2]
                M = workloads.random_m(n, 8e5, 90 + i)
                if i % 2:
                    M = workloads.masked(M, workloads.checkerboard_mask(n, 4))
                bt.set_m(i, to_dev(M, prec))
        bt.run_fixed(llgx.make_stepper(method, extrap=p, h=1e-14), p + 4, use_graph=True)
        assert bt.info()["job_table"] == (launch == "jobs"), bt.last_error()
        got.append([to_host(bt.get_m(i)) for i in range(4)])
        bt.close()
    for a, b in zip(*got):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("op", ["heff", "rhs"])
def test_field_call_finds_empty_cells_itself(op):
    """A field call tests every neighbour; the same M held as a handle's state
    does so because its flag is set, and a full mesh takes the same values as one
    whose only empty cell is elsewhere."""
    from tests.gpu_util import sim
    n = (20, 12, 2)
    M = workloads.random_m(n, 8e5, 95)
    s = sim(film(n, CELL), "f64")
    full = to_host(getattr(s, op)(to_dev(M, "f64")))
    s.set_m(to_dev(workloads.masked(M, workloads.checkerboard_mask(n, 4)), "f64"))
    # the state's flag does not reach a field call
    assert np.array_equal(to_host(getattr(s, op)(to_dev(M, "f64"))), full)


# blocks of the update: 2 | 512 (all write their maximum to the host) | 520 and 2080
# (reduced to 1 and 3 values first)
@pytest.mark.parametrize("extrap", [None, 0])
@pytest.mark.parametrize("n", [(33, 5, 1), (256, 256, 2), (256, 520, 1), (256, 520, 4)])
def test_error_norm_of_a_heun_step(n, extrap):
    """HEUN's estimate is (h/2)(F_1 - F_0) = M_new - M_0 - h F_0, so the reported
    norm follows from public results.  Each term is rounded at 2^-53 Ms or less:
    the difference of two M and the product leave below 2^-51 of Ms."""
    import torch

    import paper_2107_06729_amd as llgx
    from tests.gpu_util import sim
    s = sim(film(n, CELL), "f64", stream=torch.cuda.Stream())
    M0 = workloads.random_m(n, 8e5, 96)
    s.set_m(to_dev(M0, "f64"))
    F0 = to_host(s.rhs(to_dev(M0, "f64")))
    h = 1e-14
    st = llgx.make_stepper("HEUN", extrap=extrap, h=h, adaptive=True, h_max=h, e_max=10.0)
    info = s.step(st)
    e = to_host(s.get_m()) - M0 - h * F0
    want = float(np.sqrt((e * e).sum(axis=0)).max()) / 8e5
    log(f"heun {n} {extrap}: {info['err']:.6e} want {want:.6e}")
    assert want > 1e-6 and info["h_used"] == h
    assert abs(info["err"] - want) < 2.0 ** -51 * 4
