"""What a batch reports of its launches: the form of the latest steps taken from
graphs, unchanged by calls that replay nothing, and the reason for a step without
job tables once, when it is found."""

import numpy as np
import pytest

import workloads
from tests.gpu_util import film, log, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 4e-9, 3e-9)


def _batch(meshes, spectral=0):
    import torch

    import paper_2107_06729_amd as llgx
    bt = llgx.Batch([film(n, CELL) for n in meshes], "f32", stream=torch.cuda.Stream(), spectral=spectral)
    bt.precompute_demag()
    return bt


def _load(bt, meshes, seed):
    for i, n in enumerate(meshes):
        bt.set_m(i, to_dev(workloads.random_m(n, 8e5, seed + i), "f32"))


def test_launch_info_follows_replays():
    import paper_2107_06729_amd as llgx
    meshes = [(20, 12, 2), (9, 6, 10)]
    log("batch launch info")
    st = llgx.make_stepper("RK4", extrap=2, h=1e-14)
    bt = _batch(meshes)
    _load(bt, meshes, 20)
    bt.run_fixed(st, 2)  # priming: nothing replayed
    assert (bt.info()["job_table"], bt.info()["kernels_per_step"]) == (False, 0)
    bt.run_fixed(st, 3)
    assert (bt.info()["job_table"], bt.info()["kernels_per_step"]) == (False, -1)
    bt.set_launch("jobs")
    bt.run_fixed(st, 3)
    nk = bt.info()["kernels_per_step"]
    assert bt.info()["job_table"] and nk > 0
    bt.set_launch("streams")
    _load(bt, meshes, 30)
    bt.run_fixed(st, 2)  # priming again, with the groups' graphs of the first call at hand
    assert (bt.info()["job_table"], bt.info()["kernels_per_step"]) == (True, nk)
    bt.run_fixed(st, 1)
    assert (bt.info()["job_table"], bt.info()["kernels_per_step"]) == (False, -1)
    bt.close()


# no job-table form: 16-bit spectra, and a mesh whose z length is above 64
@pytest.mark.parametrize("spectral,meshes", [("bf16", [(20, 12, 2), (9, 6, 10)]), ("native", [(5, 4, 40), (9, 6, 10)])])
def test_no_job_table_is_found_once(spectral, meshes):
    import paper_2107_06729_amd as llgx
    log(f"no job table {spectral} {meshes}")
    spec = {"bf16": llgx.SPEC_BF16, "native": llgx.SPEC_NATIVE}[spectral]
    st = llgx.make_stepper("RK4", extrap=1, h=1e-14)
    bt, ref = _batch(meshes, spec), _batch(meshes, spec)
    bt.set_launch("jobs")
    for b in (bt, ref):
        _load(b, meshes, 40)
        b.run_fixed(st, 4)
    assert "job-table launch not used" in bt.last_error()
    with pytest.raises(llgx.LlgxError):
        bt.autotune(0)  # an error of its own, refused before anything changes
    note = bt.last_error()
    assert "job-table" not in note
    for _ in range(3):  # every history phase
        for b in (bt, ref):
            b.run_fixed(st, 1)
    assert bt.last_error() == note
    assert (bt.info()["job_table"], bt.info()["kernels_per_step"]) == (False, -1)
    for i in range(2):
        assert np.array_equal(to_host(bt.get_m(i)), to_host(ref.get_m(i))), i
    # another order is looked at for itself
    bt.run_fixed(llgx.make_stepper("RK4", extrap=0, h=1e-14), 2)
    assert "job-table launch not used" in bt.last_error()
    bt.close()
    ref.close()
