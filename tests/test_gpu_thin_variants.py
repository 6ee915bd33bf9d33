"""Every variant of the fused y/z/y pass of thin meshes (thread counts: one or
several product units a thread, partial last rounds) gives the same bits, in the
precisions that take it only up to four layers, at one-, two- and three-stage y
lengths; and every variant of the separate y passes on an FP32 mesh of more layers
than the fused pass takes."""

import numpy as np
import pytest

import workloads
from tests.gpu_util import film, log, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 3e-9, 2e-9)
MESHES = [(9, 4, 1), (20, 3, 4), (33, 16, 2), (7, 20, 3), (18, 30, 4), (5, 65, 1), (12, 100, 3), (40, 129, 4)]


@pytest.mark.parametrize("prec,spectral", [("f64", "native"), ("f32", "bf16"), ("f32", "f16"), ("f32", "native")])
@pytest.mark.parametrize("n", MESHES, ids=lambda n: "x".join(map(str, n)))
def test_fused_variants_bitwise(n, prec, spectral):
    _all_variants(n, prec, spectral, (2,))


@pytest.mark.parametrize("n", [(40, 36, 12), (6, 130, 9), (5, 4, 10)], ids=lambda n: "x".join(map(str, n)))
def test_separate_y_variants_bitwise_f32(n):
    _all_variants(n, "f32", "native", (1, 2, 3))


def _all_variants(n, prec, spectral, kinds):
    import paper_2107_06729_amd as llgx
    log(f"variants {n} {prec} {spectral}")
    p = film(n, CELL)
    spec = {"native": llgx.SPEC_NATIVE, "bf16": llgx.SPEC_BF16, "f16": llgx.SPEC_F16}[spectral]
    s = llgx.Sim(p, prec, spectral=spec)
    s.precompute_demag()
    M = to_dev(workloads.random_m(n, p["Ms"], 55), prec)
    h, f = to_host(s.demag(M)), to_host(s.rhs(M))
    assert np.abs(h).max() > 0
    for k in kinds:
        for v in range(llgx.variant_counts()[k]):
            var = s.variants()
            var[k] = v
            s.set_variants(var)
            assert np.array_equal(to_host(s.demag(M)), h), (k, v)
            assert np.array_equal(to_host(s.rhs(M)), f), (k, v)
    s.close()
