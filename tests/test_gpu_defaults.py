"""The variants that a handle starts with are not slower than the widest tiles
(variant 0) where tiles are many and short, or few and long.  Fastest of six rounds
in turn; the wrong variant of some pass takes 1.23 to 2.1 times as long on each of
these."""

import pytest

import workloads
from tests.gpu_util import film, log, sim, to_dev

pytestmark = pytest.mark.gpu

PASSES = ("xfwd", "yfwd", "zmul", "yinv", "xinv")


@pytest.mark.parametrize("n,prec", [((8, 488, 113), "f32"), ((150, 400, 20), "f32"), ((600, 100, 2), "f64"),
                                    ((400, 190, 45), "f64"), ((90, 15, 11), "f64")])
def test_default_variants_are_not_slower_than_the_widest_tiles(n, prec):
    log(f"defaults {n} {prec}")
    s = sim(film(n, (4e-9, 4e-9, 4e-9)), prec)
    s.set_m(to_dev(workloads.random_m(n, 8e5, 1), prec))
    own = s.variants()
    t = {}
    for _ in range(6):
        for name, v in (("own", own), ("wide", [0] * 5)):
            s.set_variants(v)
            for k, us in s.time_passes(40).items():
                t[name, k] = min(t.get((name, k), 1e9), us)
    s.close()
    log({k: (round(t["own", k], 2), round(t["wide", k], 2)) for k in PASSES})
    for k in PASSES:
        assert t["own", k] <= 1.2 * t["wide", k], (k, own)
