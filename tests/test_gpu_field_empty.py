"""Field calls on an M with empty cells while the handle's own state is full (and
the other way round): the call's own M decides which neighbours are missing."""

import numpy as np
import pytest

import workloads
from oracle import fields, integrate, newell
from tests.gpu_util import film, log, sim, to_dev, to_host

pytestmark = pytest.mark.gpu

CELL = (4e-9, 4e-9, 3e-9)


@pytest.mark.parametrize("n", [(20, 12, 2), (9, 6, 10), (12, 1, 1)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("state", ["full", "empty cells"])
def test_field_call_on_another_state(n, state):
    log(f"field call {n}, state {state}")
    p = film(n, CELL)
    full = workloads.random_m(n, p["Ms"], 97)
    holes = workloads.masked(full, workloads.checkerboard_mask(n, 3))
    Nf = newell.tensor_full(n, CELL)
    s = sim(p, "f64", tensor=Nf)
    s.set_m(to_dev(full if state == "full" else holes, "f64"))
    for M in (full, holes):
        it = integrate.Integrator(p, M, method="RK4", Nfull=Nf)
        Hd = it.demag(M)
        H, F = fields.effective_field(M, Hd, it.pa), it.rhs(M, Hd)
        gh, gf = to_host(s.heff(to_dev(M, "f64"))), to_host(s.rhs(to_dev(M, "f64")))
        # bounds of the other FP64 field tests: 1e-12 of the largest value, ten times
        # that with the two cross products of Eq. (1)
        assert np.max(np.abs(gh - H)) <= 1e-12 * np.max(np.abs(H))
        assert np.max(np.abs(gf - F)) <= 1e-11 * np.max(np.abs(F))
    s.close()
