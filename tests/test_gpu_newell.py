"""The GPU tensor's two kernels at every rule of the far-field quadrature
(R from the switch to past 300 longest sides), with waves that mix rules and
that mix near and far offsets, for cubes and for flat and elongated cells.

Oracle: the moment expansion (far) and the serial exact form (near).  Both
sides of the near field are float64 second differences, each within 2e-10 of
V/(4 pi R^3); just past the switch the oracle's truncation error is of the
same size: 5e-10 in all.  From R = 16 on the oracle's truncation error has
fallen by (16/6)^16 to below 1e-16 and only rounding is left: each side adds
fewer than 1000 terms of alternating sign no larger than 10, so 1000 * 10 *
2^-53 = 1.1e-12."""

import numpy as np
import pytest

from oracle import newell
from tests.gpu_util import film, log, scaled_tensor_error, sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cell", [((310, 3, 2), (4e-9, 4e-9, 4e-9)), ((3, 70, 9), (5e-9, 5e-9, 1.5e-9)),
                                    ((9, 2, 65), (3e-9, 2e-9, 1e-9)), ((1, 1, 1), (5e-9, 4e-9, 3e-9)),
                                    ((1, 40, 1), (2e-9, 2e-9, 6e-9))])
def test_newell_rules(n, cell):
    log(f"newell rules {n}")
    s = sim(film(n, cell), "f64")
    got, ref = s.get_demag_tensor(), newell.tensor_octant(n, cell)
    assert scaled_tensor_error(got, ref, cell) < 5e-10
    iz, iy, ix = np.meshgrid(*(np.arange(v) for v in n[::-1]), indexing="ij")
    R = np.sqrt((ix * cell[0]) ** 2 + (iy * cell[1]) ** 2 + (iz * cell[2]) ** 2) / max(cell)
    far = R >= 16.0
    assert scaled_tensor_error(np.where(far, got, 0.0), np.where(far, ref, 0.0), cell) < 1.1e-12
    # components odd along an axis vanish exactly at zero offset along it
    assert not got[[3, 4], :, :, 0].any() and not got[[3, 5], :, 0, :].any() and not got[[4, 5], 0].any()
