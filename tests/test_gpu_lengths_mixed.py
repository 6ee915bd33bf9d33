"""Oracle parity of Eq. (2) at every padded length 3 2^m and 5 2^m the passes
are built for, along each axis in turn: the smallest and the largest cell
count of each length, with short other axes (nz > 4 where the separate y and z
passes are meant), and meshes that pad all three axes that way.  Tolerances as
for the powers of two: FP64 1e-12 relative, FP32 1e-5 Ms, 16-bit spectra 8 u
Ms, the GPU's own tensor 1e-9 relative."""

import numpy as np
import pytest

import workloads
from oracle import demag, newell
from tests.gpu_util import f32_round, film, log, sim, to_dev, to_host

pytestmark = pytest.mark.gpu

U16 = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}
CELL = (2e-9, 3e-9, 2.5e-9)
LENGTHS = [2, 4, 8, 16, 24, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320, 384, 512, 640, 768, 1024, 1280, 1536, 2048]


def _meshes():
    out = []
    for axis in range(3):
        for low, L in zip(LENGTHS, LENGTHS[1:]):
            if L & (L - 1) == 0 or (axis == 2 and L > 1024) or (axis == 0 and L // 2 not in LENGTHS):
                continue
            # lengths take turns: the largest mesh of one, the smallest of the next, and
            # two z counts (the fused thin pass and the separate ones)
            k = len(out)
            n = [3, 3, 2 if k % 4 < 2 else 5]
            n[axis] = L // 2 if k % 2 else low // 2 + 1
            out.append(tuple(n))
    return out + [(20, 23, 12), (33, 40, 19), (75, 12, 33)]


MESHES = _meshes()


@pytest.mark.parametrize("n", MESHES, ids=lambda n: "x".join(map(str, n)))
def test_demag_mixed_length(n):
    import paper_2107_06729_amd as llgx
    log(f"mixed lengths {n}")
    Nf = newell.tensor_full(n, CELL)
    M = workloads.random_m(n, 8e5, 62)
    ref64, ref32 = demag.demag_fft(M, Nf), demag.demag_fft(f32_round(M), Nf)
    p = film(n, CELL)
    got = to_host(sim(p, "f64", tensor=Nf).demag(to_dev(M, "f64")))
    assert np.max(np.abs(got - ref64)) <= 1e-12 * np.max(np.abs(ref64))
    s = sim(p, "f32", tensor=Nf)
    Md = to_dev(f32_round(M), "f32")
    got = to_host(s.demag(Md))
    assert np.max(np.abs(got - ref32)) <= 1e-5 * p["Ms"]
    for v in (1, 2):  # every tile of the passes: the same bits
        s.set_variants([v] * 5)
        assert np.array_equal(to_host(s.demag(Md)), got), v
    for mode, spec in (("bf16", llgx.SPEC_BF16), ("f16", llgx.SPEC_F16)):
        s = llgx.Sim(p, "f32", spectral=spec)
        s.set_demag_tensor(Nf)
        err = np.max(np.abs(to_host(s.demag(Md)) - ref32)) / p["Ms"]
        assert err <= 8 * U16[mode], (mode, err)
    got = to_host(sim(p, "f64").demag(to_dev(M, "f64")))
    assert np.max(np.abs(got - ref64)) <= 1e-9 * np.max(np.abs(ref64))


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_batch_modes_mixed_lengths(prec):
    """Job-table launches (one per length) and forked streams: the same bits."""
    import torch

    import paper_2107_06729_amd as llgx
    meshes = [(20, 12, 9), (33, 40, 2), (40, 20, 17), (24, 36, 6)]
    stream = torch.cuda.Stream()
    got = []
    for launch in ("jobs", "streams"):
        bt = llgx.Batch([film(n, CELL) for n in meshes], prec, stream=stream)
        bt.set_launch(launch)
        bt.precompute_demag()
        with torch.cuda.stream(stream):
            for i, n in enumerate(meshes):
                bt.set_m(i, to_dev(workloads.random_m(n, 8e5, 80 + i), prec))
        bt.run_fixed(llgx.make_stepper("RK4", extrap=2, h=1e-14), 6, use_graph=True)
        assert bt.info()["job_table"] == (launch == "jobs"), bt.last_error()
        got.append([to_host(bt.get_m(i)) for i in range(len(meshes))])
    for i in range(len(meshes)):
        assert np.array_equal(got[0][i], got[1][i]), i
