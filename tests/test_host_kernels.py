"""The library's own kernels, launchers and host code on the CPU (host_build.py):
every global and LDS access of every kernel lies inside its allocation, no value is
read that nothing wrote (fresh memory is NaN and would reach a result), and no
result depends on the order of a block's threads between two barriers.  Results are
compared with the oracle, and between the launch variants bit for bit.

This runs the code itself, so it follows every change of an index.  (The address
model in test_address_model.py restates the passes' indices as they were with
power-of-two lengths, plain spectra and the z product in LDS.)  Each case runs
twice, each time in a process of its own: allocations that end at an inaccessible
page and threads in ascending order, and allocations that start at one and threads
in descending order.  Both must give the same bits.
"""

import ctypes
import hashlib
import multiprocessing

import numpy as np
import pytest

import workloads
from oracle import fields, integrate, newell
from tests import host_build
from tests.gpu_util import f32_round, scaled_tensor_error

CELL = (4e-9, 3e-9, 2e-9)
MS = 8e5
STREAM = ctypes.c_void_p(16)  # a stream that is not the default one; never dereferenced


@pytest.fixture(scope="module")
def lib_path():
    import paper_2107_06729_amd  # noqa: F401  (the signatures; once, the children inherit it)
    return host_build.build()


# ---- the C interface on host memory ------------------------------------------
class Lib:
    def __init__(self, path):
        import paper_2107_06729_amd as llgx
        self.llgx = llgx
        self.c = ctypes.CDLL(path)
        for name, (res, args) in llgx._sig.items():
            f = getattr(self.c, name)
            f.restype, f.argtypes = res, args
        self.c.host_malloc.restype = ctypes.c_void_p
        self.c.host_malloc.argtypes = [ctypes.c_size_t]
        self.c.host_free.argtypes = [ctypes.c_void_p]
        self.c.host_begin()

    def problem(self, p):
        return self.llgx.make_problem(p)

    def put(self, a):
        """A guarded copy of an array: (pointer, view)."""
        ptr = self.c.host_malloc(a.nbytes)
        v = np.frombuffer((ctypes.c_char * a.nbytes).from_address(ptr), dtype=a.dtype).reshape(a.shape)
        v[...] = a
        return ptr, v

    def ok(self, st, err):
        assert st == 0, err().decode()

    def sim(self, p, prec, spectral=0, tensor=None):
        return Sim(self, p, prec, spectral, tensor)


class Sim:
    def __init__(self, lib, p, prec, spectral, tensor):
        self.lib, self.p = lib, p
        self.dtype = np.float32 if prec == "f32" else np.float64
        self.h = ctypes.c_void_p()
        q = lib.problem(p)
        st = lib.c.llgx_create(ctypes.byref(q), 1 if prec == "f32" else 0, spectral, STREAM, ctypes.byref(self.h))
        lib.ok(st, lambda: lib.c.llgx_last_error(None))
        if tensor is None:
            self.ok(lib.c.llgx_precompute_demag(self.h))
        else:
            t = np.ascontiguousarray(tensor)
            self.ok(lib.c.llgx_set_demag_tensor(self.h, t.ctypes.data))

    def ok(self, st):
        self.lib.ok(st, lambda: self.lib.c.llgx_last_error(self.h))

    def tensor(self):
        t = np.empty((6,) + self.p["n"][::-1])
        self.ok(self.lib.c.llgx_get_demag_tensor(self.h, t.ctypes.data))
        return t

    def field(self, name, M):
        i, _ = self.lib.put(M.astype(self.dtype))
        o, out = self.lib.put(np.full(M.shape, np.nan, self.dtype))
        self.ok(getattr(self.lib.c, name)(self.h, i, o))
        out = out.copy()
        self.lib.c.host_free(i)
        self.lib.c.host_free(o)
        return out

    def variants(self, v=None):
        a = (ctypes.c_int32 * 5)(*(v or [0] * 5))
        self.ok((self.lib.c.llgx_set_variants if v else self.lib.c.llgx_get_variants)(self.h, a))
        return list(a)

    def set_m(self, M):
        i, _ = self.lib.put(M.astype(self.dtype))
        self.ok(self.lib.c.llgx_set_m(self.h, i))
        self.lib.c.host_free(i)

    def get_m(self):
        o, out = self.lib.put(np.full((3,) + self.p["n"][::-1], np.nan, self.dtype))
        self.ok(self.lib.c.llgx_get_m(self.h, o))
        out = out.copy()
        self.lib.c.host_free(o)
        return out

    def close(self):
        self.lib.c.host_check()
        self.lib.c.llgx_destroy(self.h)


# ---- one case, twice, each time in a process of its own ------------------------
def _child(path, work, args, side, order, out):
    lib = Lib(path)
    lib.c.host_side(side)
    lib.c.host_order(order)
    out.send([hashlib.sha256(np.ascontiguousarray(a).tobytes()).hexdigest() for a in work(lib, *args)])


def twice(path, work, *args):
    fork = multiprocessing.get_context("fork")
    runs = []
    for side, order in ((1, 0), (0, 1)):
        got, out = fork.Pipe(duplex=False)
        p = fork.Process(target=_child, args=(path, work, args, side, order, out))
        p.start()
        out.close()
        runs.append((p, got))
    results = []
    for p, got in runs:
        try:
            results.append(got.recv())
        except EOFError:
            results.append(None)
        p.join()
    assert [p.exitcode for p, _ in runs] == [0, 0], f"exit code {max(p.exitcode for p, _ in runs)} (message above)"
    differ = [k for k, (a, b) in enumerate(zip(*results)) if a != b]
    assert not differ, f"results {differ} depend on the threads' order or on what memory held"


def problem(n, Ha=(-2e4, 1e3, 0.0), **kw):
    return workloads.problem(n, CELL, MS, 1.3e-11, 0.02, K=2e4, easy=(0.0, 0.6, 0.8), Ha=Ha, **kw)


def holes(n, seed):
    return workloads.masked(workloads.random_m(n, MS, seed), workloads.checkerboard_mask(n, 3))


# ---- fields -------------------------------------------------------------------
# thin (one to four layers; FP32 to eight), thick, missing axes, odd rows, rows that
# fill the padded length and that leave most of it empty; every first radix along
# every axis, one to three stages
MESHES = [(1, 1, 1), (7, 1, 1), (1, 6, 1), (1, 1, 9), (2, 2, 2), (1, 5, 4), (6, 1, 5), (13, 2, 1), (33, 9, 2),
          (10, 17, 3), (25, 20, 4), (3, 41, 1), (40, 65, 2), (4, 33, 5), (21, 12, 6), (9, 24, 7), (5, 48, 8),
          (70, 2, 9), (5, 13, 12), (20, 4, 13), (66, 3, 17), (3, 2, 24), (3, 4, 33), (2, 3, 49), (4, 30, 10),
          (129, 2, 2), (5, 80, 3), (160, 3, 11), (3, 5, 65)]


FORMATS = [("f32", 0), ("f64", 0), ("f32", 1), ("f32", 2)]


def _fields(lib, p, Nf, M, ref):
    n, out = p["n"], []
    counts = (ctypes.c_int32 * 5)()
    lib.c.llgx_variant_counts(counts)
    for prec, spectral in FORMATS:
        if spectral and (n[0] > 128 or max(n[1:]) > 64):
            continue  # 16-bit spectra keep powers of two; these are not built here
        s = lib.sim(p, prec, spectral, Nf)
        # rounding of the stored spectra in 16 bits (8 units in the last place), of the
        # arithmetic in FP32, and the FP64 bound of the GPU's field tests
        tol = {0: 1e-5 if prec == "f32" else 1e-12, 1: 8 * 2.0 ** -9, 2: 8 * 2.0 ** -12}[spectral]
        got = [s.field(f, M) for f in ("llgx_demag", "llgx_heff", "llgx_rhs", "llgx_demag_noalloc")]
        for g, r in zip(got, ref):
            assert np.isfinite(g).all()
            scale = np.max(np.abs(r)) if r is ref[2] else max(np.max(np.abs(r)), MS)
            assert np.max(np.abs(g - r)) <= tol * scale * (10 if r is ref[2] else 1), (prec, spectral)
        assert np.array_equal(got[0], got[3])
        for v in range(max(counts)):
            s.variants([min(v, k - 1) for k in counts])
            assert np.array_equal(s.field("llgx_rhs", M), got[2]), (prec, spectral, v)
        s.close()
        out += got
    return out


@pytest.mark.parametrize("n", MESHES, ids=lambda n: "x".join(map(str, n)))
def test_fields(lib_path, n):
    p = problem(n)
    M = f32_round(holes(n, 5))
    Nf = newell.tensor_full(n, CELL)
    it = integrate.Integrator(p, M, method="RK4", Nfull=Nf)
    Hd = it.demag(M)
    twice(lib_path, _fields, p, Nf, M, [Hd, fields.effective_field(M, Hd, it.pa), it.rhs(M, Hd)])


# ---- steps --------------------------------------------------------------------
METHODS = ["RK4", "RKF45", "RKCK45", "RKDP54", "HEUN", "RK23", "RKF56", "ABM2"]


def _steps(lib, p, Nf, M0, cases, precs=(("f64", 1e-12), ("f32", 1e-5))):
    """Cases (method, extrap, adaptive, renormalize, steps); the oracle takes the
    accepted step lengths, since the controller passes rounding of the estimate on
    to them."""
    out = []
    for method, extrap, adaptive, renormalize, count in cases:
        st = lib.llgx.make_stepper(method, extrap=extrap, h=5e-14, adaptive=adaptive, renormalize=renormalize,
                                   h_max=1e-12)
        for prec, tol in precs:  # with the bounds of the GPU's step tests
            ora = integrate.Integrator(p, M0, method=method, h=5e-14, adaptive=False, extrap=extrap, Nfull=Nf,
                                       renormalize=renormalize)
            s = lib.sim(p, prec, 0, Nf)
            s.set_m(M0)
            for k in range(count):
                info = lib.llgx.StepInfo()
                s.ok(lib.c.llgx_step(s.h, ctypes.byref(st), ctypes.byref(info)))
                ora.step(info.h_used)
                got = s.get_m()
                assert np.max(np.abs(got - ora.M)) <= tol * MS, (method, extrap, adaptive, prec, k)
            out.append(got)
            s.close()
            if not adaptive:
                s = lib.sim(p, prec, 0, Nf)
                s.set_m(M0)
                s.ok(lib.c.llgx_run_fixed(s.h, ctypes.byref(st), count, 1, None))
                # replayed steps take the Eq. (6) weights of the captured one, whose node
                # times differ by the rounding of t
                got = s.get_m()
                assert np.max(np.abs(got - ora.M)) <= tol * MS, (method, extrap, prec, "graphs")
                out.append(got)
                s.close()
    return out


@pytest.mark.parametrize("n,orders,method", [((13, 5, 2), (None, 0, 1, 2, 3, 4, 5), m) for m in METHODS]
                         + [((5, 6, 9), (None, 1, 4), m) for m in ("RK4", "RKDP54")],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) and None not in v else
                         v if isinstance(v, str) else "")
def test_steps(lib_path, n, orders, method):
    """Orders of Eq. (6) and full evaluations, fixed (stepped and replayed) and
    adaptive, past the priming steps."""
    p, M0, Nf = problem(n), f32_round(holes(n, 6)), newell.tensor_full(n, CELL)
    cases = [(method, extrap, adaptive, extrap in (None, 2), (extrap or 0) + 3) for extrap in orders
             for adaptive in [False] + [True] * (method != "RK4")]
    twice(lib_path, _steps, p, Nf, M0, cases)


def test_steps_with_fields_of_eq6(lib_path):
    """Above 512 KiB a component, Eq. (6) in fields of its own: formed with the first
    sub-step (RK4, at most two distinct times) or by a launch of their own."""
    n = (130, 64, 8)
    p, M0, Nf = problem(n), f32_round(holes(n, 7)), newell.tensor_full(n, CELL)
    twice(lib_path, _steps, p, Nf, M0, [("RK4", 1, False, False, 2), ("RKCK45", 1, True, False, 2)],
          (("f64", 1e-12),))


# ---- batches ------------------------------------------------------------------
def _batch(lib, meshes, states, method, extrap, prec, spectral):
    """Steps of samples of several meshes: job tables and streams, replayed and not."""
    out = []
    dtype = np.float32 if prec == "f32" else np.float64
    fields_of = [(1e4, 1e3, 0.0), (-2e4, 0.0, 3e3)]
    probs = [problem(n, Ha=h) for n in meshes for h in fields_of]
    arr = (lib.llgx.Problem * len(probs))(*[lib.problem(q) for q in probs])
    st = lib.llgx.make_stepper(method, extrap=extrap, h=5e-14)
    for mode, graph in ((0, 1), (1, 1), (1, 0)):
        b = ctypes.c_void_p()
        lib.ok(lib.c.llgx_batch_create(len(probs), arr, 1 if prec == "f32" else 0, spectral, STREAM, ctypes.byref(b)),
               lambda: lib.c.llgx_last_error(None))
        err = lambda: lib.c.llgx_batch_last_error(b)
        lib.ok(lib.c.llgx_batch_set_launch(b, mode), err)
        lib.ok(lib.c.llgx_batch_precompute_demag(b), err)
        for i, q in enumerate(probs):
            ptr, _ = lib.put(states[i].astype(dtype))
            lib.ok(lib.c.llgx_batch_set_m(b, i, ptr), err)
            lib.c.host_free(ptr)
        lib.ok(lib.c.llgx_batch_run_fixed(b, ctypes.byref(st), 9, graph), err)
        jobs, kernels = ctypes.c_int32(), ctypes.c_int32()
        lib.ok(lib.c.llgx_batch_launch_info(b, ctypes.byref(jobs), ctypes.byref(kernels)), err)
        assert jobs.value == (mode == 0 and not spectral), err()
        got = []
        for i, q in enumerate(probs):
            ptr, v = lib.put(np.full((3,) + q["n"][::-1], np.nan, dtype))
            lib.ok(lib.c.llgx_batch_get_m(b, i, ptr), err)
            got.append(v.copy())
            lib.c.host_free(ptr)
            assert np.isfinite(got[i]).all()
        lib.c.host_check()
        lib.c.llgx_batch_destroy(b)
        for a, g in zip(out, got):
            if graph:
                assert np.array_equal(a, g), mode
            else:  # (the weights of Eq. (6) again)
                assert np.max(np.abs(a - g)) <= (1e-12 if prec == "f64" else 1e-5) * MS
        out = out or got
    return out


@pytest.mark.parametrize("method,extrap,prec,spectral", [("RK4", 4, "f32", 0), ("RK4", 4, "f64", 0),
                                                         ("RK4", 2, "f32", 1), ("RKCK45", 1, "f32", 0),
                                                         ("HEUN", None, "f32", 0)])
def test_batches(lib_path, method, extrap, prec, spectral):
    # five groups: one more than a job-table launch takes
    meshes = [(13, 5, 2), (6, 7, 9), (21, 1, 3), (40, 12, 1), (9, 20, 6)]
    states = [holes(n, 60 + k) if k else workloads.random_m(n, MS, 60) for n in meshes for k in range(2)]
    twice(lib_path, _batch, meshes, states, method, extrap, prec, spectral)


# ---- tensor -------------------------------------------------------------------
def _tensor(lib, n, cell, ref):
    p = workloads.problem(n, cell, MS, 1.3e-11, 0.02)
    s = lib.sim(p, "f64")
    got = s.tensor()
    assert scaled_tensor_error(got, ref, cell) < 1e-9
    s.close()
    return [got]


@pytest.mark.parametrize("n,cell", [((30, 3, 2), (4e-9, 4e-9, 4e-9)), ((3, 40, 9), (5e-9, 5e-9, 1.5e-9)),
                                    ((9, 2, 40), (3e-9, 2e-9, 1e-9)), ((1, 1, 1), (5e-9, 4e-9, 3e-9))],
                         ids=lambda v: None)
def test_tensor(lib_path, n, cell):
    twice(lib_path, _tensor, n, cell, newell.tensor_octant(n, cell))


# ---- the model itself -----------------------------------------------------------
def _read(lib, offset):
    ptr, _ = lib.put(np.zeros(16))
    ctypes.string_at(ptr + offset, 8)
    return []


def _store(lib, offset):
    ptr, _ = lib.put(np.zeros(17, np.float32))
    ctypes.memset(ptr + offset, 0, 1)
    lib.c.host_check()
    return []


@pytest.mark.parametrize("work,offset", [(_read, 128), (_read, 121), (_read, -8), (_store, 68), (_store, -1)])
def test_accesses_out_of_range_are_found(lib_path, work, offset):
    twice(lib_path, _read, 120)
    with pytest.raises(AssertionError, match="exit code 3"):
        twice(lib_path, work, offset)
