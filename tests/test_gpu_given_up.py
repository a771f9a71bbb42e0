"""Calls whose resident launch gives up waiting (OV_RES_WAIT_US=0: at its first unfinished
wait) run again with the per-pass kernels.  The second run needs the inputs as they were, so
every result is compared bit for bit with a context that has only the per-pass kernels
(OV_PERSISTENT=0); kernel sampling shows that a resident launch was made (kernel 2) and that
the per-pass kernels followed (kernel 3, the FP64 t pass)."""
import ctypes as C

import numpy as np
import pytest

from paper_1005_3276_amd import _lib as L
from paper_1005_3276_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_util import CFG2, bits, dev, host, lattice, require_gpu

DIMS = (8, 8, 8, 8)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu(torch)


def per_pass(monkeypatch, dims=DIMS, **kw):
    """A context without the resident kernel."""
    monkeypatch.setenv("OV_PERSISTENT", "0")
    lat = lattice(dims, **kw)
    monkeypatch.delenv("OV_PERSISTENT")
    return lat


def giving_up(monkeypatch, dims=DIMS, **kw):
    """A context whose resident launches give up at once."""
    monkeypatch.setenv("OV_RES_WAIT_US", "0")
    lat = lattice(dims, **kw)
    monkeypatch.delenv("OV_RES_WAIT_US")
    return lat


def same_bits(a, b):
    return np.array_equal(bits(a), bits(b))


def ptr(t):
    return C.c_void_p(t.data_ptr())


def gave_up(lat, call):
    """Runs call; True if a resident launch was made and the per-pass kernels followed."""
    lat.kernel_sampling(4)
    for k in (2, 3):
        lat.kernel_times(k)
    call()
    n = [lat.kernel_times(k)[1] for k in (2, 3)]
    lat.kernel_sampling(0)
    return n[0] > 0 and n[1] > 0


def operate(lat, op, out, x, phi, nrhs, noalloc=False):
    st = (L.OvStats * nrhs)()
    if op == "sign":
        L.check(L.lib().ov_sign(lat._h, ptr(out), ptr(x), nrhs, st), lat._h)
    else:
        fn = L.lib().ov_apply_noalloc if noalloc else L.lib().ov_apply
        L.check(fn(lat._h, L.OPS[op], ptr(out), ptr(x), ptr(phi), nrhs, st), lat._h)


@pytest.mark.parametrize("op", ["sign", "dov", "dov_dag", "m", "m_dag", "mdagm"])
@pytest.mark.parametrize("shift", [0, 1])
def test_in_place(monkeypatch, op, shift):
    """out on top of in, exactly or one field on."""
    print(f"[given up] {op} shift={shift}", flush=True)
    nrhs = 2
    phi, src = inputs.draw(DIMS, nrhs=nrhs, sigma2=0.25, seed=90)
    p = dev(phi)
    kw = dict(inner_tol=1e-10, **CFG2)

    def run(lat, noalloc=False):
        buf = torch.cat([dev(src), torch.zeros_like(dev(src)[:1])])
        out = buf[shift:shift + nrhs]
        torch.cuda.synchronize()
        operate(lat, op, out, buf, p, nrhs, noalloc)
        return host(out)

    want = run(per_pass(monkeypatch, **kw))
    lat = giving_up(monkeypatch, **kw)
    got = []
    assert gave_up(lat, lambda: got.append(run(lat)))
    if op != "sign":
        got.append(run(lat, noalloc=True))
    for g in got:
        assert same_bits(g, want), op


def test_fallback_engine_of_a_batch(orc, monkeypatch):
    """A batch whose first system converges at once (b = 0) and whose second is handed to the
    FP64 solver, which the second context leads and whose launches give up: the batch runs
    again and is certified under the oracle."""
    from paper_1005_3276_amd import solve_batch
    monkeypatch.setenv("OV_FORCE_FALLBACK", "1")
    kw = dict(precision="mixed", outer_tol=1e-10, **CFG2)
    phi, src = inputs.draw(DIMS, nrhs=1, sigma2=0.25, seed=91)
    lats = [lattice(DIMS, **kw), giving_up(monkeypatch, **kw)]
    xs = []

    def call():
        xs[:], st = solve_batch(lats, [torch.zeros_like(dev(src)), dev(src)], [dev(phi)] * 2)
        assert st[1]["fp64_fallback"]

    print("[given up] batch, FP64 fallback", flush=True)
    assert gave_up(lats[1], call)
    assert not host(xs[0]).any()
    o = orc.Oracle(DIMS, inner_tol=1e-13, **CFG2)
    assert o.residual(src[0], host(xs[1])[0], phi) <= 1e-10
    x, _ = lats[1].solve(dev(src), dev(phi))  # and the context goes on
    assert o.residual(src[0], host(x)[0], phi) <= 1e-10


@pytest.mark.parametrize("onto", ["phi", "xi"])
@pytest.mark.parametrize("rational", [False, True])
def test_gradient_over_inputs(monkeypatch, onto, rational):
    """Eight sources, whose two-source multi-shifts (the solve's) run per pass and whose
    one-source ones (Y = M X, just before the gradient is written) as resident launches: the
    wait runs out there, with the gradient on top of phi or inside xi."""
    dims, nrhs = (8, 8, 8, 16), 8
    print(f"[given up] gradient on {onto}, rational={rational}", flush=True)
    phi, src = inputs.draw(dims, nrhs=nrhs, sigma2=0.25, seed=92)
    kw = dict(m=0.05, g=0.3, n_poles=12, lambda_min=0.2, lambda_max=8.0, outer_tol=1e-10)
    al, be = np.array([0.4, 0.6]), np.array([0.1, 1.0])
    vp = lambda a: a.ctypes.data_as(C.c_void_p)

    def run(lat):
        x, p = dev(src), dev(phi)
        grad = p.view(-1) if onto == "phi" else x.view(-1)[lat.V:2 * lat.V]
        torch.cuda.synchronize()
        S, st = (C.c_double * nrhs)(), (L.OvStats * nrhs)()
        if rational:
            rc = L.lib().ov_rational_force(lat._h, 0.2, 2, vp(al), vp(be), ptr(grad), S, ptr(x),
                                           ptr(p), nrhs, st)
        else:
            rc = L.lib().ov_force(lat._h, ptr(grad), S, ptr(x), ptr(p), nrhs, st)
        L.check(rc, lat._h)
        return list(S), host(grad)

    want = run(per_pass(monkeypatch, dims, **kw))
    lat = giving_up(monkeypatch, dims, **kw)
    got = []
    assert gave_up(lat, lambda: got.append(run(lat)))
    assert got[0][0] == want[0]
    assert same_bits(got[0][1], want[1])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves(monkeypatch, precision):
    """Calls of many launches: a solve and a rational function with their own outputs."""
    print(f"[given up] solves {precision}", flush=True)
    phi, src = inputs.draw(DIMS, nrhs=2, sigma2=0.25, seed=99)
    b, p = dev(src), dev(phi)
    kw = dict(precision=precision, inner_tol=1e-10, outer_tol=1e-10, **CFG2)
    al, be = np.array([0.4, 0.6]), np.array([0.1, 1.0])
    calls = [lambda lat: host(lat.solve(b, p)[0]), lambda lat: host(lat.rational(b, p, 0.2, al, be)[0])]
    ref = per_pass(monkeypatch, **kw)
    want = [f(ref) for f in calls]
    lat = giving_up(monkeypatch, **kw)
    for f, w in zip(calls, want):
        got = []
        assert gave_up(lat, lambda: got.append(f(lat)))
        assert same_bits(got[0], w)
