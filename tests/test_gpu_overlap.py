"""Results written over a field that the call reads besides its input: the call reads it
first.  The fields are large enough in all that late workgroups start long after early ones
have written."""
import ctypes as C

import numpy as np
import pytest

from paper_1005_3276_amd import _lib as L
from paper_1005_3276_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_util import bits, check, dev, host, lattice, require_gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu(torch)


def ptr(t):
    return C.c_void_p(t.data_ptr())


@pytest.mark.parametrize("dirac,dims,nrhs", [("overlap", (16, 16, 16, 16), 8),
                                             ("overlap_exact", (8, 8, 8, 16), 64)])
@pytest.mark.parametrize("op", ["m", "m_dag", "mdagm"])
def test_result_over_phi(dirac, dims, nrhs, op):
    """phi inside out, against the call with buffers apart.  The two may take different
    routes: FP64 sums of at most 64 terms eight times over (1e-12), for the overlap form with
    multi-shifts at 1e-12 on both sides (1e-11), as in the parity tests."""
    print(f"[overlap] {dirac} {op}", flush=True)
    phi, src = inputs.draw(dims, nrhs=1, sigma2=0.25, seed=92)
    x = dev(src).expand(nrhs, *src.shape[1:]).contiguous()
    kw = dict(m=0.05, g=0.3, n_poles=12, lambda_min=0.2, lambda_max=8.0)
    lat = lattice(dims, dirac=dirac, inner_tol=1e-12, **kw)
    want, _ = lat.apply(op, x, dev(phi))
    out = torch.zeros_like(x)
    p = out.view(-1)[lat.V // 2:lat.V // 2 + lat.V]  # in the first field's part
    p.copy_(dev(phi).view(-1))
    torch.cuda.synchronize()
    st = (L.OvStats * nrhs)()
    L.check(L.lib().ov_apply(lat._h, L.OPS[op], ptr(out), ptr(x), ptr(p), nrhs, st), lat._h)
    for r in (0, nrhs // 2, nrhs - 1):
        check(host(out[r]), host(want[r]), 1e-12 if dirac == "overlap_exact" else 1e-11, f"rhs {r}")


@pytest.mark.parametrize("which", ["G", "F"])
def test_boson_over_phi(which):
    """G or F half a field above phi: the same kernels as with buffers apart, bit for bit."""
    dims = (32, 32, 32, 32)
    print(f"[overlap] boson {which}", flush=True)
    phi, _ = inputs.draw((2, 2, 2, 2), nrhs=1, sigma2=0.25, seed=93)
    phi = np.resize(phi, dims[::-1]) * np.linspace(0.5, 1.5, dims[3])[:, None, None, None]
    lat = lattice(dims, m=0.05, g=0.3)
    S, G, F = lat.boson(dev(phi))
    buf = torch.zeros(3 * lat.V // 2, dtype=torch.complex128, device="cuda")
    p, out, other = buf[:lat.V], buf[lat.V // 2:], torch.zeros_like(buf[:lat.V])
    p.copy_(dev(phi).view(-1))
    torch.cuda.synchronize()
    s = C.c_double()
    g, f = (out, other) if which == "G" else (other, out)
    L.check(L.lib().ov_boson(lat._h, ptr(p), C.byref(s), ptr(g), ptr(f)), lat._h)
    assert s.value == S
    same = [np.array_equal(bits(host(a)), bits(host(b).ravel())) for a, b in ((g, G), (f, F))]
    assert all(same)


@pytest.mark.parametrize("onto", ["phi", "xi"])
def test_gradient_over_its_inputs(onto):
    """grad_phi on top of phi, or inside xi: the same kernels as with buffers apart, bit for
    bit, in ov_force and ov_rational_force."""
    dims = (8, 8, 4, 4)
    print(f"[overlap] gradient on {onto}", flush=True)
    phi, src = inputs.draw(dims, nrhs=2, sigma2=0.25, seed=94)
    kw = dict(m=0.05, g=0.3, n_poles=12, lambda_min=0.2, lambda_max=8.0)
    al, be = np.array([0.4, 0.6]), np.array([0.1, 1.0])
    vp = lambda a: a.ctypes.data_as(C.c_void_p)
    for rational in (False, True):
        lat = lattice(dims, outer_tol=1e-10, **kw)
        want = (lat.rational_force(dev(src), dev(phi), 0.2, al, be) if rational
                else lat.force(dev(src), dev(phi)))
        x, p = dev(src), dev(phi)
        grad = p.view(-1) if onto == "phi" else x.view(-1)[lat.V:2 * lat.V]
        torch.cuda.synchronize()
        S, st = (C.c_double * 2)(), (L.OvStats * 2)()
        if rational:
            rc = L.lib().ov_rational_force(lat._h, 0.2, 2, vp(al), vp(be), ptr(grad), S, ptr(x),
                                           ptr(p), 2, st)
        else:
            rc = L.lib().ov_force(lat._h, ptr(grad), S, ptr(x), ptr(p), 2, st)
        L.check(rc, lat._h)
        assert list(S) == want[0]
        same = np.array_equal(bits(host(grad)), bits(host(want[1]).ravel()))
        assert same, f"rational={rational}"
