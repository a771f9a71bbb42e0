"""Operators on the caller's own fields (no planar copy): the plain and the z-marching H_W,
their remainders, and a call in place.  Tolerance: nine FP64 terms of unit-size coefficients
per value, 1e-14 of the field's norm as in the parity tests."""
import ctypes as C

import numpy as np
import pytest

from paper_1005_3276_amd import _lib as L
from paper_1005_3276_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_util import CFG2, check, dev, host, lattice, require_gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu(torch)


# plain: partial blocks, extents of 2; marching (planes of 128..256 sites, at least 768
# workgroups of 4 or 2 z planes): a full plane, partial waves, two planes in z, T = 2
@pytest.mark.parametrize("dims,nrhs,bc", [((2, 2, 2, 2), 3, -1), ((2, 10, 2, 6), 2, 1),
                                          ((16, 18, 4, 2), 2, -1),
                                          ((16, 16, 4, 4), 192, -1), ((6, 22, 10, 4), 39, 1),
                                          ((12, 12, 2, 2), 384, -1), ((14, 10, 6, 16), 16, -1)])
def test_hw_on_caller_fields_vs_oracle(orc, dims, nrhs, bc):
    print(f"[hw io] {dims} nrhs={nrhs} bc={bc}", flush=True)
    x = inputs.gaussian_field(dims, nrhs=nrhs, seed=81)
    out, _ = lattice(dims, bc_t=bc, **CFG2).apply("hw", dev(x))
    o = orc.Oracle(dims, bc_t=bc, **CFG2)
    for r in {0, nrhs // 2, nrhs - 1}:
        check(host(out)[r], o.hw(x[r]), 1e-14, f"rhs {r}")


@pytest.mark.parametrize("shift", [0, 1])
def test_hw_in_place(orc, shift):
    """out on top of in, exactly or one field on: the call reads its input first."""
    dims, nrhs = (4, 6, 8, 2), 3
    x = inputs.gaussian_field(dims, nrhs=nrhs, seed=82)
    lat = lattice(dims, **CFG2)
    buf = torch.cat([dev(x), torch.zeros_like(dev(x)[:1])])
    out = buf[shift:shift + nrhs]
    torch.cuda.synchronize()
    st = (L.OvStats * nrhs)()
    assert L.lib().ov_apply(lat._h, L.OPS["hw"], C.c_void_p(out.data_ptr()),
                            C.c_void_p(buf.data_ptr()), None, nrhs, st) == 0
    ref = orc.Oracle(dims, **CFG2)
    for r in range(nrhs):
        check(host(out)[r], ref.hw(x[r]), 1e-14, f"rhs {r}")


@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 514), 1), ((22, 24, 22, 24), 1)])
def test_sign_with_per_pass_kernels_vs_oracle(orc, dims, nrhs):
    """Lattices without a resident decomposition: a small one (T = 2 x 257), and one of more
    than 1024 workgroups (several sites per thread, a last workgroup that is not full).
    Both sides run the multi-shift at 1e-12."""
    print(f"[per-pass sign] {dims}", flush=True)
    x = inputs.gaussian_field(dims, nrhs=nrhs, seed=83)
    kw = dict(CFG2, lambda_min=0.2, n_poles=12, inner_tol=1e-12)
    lat = lattice(dims, precondition=0, **kw)
    lat.kernel_sampling(4)
    lat.kernel_times(3)
    out, _ = lat.sign(dev(x))
    assert lat.kernel_times(3)[1] > 0
    check(host(out)[0], orc.Oracle(dims, **kw).sign(x[0])[0], 1e-11)


def test_uneven_batch_with_per_pass_kernels(orc):
    """Two lattices of different sizes that share a launch of the per-pass kernels."""
    from paper_1005_3276_amd import solve_batch
    dims = [(4, 4, 4, 4), (2, 2, 2, 514)]
    kw = dict(precision="mixed", outer_tol=1e-10, precondition=0, **CFG2)
    phi, src = zip(*(inputs.draw(d, nrhs=1 + k, sigma2=0.25, seed=84 + k)
                     for k, d in enumerate(dims)))
    print(f"[per-pass batch] {dims}", flush=True)
    xs, _ = solve_batch([lattice(d, **kw) for d in dims], [dev(b) for b in src],
                        [dev(p) for p in phi])
    for d, b, p, x in zip(dims, src, phi, xs):
        o = orc.Oracle(d, inner_tol=1e-13, **CFG2)
        for r in range(b.shape[0]):
            assert o.residual(b[r], host(x)[r], p) <= 1e-10, (d, r)


# momentum-space operators: the smallest, planes and slabs of 1024 sites, extents of 2 mod
# 4, and (z, t) lines beyond LDS (2 x 4 x 64 x 64: separate z and t passes)
MOMENTUM = [((2, 2, 2, 2), 1), ((64, 16, 2, 4), -1), ((16, 2, 64, 6), -1), ((22, 6, 10, 14), -1),
            ((4, 2, 26, 46), 1), ((2, 4, 64, 64), -1)]


@pytest.mark.parametrize("dims,bc", MOMENTUM)
def test_momentum_operators_closed_form(dims, bc):
    """D, D^dag, M, M^dag and MdagM of the exact overlap form on the caller's fields and in
    place, against the momentum-space 4 x 4 matrix.  Sums of at most 64 terms per axis
    and direction, eight of them: 1e-12 as for the full sizes in the parity tests."""
    import closed_form as cf
    print(f"[momentum] {dims} bc={bc}", flush=True)
    phi, x = inputs.draw(dims, nrhs=2, sigma2=0.25, seed=86)
    lat = lattice(dims, bc_t=bc, dirac="overlap_exact", m=0.05, g=0.3)
    sym = cf.dov_symbol(cf.exact_sign_symbol(dims, bc))
    dag = np.conj(np.swapaxes(sym, -1, -2))
    cp = (0.05 + 0.3 * phi)[..., None]
    c = np.concatenate([np.conj(cp), np.conj(cp), cp, cp], axis=-1)  # Y psi = c psi
    D = lambda v: cf.apply_symbol(sym, v, dims, bc)
    Dd = lambda v: cf.apply_symbol(dag, v, dims, bc)
    M = lambda v: D(v) + c * v
    Md = lambda v: Dd(v) + np.conj(c) * v
    want = dict(dov=D, dov_dag=Dd, m=M, m_dag=Md, mdagm=lambda v: Md(M(v)))
    for op, f in want.items():
        y = host(lat.apply(op, dev(x), dev(phi))[0])
        z = dev(x)
        p = dev(phi)
        torch.cuda.synchronize()
        st = (L.OvStats * 2)()
        assert L.lib().ov_apply(lat._h, L.OPS[op], C.c_void_p(z.data_ptr()), C.c_void_p(z.data_ptr()),
                                C.c_void_p(p.data_ptr()), 2, st) == 0
        for r in range(2):
            w = f(x[r])
            check(y[r], w, 1e-12, f"{op} rhs {r}")
            check(host(z)[r], w, 1e-12, f"{op} in place rhs {r}")


@pytest.mark.parametrize("dims", [(6, 4, 10, 2), (2, 2, 40, 44)])
def test_boson_ragged_vs_oracle(orc, dims):
    """The bosonic action's three planes, in one (z, t) pass and in separate passes; 1e-12
    as above."""
    print(f"[boson] {dims}", flush=True)
    kw = dict(m=0.05, g=0.3)
    phi, _ = inputs.draw(dims, nrhs=1, sigma2=0.25, seed=87)
    S, G, F = lattice(dims, **kw).boson(dev(phi))
    So, Go, Fo = orc.Oracle(dims, **kw).boson(phi)
    assert abs(S - So) <= 1e-12 * abs(So)
    check(host(G), Go, 1e-12)
    check(host(F), Fo, 1e-12)


@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 1), ((2, 4, 6, 10), 3), ((8, 8, 12, 14), 2)])
def test_overlap_operators_on_caller_fields_vs_oracle(orc, dims, nrhs):
    """sign, D, M and their adjoints with the multi-shift's source read from, and the
    combination written to, the caller's fields (workgroups of 64 threads in four groups per
    site and of 256 in two, a last workgroup that is not full), and in place, on the packed
    copies.  Both sides run the multi-shift at 1e-12, as in the parity tests."""
    print(f"[overlap io] {dims}", flush=True)
    phi, x = inputs.draw(dims, nrhs=nrhs, sigma2=0.25, seed=88)
    lat = lattice(dims, inner_tol=1e-12, **CFG2)
    o = orc.Oracle(dims, inner_tol=1e-12, **CFG2)
    r = nrhs - 1
    ops = dict(dov=orc.OP_DOV, dov_dag=orc.OP_DOV_DAG, m=orc.OP_M, m_dag=orc.OP_M_DAG,
               mdagm=orc.OP_MDAGM)
    check(host(lat.sign(dev(x))[0])[r], o.sign(x[r])[0], 1e-11, "sign")
    for op, code in ops.items():
        want = o.apply(code, x[r], phi)
        check(host(lat.apply(op, dev(x), dev(phi))[0])[r], want, 1e-11, op)
        z, p = dev(x), dev(phi)
        torch.cuda.synchronize()
        st = (L.OvStats * nrhs)()
        assert L.lib().ov_apply(lat._h, L.OPS[op], C.c_void_p(z.data_ptr()), C.c_void_p(z.data_ptr()),
                                C.c_void_p(p.data_ptr()), nrhs, st) == 0
        check(host(z)[r], want, 1e-11, f"{op} in place")
