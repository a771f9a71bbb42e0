"""Operators on the caller's own fields (no planar copy): the plain and the z-marching H_W,
their remainders, and a call in place.  Tolerance: nine FP64 terms of unit-size coefficients
per value, 1e-14 of the field's norm as in the parity tests."""
import ctypes as C

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
