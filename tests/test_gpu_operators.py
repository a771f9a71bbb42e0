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
