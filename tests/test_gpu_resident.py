"""The resident multi-shift kernel (one launch per multi-shift solve, r and t on the chip)
where its blocks and exchange can go wrong: one workgroup without faces, partial waves,
axes of one block and of two, two-site blocks, both time boundaries, several lattices in one
launch, two sites per thread (FP32), and a wait that runs out.  Signs against the oracle at
1e-11: both sides run the multi-shift at 1e-12, as in the parity tests."""
import numpy as np
import pytest

from paper_1005_3276_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_util import CFG2, bits, check, dev, host, lattice, require_gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu(torch)


def resident_launches(lat, call):
    lat.kernel_sampling(4)
    lat.kernel_times(2)
    out = call()
    n = lat.kernel_times(2)[1]
    lat.kernel_sampling(0)
    return out, n


@pytest.mark.parametrize("dims,bc", [((2, 2, 2, 2), -1), ((4, 4, 4, 4), 1), ((6, 4, 2, 10), -1),
                                     ((8, 8, 8, 8), 1), ((2, 26, 2, 38), -1),
                                     ((12, 6, 10, 14), -1), ((14, 14, 14, 14), -1)])
def test_resident_sign_vs_oracle(orc, dims, bc):
    print(f"[resident] {dims} bc={bc}", flush=True)
    x = inputs.gaussian_field(dims, nrhs=2, seed=61)
    lat = lattice(dims, bc_t=bc, inner_tol=1e-12, **CFG2)
    (out, st), n = resident_launches(lat, lambda: lat.sign(dev(x)))
    assert n > 0
    o = orc.Oracle(dims, bc_t=bc, inner_tol=1e-12, **CFG2)
    for r in range(2):
        check(host(out)[r], o.sign(x[r])[0], 1e-11, f"rhs {r}")


def test_resident_uneven_launch_and_fp32(orc):
    """Lattices of different block shapes in one launch, and an FP32 block of two sites per
    thread (16^3 x 32): every solution certified under its own oracle or its residual."""
    from paper_1005_3276_amd import solve_batch
    dims = [(4, 4, 4, 4), (2, 4, 6, 8), (8, 8, 8, 8)]
    lats, bs, ps = [], [], []
    for k, d in enumerate(dims):
        phi, src = inputs.draw(d, nrhs=1 + k % 2, sigma2=0.25, seed=70 + k)
        lats.append(lattice(d, precision="mixed", outer_tol=1e-10, **CFG2))
        bs.append(src)
        ps.append(phi)
    (xs, _), n = resident_launches(lats[0], lambda: solve_batch(lats, [dev(b) for b in bs],
                                                                [dev(p) for p in ps]))
    assert n > 0
    for d, b, p, x in zip(dims, bs, ps, xs):
        o = orc.Oracle(d, inner_tol=1e-13, **CFG2)
        for r in range(b.shape[0]):
            assert o.residual(b[r], host(x)[r], p) <= 1e-10, (d, r)
    d = (16, 16, 16, 32)
    phi, src = inputs.draw(d, nrhs=1, sigma2=0.25, seed=75)
    lat = lattice(d, precision="mixed", outer_tol=1e-10, **CFG2)
    print(f"[resident] {d} mixed", flush=True)
    (x, st), n = resident_launches(lat, lambda: lat.solve(dev(src), dev(phi)))
    assert n > 0 and st[0]["true_rel_res"] <= 1e-10


def test_wait_limit_falls_back(monkeypatch):
    """A wait limit of zero ticks: the resident launch gives up at its first unfinished wait
    and the call runs again with the per-pass kernels, bit for bit what they give."""
    dims = (8, 8, 8, 8)
    phi, src = inputs.draw(dims, nrhs=2, sigma2=0.25, seed=80)
    b, p = dev(src), dev(phi)
    kw = dict(inner_tol=1e-12, outer_tol=1e-10, **CFG2)
    monkeypatch.setenv("OV_PERSISTENT", "0")
    ref = lattice(dims, **kw)
    want = [host(ref.sign(b)[0]), host(ref.solve(b, p)[0])]
    monkeypatch.setenv("OV_PERSISTENT", "1")
    monkeypatch.setenv("OV_RES_WAIT_US", "0")
    lat = lattice(dims, **kw)
    got = [host(lat.sign(b)[0]), host(lat.solve(b, p)[0])]
    for g, w in zip(got, want):
        assert np.array_equal(bits(g), bits(w))
