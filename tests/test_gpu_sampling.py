"""Bytes that kernel sampling reports for the resident kernel: one field per site and iteration
of every entry of a launch (t_n to the basis), so the sum over a call is what its iteration
counts give."""
import pytest

from paper_1005_3276_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_util import CFG2, dev, lattice, require_gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu(torch)


def test_resident_bytes(orc):
    """FP64 throughout, 64 bytes per site and iteration: several sources of one lattice, one of
    them zero, and a batch of two lattices (two launches' worth of entries, some of which
    leave before the others, and solves that end at different times).  Sums of integers
    scaled by one quotient: 1e-12."""
    from paper_1005_3276_amd import solve_batch
    d4, d8 = (4, 4, 4, 4), (8, 8, 8, 8)
    kw = dict(inner_tol=1e-10, outer_tol=1e-10, precision="fp64", **CFG2)
    l4, l8 = lattice(d4, **kw), lattice(d8, **kw)
    (p4, b4), (p8, b8) = (inputs.draw(d, nrhs=2, sigma2=0.25, seed=98) for d in (d4, d8))

    def sampled(lat, call):
        lat.kernel_sampling(64)
        lat.kernel_times(2)
        st = call()
        _, n, by = lat.kernel_times(2)
        lat.kernel_sampling(0)
        assert n > 0
        return st, by

    x = dev(b8)
    x[1] = 0
    st, by = sampled(l8, lambda: l8.sign(x)[1])
    its = [s["inner_iters"] for s in st]
    print(f"[sampling] sign {its} {by}", flush=True)
    assert its[1] == 0 < its[0]
    assert by == pytest.approx(64 * l8.V * sum(its), rel=1e-12)
    st, by = sampled(l4, lambda: solve_batch([l4, l8], [dev(b4), dev(b8)], [dev(p4), dev(p8)])[1])
    its = [s["inner_iters"] for s in st]
    print(f"[sampling] batch {its} {by}", flush=True)
    assert by == pytest.approx(64 * (l4.V * sum(its[:2]) + l8.V * sum(its[2:])), rel=1e-12)
