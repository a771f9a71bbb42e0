"""NaNs of the caller against the resident kernel's mark of a face value that has not arrived:
whatever their bits, they travel as values."""
import numpy as np
import pytest

from paper_1005_3276_amd import _lib as L
from paper_1005_3276_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_util import CFG2, dev, lattice, require_gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu(torch)


# doubles that the solver rounds to the floats 0x7ff45a5a (0xfff45a5a) and 0x7fe45a5a, the
# quieted marks of either word, and doubles with the mark in their own high word
@pytest.mark.parametrize("bits", [0x7FFE8B4B40000000, 0x7FFC8B4B40000000, 0x7FF45A5A7FA45A5A])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_nan_in_phi_is_a_breakdown(bits, precision):
    """A NaN in phi ends a solve at the first multi-shift that it reaches, in resident launches:
    none gives up waiting for it (kernels 0, 1, 3 and 4 are the per-pass ones)."""
    dims = (8, 8, 8, 8)
    print(f"[nan] {bits:#x} {precision}", flush=True)
    phi, src = inputs.draw(dims, nrhs=1, sigma2=0.25, seed=97)
    v = phi.view(np.uint64).reshape(-1, 2)
    v[::3] = bits, bits
    v[1::3] = bits | 1 << 63, bits | 1 << 63
    lat = lattice(dims, precision=precision, outer_tol=1e-10, **CFG2)
    lat.kernel_sampling(4)
    for k in range(5):
        lat.kernel_times(k)
    with pytest.raises(L.OvError) as e:
        lat.solve(dev(src), dev(phi))
    n = [lat.kernel_times(k)[1] for k in range(5)]
    assert e.value.status == 3
    assert n[2] > 0 and n[0] + n[1] + n[3] + n[4] == 0, n
