"""Multi-shift passes that store past the caches: launches whose fields exceed the last-level
cache, in the z-marching form and the plain one, against the same sources one at a time (below
the limit).  Both sides run the multi-shift at 1e-12: 1e-11 as in the parity tests."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_util import dev, check, host, lattice, require_gpu
from paper_1005_3276_amd import inputs

KW = dict(m=0.05, g=0.3, n_poles=12, lambda_min=0.2, lambda_max=8.0)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu(torch)


# 6 fields: 302 MB in a pass; the solve's two sources of 6 systems in FP32 as much
@pytest.mark.parametrize("dims", [(16, 16, 16, 64), (32, 32, 16, 16)])
def test_fields_beyond_the_cache(monkeypatch, dims):
    monkeypatch.setenv("OV_PERSISTENT", "0")
    print(f"[streaming] {dims}", flush=True)
    phi, src = inputs.draw(dims, nrhs=1, sigma2=0.25, seed=71)
    x = torch.stack([dev(src)[0] * (1 + r) for r in range(6)])
    x[3] = x[3].roll(1, 0)
    lat = lattice(dims, inner_tol=1e-12, **KW)
    out, _ = lat.sign(x)
    for r in (0, 3, 5):
        one, _ = lat.sign(x[r:r + 1].contiguous())
        check(host(out[r]), host(one[0]), 1e-11, f"rhs {r}")
    lat = lattice(dims, precision="mixed", outer_tol=1e-10, **KW)
    y, st = lat.solve(x, dev(phi))
    assert max(s["true_rel_res"] for s in st) <= 1e-10
    one, _ = lat.apply("mdagm", y[3:4].contiguous(), dev(phi))
    # the residual by the operator itself: 1e-10 and its multi-shift at mixed defaults
    r = (one[0] - x[3]).norm() / x[3].norm()
    print(f"[streaming] residual {float(r):.2e}", flush=True)
    assert float(r) <= 1e-7
