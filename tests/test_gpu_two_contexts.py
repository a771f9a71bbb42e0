"""Two contexts on two threads and streams of one process: their resident launches are
ordered, so none gives up waiting for workgroups that the other one's hold, and each result
has the bits of the same call on its own."""
import ctypes as C
import threading

import numpy as np
import pytest

from paper_1005_3276_amd import _lib as L
from paper_1005_3276_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_util import CFG2, bits, dev, host, lattice, require_gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu(torch)


def ptr(t):
    return C.c_void_p(t.data_ptr())


class Work:
    """A lattice on a stream of its own whose resident launches take most of the CUs, with
    its fields and the results of calls made alone."""

    def __init__(self, dims, seed):
        self.stream = torch.cuda.Stream()
        phi, src = inputs.draw(dims, nrhs=1, sigma2=0.25, seed=seed)
        self.b, self.phi = dev(src), dev(phi)
        self.out, self.x = torch.zeros_like(self.b), torch.zeros_like(self.b)
        with torch.cuda.stream(self.stream):
            self.lat = lattice(dims, precision="mixed", inner_tol=1e-10, outer_tol=1e-10, **CFG2)
        torch.cuda.synchronize()

    def sign(self):
        L.check(L.lib().ov_sign(self.lat._h, ptr(self.out), ptr(self.b), 1, None), self.lat._h)
        return bits(host(self.out))

    def solve(self):
        with torch.cuda.stream(self.stream):
            self.x.zero_()
        self.stream.synchronize()
        L.check(L.lib().ov_solve(self.lat._h, ptr(self.x), ptr(self.b), ptr(self.phi), 1, None),
                self.lat._h)
        return bits(host(self.x))


@pytest.mark.parametrize("graphs", ["0", "1"])
def test_two_threads(monkeypatch, graphs):
    monkeypatch.setenv("OV_GRAPHS", graphs)
    works = [Work((16, 16, 16, 16), 95), Work((12, 12, 12, 16), 96)]
    want = [(w.sign(), w.solve()) for w in works]
    if graphs == "0":
        for w in works:
            w.lat.kernel_sampling(8)
            for k in range(5):
                w.lat.kernel_times(k)
    print(f"[two contexts] graphs={graphs}", flush=True)
    start = threading.Barrier(2)
    wrong = []

    def go(w, ref):
        start.wait()
        try:
            for n in range(6):
                if not np.array_equal(w.sign(), ref[0]):
                    wrong.append(f"sign {n}")
                if not np.array_equal(w.solve(), ref[1]):
                    wrong.append(f"solve {n}")
        except Exception as e:  # an error of the library
            wrong.append(repr(e))

    threads = [threading.Thread(target=go, args=a) for a in zip(works, want)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    if graphs == "0":  # resident launches only: none was given up
        for w in works:
            n = [w.lat.kernel_times(k)[1] for k in range(5)]
            assert n[2] > 0 and n[0] + n[1] + n[3] + n[4] == 0, n
