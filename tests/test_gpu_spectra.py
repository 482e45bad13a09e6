"""The Fourier-sum kernels at the edges of their shapes: one sample, fewer
lines than a wave's lanes, batch and quarter remainders, the longest length
with a table of roots and one past it, both signs, and the allocation-free
call, against numpy's FFT.

Tolerance: a sum of n products carries at most n eps (1.1e-16) of its terms'
size and sqrt(n) eps on average, so 1e-13 relative L2 holds up to 10^4
samples with a factor of ten to spare.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import torch
    import paper_2509_25840_amd as pk
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    torch.zeros(1, device="cuda")
    return pk


def close(got, ref, scale):
    err = np.linalg.norm(got - ref)
    print(f"    {err / max(np.linalg.norm(ref), scale):.2e}", flush=True)
    assert err <= 1e-13 * max(np.linalg.norm(ref), scale)


@pytest.mark.parametrize("n", [1, 2, 7, 16, 17, 127, 257, 1000, 4000, 8192, 8193])
def test_spectrum_1d(pk, n):
    print(f"[1d] {n}", flush=True)
    R = np.random.default_rng(n).normal(size=n)
    tau = 0.01
    om, I = pk.spectrum_1d(R, tau)
    ref_om = 2 * np.pi * np.arange(n) / (n * tau)
    assert np.allclose(om, ref_om, rtol=1e-15)
    close(I, ref_om * (tau * n * np.fft.ifft(R)).imag, tau * np.linalg.norm(ref_om))


@pytest.mark.parametrize("n1,n2", [(1, 1), (1, 9), (9, 1), (3, 5), (8, 512), (512, 8), (63, 65), (65, 33), (64, 256),
                                   (40, 8193), (8193, 3)])
def test_spectrum_2d(pk, n1, n2):
    print(f"[2d] {n1} x {n2}", flush=True)
    R = np.random.default_rng(n1 * 1000 + n2).normal(size=(n2, n1))
    t1, t2 = 0.01, 0.02
    z = np.fft.fft(R, axis=1)
    scale = t1 * t2 * np.sqrt(n1 * n2)
    for sign, f in ((-1, pk.spectrum_2d), (1, pk.spectrum_2dir)):
        ref = t1 * t2 * (np.fft.fft(z, axis=0) if sign < 0 else np.fft.ifft(z, axis=0) * n2).imag
        close(f(R, t1, t2), ref, scale)
    if n1 * n2 <= 131072:
        import torch
        I = np.empty_like(R)
        dp = ctypes.POINTER(ctypes.c_double)
        f = pk.lib().chfpe_spectrum_2d_noalloc
        f.argtypes = pk.lib().chfpe_spectrum_2d.argtypes
        assert f(R.ctypes.data_as(dp), n1, n2, t1, t2, I.ctypes.data_as(dp),
                 ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        close(I, t1 * t2 * np.fft.fft(z, axis=0).imag, scale)
