"""Pass B with wave-private transforms and the real coupling: every padded y-length 16..1024 (whole and
ragged), L = 0..17 (FP32 up to 16 here, the others in split form), column groups with a dead column, columns in two halves (FP64, padded y = 1024,
L >= 5), more columns than blocks on the chip, and the single-channel right-hand side, against the
oracle's FP64 FFT apply.  Tolerances are the apply's: 1e-6 (FP32, a factor of about 5 over the
rounding of the transforms' stages) and 1e-12 (FP64)."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, relerr, say
from oracle import operator2d as op2
from paper_1802_03061_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rte():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1802_03061_amd import rte as r
    r.load()
    return r


CASES = [(5, 2, 0), (9, 8, 3), (3, 9, 1), (13, 16, 8), (7, 17, 2), (17, 32, 5), (6, 33, 7), (11, 64, 1), (5, 65, 8),
         (9, 128, 4), (6, 129, 6), (7, 256, 8), (4, 257, 5), (9, 300, 8), (6, 511, 6), (5, 512, 7), (3, 512, 8),
         (5, 400, 4), (3, 512, 0), (70, 64, 0), (7, 8, 0), (40, 33, 0), (300, 129, 0), (9, 300, 0), (512, 20, 8), (300, 257, 5),
         (6, 256, 16), (5, 130, 16), (9, 40, 9), (4, 200, 12), (300, 10, 13), (7, 8, 11), (3, 257, 16), (5, 64, 17)]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("nx,ny,L", CASES)
@pytest.mark.parametrize("prec", [0, 1])
def test_pass_b_matches_oracle(rte, nx, ny, L, prec):
    say("pass B", nx, ny, L, prec)
    mu_a, mu_s, h = 0.2, 3.0, 1.0 / max(nx, ny)
    sh = inputs.hg_sigma_hat(0.6, L)
    ctx = rte.Context((nx, ny), h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=prec)
    rng = np.random.default_rng(nx + 100 * ny + L)
    M = 2 * L + 1
    u = rng.standard_normal((M, ny, nx)) + 1j * rng.standard_normal((M, ny, nx))   # two channel vectors
    spectra = op2.kernel_spectra(ny, nx, L, h, mu_a + mu_s, workers=16)
    bar = 1e-6 if prec == rte.PREC_FP32 else 1e-12
    for op, name in ((rte.OP_KT, "KT"), (rte.OP_A, "A")):
        ref = op2.apply_fft(u, L, h, mu_a + mu_s, mu_s, sh, name, spectra=spectra, workers=16)
        e = relerr(host(ctx.apply(dev(u), op=op)), ref)
        say(f"  {name}: relerr vs oracle {e:.2e}")
        assert e <= bar
    f = rng.standard_normal((ny, nx))
    e = relerr(host(ctx.rhs(dev(f))), op2.rhs(f, L, h, mu_a + mu_s, spectra=spectra, workers=16))
    say(f"  right-hand side: relerr vs oracle {e:.2e}")
    assert e <= 1e-12
    ctx.close()
