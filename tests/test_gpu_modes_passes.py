"""The 2D (and 3D) apply on general complex modes, whose conversions run inside passes A and C: every padded
x-length 16..1024 (whole rows, odd rows, rows one past a power of two), row tiles with remainders down to
one row, both row counts per block, one mode, packed and unpacked (L = 17) spectra, operators A and K~,
against the oracle's FP64 FFT apply.  Tolerances are the apply's: 1e-6 (FP32) and 1e-12 (FP64)."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, relerr, say
from oracle import operator2d as op2
from oracle import operator3d_sh as o3s
from paper_1802_03061_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rte():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1802_03061_amd import rte as r
    r.load()
    return r


CASES = [(2, 2, 0), (3, 9, 1), (8, 3, 2), (9, 2, 1), (16, 17, 3), (17, 8, 0), (31, 31, 2), (32, 5, 17), (33, 12, 4),
         (64, 40, 8), (65, 7, 1), (127, 66, 3), (128, 129, 2), (129, 4, 17), (256, 300, 7), (257, 9, 1), (511, 70, 8),
         (512, 3, 2), (300, 512, 4), (512, 512, 0)]


@pytest.mark.parametrize("nx,ny,L", CASES)
@pytest.mark.parametrize("prec", [0, 1])
def test_modes_match_oracle(rte, nx, ny, L, prec):
    say("modes apply", nx, ny, L, prec)
    mu_a, mu_s, h = 0.2, 3.0, 1.0 / max(nx, ny)
    sh = inputs.hg_sigma_hat(0.6, L)
    ctx = rte.Context((nx, ny), h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=prec)
    rng = np.random.default_rng(nx + 100 * ny + L)
    M = 2 * L + 1
    u = rng.standard_normal((M, ny, nx)) + 1j * rng.standard_normal((M, ny, nx))
    spectra = op2.kernel_spectra(ny, nx, L, h, mu_a + mu_s, workers=16)
    bar = 1e-6 if prec == rte.PREC_FP32 else 1e-12
    for op, name in ((rte.OP_KT, "KT"), (rte.OP_A, "A")):
        ref = op2.apply_fft(u, L, h, mu_a + mu_s, mu_s, sh, name, spectra=spectra, workers=16)
        e = relerr(host(ctx.apply(dev(u), op=op)), ref)
        say(f"  {name}: relerr vs oracle {e:.2e}")
        assert e <= bar
    ctx.close()


CASES3 = [((2, 2, 2), 1), ((9, 3, 5), 0), ((17, 10, 4), 2), ((33, 7, 3), 3), ((70, 5, 6), 0), ((129, 4, 3), 0), ((30, 40, 33), 0)]


@pytest.mark.parametrize("n,L", CASES3)
@pytest.mark.parametrize("prec", [0, 1])
def test_modes_match_oracle_3d(rte, n, L, prec):
    say("3D modes apply", n, L, prec)
    mu_a, mu_s, h = 0.2, 3.0, 1.0 / max(n)
    sh = inputs.hg_sigma_hat(0.6, L)
    ctx = rte.Context(n, h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=prec)
    rng = np.random.default_rng(sum(n) + L)
    shape = ((L + 1) ** 2,) + tuple(reversed(n))
    u = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    bar = 1e-6 if prec == rte.PREC_FP32 else 1e-12
    for op, name in ((rte.OP_KT, "KT"), (rte.OP_A, "A")):
        ref = sum(f * o3s.apply_fft(v, L, h, mu_a + mu_s, mu_s, sh, name) for f, v in ((1.0, u.real), (1j, u.imag)))
        e = relerr(host(ctx.apply(dev(u), op=op)).reshape(shape), ref)
        say(f"  {name}: relerr vs oracle {e:.2e}")
        assert e <= bar
    ctx.close()
