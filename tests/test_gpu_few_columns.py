"""FP64 pass B with 11 to 17 modes at padded y = 1024: in split form on few columns (up to 64 over the batch
entries) and in two halves on more, whole and ragged, up to the line and beyond it, several columns per block of
the halves, the right-hand side (halves on any number) and several sources at once.  Against the oracle's FP64 FFT
apply; tolerance the FP64 apply's, 1e-12, and for solves to 1e-10 the oracle's residual."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, relerr, say
from oracle import operator2d as op2
from paper_1802_03061_amd import inputs
from test_gpu_diffusive import source
from test_gpu_modes_widths import channels
from test_gpu_update_a import residual

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rte():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1802_03061_amd import rte as r
    r.load()
    return r


# columns of a channel vector: 8, 16, 32, 64 (split form); 128 and more (halves); a mode vector has twice as many
CASES = [(2, 257, 5), (8, 512, 8), (7, 300, 7), (16, 511, 6), (17, 257, 8), (32, 512, 7), (33, 400, 5), (64, 300, 6),
         (64, 512, 8), (65, 512, 6), (100, 257, 8), (128, 300, 7), (66, 400, 5), (260, 259, 6)]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("nx,ny,L", CASES)
def test_apply(rte, nx, ny, L):
    say("few columns", nx, ny, L)
    mu_a, mu_s, h = 0.2, 3.0, 1.0 / max(nx, ny)
    sh = inputs.hg_sigma_hat(0.6, L)
    ctx = rte.Context((nx, ny), h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=rte.PREC_FP64)
    rng = np.random.default_rng(nx + 100 * ny + L)
    u = rng.standard_normal((2 * L + 1, ny, nx)) + 1j * rng.standard_normal((2 * L + 1, ny, nx))
    g = 0.5 * (u + np.conj(u[::-1]))
    spectra = op2.kernel_spectra(ny, nx, L, h, mu_a + mu_s, workers=16)
    for op, name in ((rte.OP_KT, "KT"), (rte.OP_A, "A")):
        ref, refg = (op2.apply_fft(x, L, h, mu_a + mu_s, mu_s, sh, name, spectra=spectra, workers=16) for x in (u, g))
        e = relerr(host(ctx.apply(dev(u), op=op)), ref)
        y = host(ctx.apply(dev(channels(g, L)), op=op, layout=rte.LAYOUT_CHANNELS))
        ec = relerr(y, channels(refg, L))
        say(f"  {name}: modes {e:.2e} channels {ec:.2e}")
        assert max(e, ec) <= 1e-12
    f = rng.standard_normal((ny, nx))
    e = relerr(host(ctx.rhs(dev(f))), op2.rhs(f, L, h, mu_a + mu_s, spectra=spectra, workers=16))
    say(f"  right-hand side {e:.2e}")
    assert e <= 1e-12
    ctx.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("nx,ny,L,count", [(17, 260, 5, 2), (17, 260, 5, 3), (40, 270, 8, 2)])
def test_several_sources(rte, nx, ny, L, count):
    say("few columns, several sources", nx, ny, L, count)
    mu_a, mu_s, h = 0.1, 4.0, 1.0 / max(nx, ny)
    sh = inputs.hg_sigma_hat(0.5, L)
    ctx = rte.Context((nx, ny), h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=rte.PREC_FP64)
    fs = [source((nx, ny), k) for k in range(count)]
    us = [(f, ctx.solve(dev(f), tol=1e-10)[0]) for f in fs]
    us += list(zip(fs, ctx.solve_multi([dev(f) for f in fs], tol=1e-10)[0]))
    for f, u in us:
        e = residual((ny, nx), L, h, mu_a, mu_s, sh, f, host(u))
        say(f"  oracle residual {e:.2e}")
        assert e <= 1.2e-10
    ctx.close()
