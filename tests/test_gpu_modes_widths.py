"""Pass B for 19 to 33 modes in FP32 at the widths and sizes that the other tests leave out: in one kernel
(padded y <= 512) every L = 9..16 at several sequences per wave and at one, and in split form (padded y =
1024) with both couplings, the mode-axis FFT of length 64 among them.  Apply of both operators in both layouts
against the oracle's FP64 FFT apply; tolerance the FP32 apply's, 1e-6."""
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


def channels(u, L):
    """Channels of conjugate-symmetric modes: u_0, then sqrt2 Re u_k, sqrt2 Im u_k."""
    out = [u[L].real]
    for k in range(1, L + 1):
        out += [np.sqrt(2) * u[L + k].real, np.sqrt(2) * u[L + k].imag]
    return np.stack(out)


ONE_KERNEL = [(7, 9, 10), (5, 200, 10), (6, 100, 14), (4, 130, 14), (3, 60, 15), (5, 256, 15), (3, 250, 9),
              (4, 129, 11), (3, 256, 13), (5, 33, 12)]
SPLIT = [(5, 300, 9), (4, 257, 15), (3, 400, 12), (2, 512, 16)]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("nx,ny,L", ONE_KERNEL + SPLIT)
def test_widths(rte, nx, ny, L):
    say("mode widths", nx, ny, L)
    mu_a, mu_s, h = 0.2, 3.0, 1.0 / max(nx, ny)
    sh = inputs.hg_sigma_hat(0.6, L)
    ctx = rte.Context((nx, ny), h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=rte.PREC_FP32)
    rng = np.random.default_rng(nx + 100 * ny + L)
    u = rng.standard_normal((2 * L + 1, ny, nx)) + 1j * rng.standard_normal((2 * L + 1, ny, nx))
    g = 0.5 * (u + np.conj(u[::-1]))
    spectra = op2.kernel_spectra(ny, nx, L, h, mu_a + mu_s, workers=16)
    for v in (range(2) if (nx, ny, L) in SPLIT else range(1)):
        ctx.set_variant(rte.PREC_FP32, 1, v)
        for op, name in ((rte.OP_KT, "KT"), (rte.OP_A, "A")):
            ref, refg = (op2.apply_fft(x, L, h, mu_a + mu_s, mu_s, sh, name, spectra=spectra, workers=16) for x in (u, g))
            e = relerr(host(ctx.apply(dev(u), op=op)), ref)
            y = host(ctx.apply(dev(channels(g, L)), op=op, layout=rte.LAYOUT_CHANNELS))
            ec = relerr(y, channels(refg, L))
            say(f"  variant {v} {name}: modes {e:.2e} channels {ec:.2e}")
            assert max(e, ec) <= 1e-6
    ctx.close()
