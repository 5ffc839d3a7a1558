"""The isotropic 3D z-pass (one wave or part of one per column) at every padded z-length 16..512, whole
and ragged, with fewer and with more columns than a launch holds at once, every waves-per-block
variant, against the oracle's FP64 FFT apply (bars as the 3D apply's: 1e-6 in FP32, 1e-12 in FP64)."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, relerr, say
from oracle import operator3d as op3

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("nx,ny,nz", [(2, 3, 2), (5, 4, 8), (3, 7, 9), (6, 5, 16), (4, 9, 17), (7, 3, 33), (5, 6, 64),
                                      (3, 5, 65), (4, 3, 128), (3, 4, 129), (2, 3, 256), (100, 90, 12)])
@pytest.mark.parametrize("prec", [0, 1])
def test_iso_z_pass_matches_oracle(nx, ny, nz, prec):
    from paper_1802_03061_amd import rte
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    mu_a, mu_s, h = 0.1, 2.0, 1.0 / max(nx, ny, nz)
    ctx = rte.Context((nx, ny, nz), h=h, mu_a=mu_a, mu_s=mu_s, L=0, prec=prec)
    u = np.random.default_rng(nx + 10 * ny + 100 * nz).standard_normal((nz, ny, nx))
    ref = op3.apply_fft(u, h, mu_a + mu_s, mu_s, "A", workers=16)
    for v in range(ctx.get_variant(prec, 2)[1]):
        ctx.set_variant(prec, 2, v)
        e = relerr(host(ctx.apply(dev(u[None]), op=rte.OP_A, layout=rte.LAYOUT_CHANNELS))[0], ref)
        say("z-pass", nx, ny, nz, "prec", prec, "variant", v, f"relerr vs oracle {e:.2e}")
        assert e <= (1e-6 if prec == rte.PREC_FP32 else 1e-12)
    ctx.close()
