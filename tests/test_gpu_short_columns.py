"""Isotropic pass B at padded y = 16 (one lane per column): rows 2..8, the packed column alone and with many
others, more columns than a wave holds, one and two batch entries, and in a batched solve, against the oracle.
Tolerances: the apply's 1e-6 (FP32) and 1e-12 (FP64); the solve's oracle residual."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, relerr, say
from oracle import operator2d as op2
from test_gpu_diffusive import source
from test_gpu_update_a import residual

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rte():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1802_03061_amd import rte as r
    r.load()
    return r


@pytest.mark.parametrize("nx,ny", [(2, 2), (8, 8), (9, 3), (33, 7), (70, 8), (300, 5), (512, 8)])
@pytest.mark.parametrize("prec", [0, 1])
def test_apply(rte, nx, ny, prec):
    say("short columns", nx, ny, prec)
    mu_a, mu_s, h = 0.2, 3.0, 1.0 / max(nx, ny)
    ctx = rte.Context((nx, ny), h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=[1.0], L=0, prec=prec)
    rng = np.random.default_rng(nx + 100 * ny)
    u = rng.standard_normal((1, ny, nx)) + 1j * rng.standard_normal((1, ny, nx))
    bar = 1e-6 if prec == rte.PREC_FP32 else 1e-12
    for op, name in ((rte.OP_KT, "KT"), (rte.OP_A, "A")):
        ref = op2.apply_fft(u, 0, h, mu_a + mu_s, mu_s, np.ones(1), name)
        e = [relerr(host(ctx.apply(dev(u), op=op)), ref)]
        e.append(relerr(host(ctx.apply(dev(u.real), op=op, layout=rte.LAYOUT_CHANNELS)), ref.real))
        say(f"  {name}: modes {e[0]:.2e} channels {e[1]:.2e}")
        assert max(e) <= bar
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_batched(rte, prec):
    ns = [(8, 8), (5, 5), (2, 2), (8, 8), (7, 7)]
    ctxs = [rte.Context(n, h=1.0 / n[0], mu_a=0.1, mu_s=2.0 + k, sigma_hat=[1.0], L=0, prec=prec)
            for k, n in enumerate(ns)]
    fs = [source(n, k) for k, n in enumerate(ns)]
    us, _, rc = rte.solve_batched(ctxs, [dev(f) for f in fs], [1e-10] * len(ns))
    assert rc == rte.RTE_OK
    for k, (n, c, f, u) in enumerate(zip(ns, ctxs, fs, us)):
        e = residual(n, 0, 1.0 / n[0], 0.1, 2.0 + k, np.ones(1), f, host(u))
        say(f"  batched {n} prec {prec}: oracle residual {e:.2e}")
        assert e <= 1.2e-10
        c.close()
