"""Diffusive media, where K v is nearly v: the single-pass Gram-Schmidt step of the plain solver must keep
the basis orthogonal there.  Grids from 16 cells a side, up to 25 mean free paths per cell, 2D and 3D,
isotropic and not, both precisions and the FP32 basis: as many iterations as with a second
Gram-Schmidt pass on every step (one or two more allowed, where the estimate meets the target late),
and the oracle's FP64 residual.  The solver stops at an FP64 residual of 1e-9 and its apply agrees with
the oracle's to 1e-12 of the largest term, which in these media is about 1e2 of the right-hand side at most."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, say
from paper_1802_03061_amd import inputs
from test_gpu_update_a import residual

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rte():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1802_03061_amd import rte as r
    r.load()
    return r


def source(n, seed):
    rng = np.random.default_rng(seed)
    x = np.meshgrid(*[(np.arange(v) + 0.5) / max(n) for v in reversed(n)], indexing="ij")
    f = np.zeros(tuple(reversed(n)))
    for _ in range(3):
        c, w = rng.uniform(0.2, 0.8, len(n)), rng.uniform(0.05, 0.15)
        f += np.exp(-sum((a - b) ** 2 for a, b in zip(x, c)) / (2 * w * w))
    return f


CASES = [((64, 64), 0, 100.0, 0.01), ((64, 64), 0, 400.0, 0.01), ((64, 64), 0, 400.0, 1.0), ((40, 33), 0, 100.0, 0.01),
         ((128, 100), 0, 200.0, 0.05), ((48, 48), 3, 100.0, 0.01), ((16, 16, 16), 0, 400.0, 0.01),
         ((16, 14, 12), 2, 200.0, 0.01)]


@pytest.mark.parametrize("n,L,mu_s,mu_a", CASES)
@pytest.mark.parametrize("prec,basis32", [(0, 0), (1, 0), (0, 1)])
def test_iterations(rte, n, L, mu_s, mu_a, prec, basis32):
    say("diffusive", n, L, mu_s, mu_a, prec, basis32)
    h = 1.0 / max(n)
    sh = inputs.hg_sigma_hat(0.4, L)
    f = source(n, L + sum(n))
    its = []
    for reorth in (2, 0):
        ctx = rte.Context(n, h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=prec)
        ctx.set_opts(reorth=reorth, basis_fp32=basis32)
        u, info = ctx.solve(dev(f), tol=1e-9)
        its.append(info["iterations"])
        ctx.close()
    e = residual(tuple(reversed(n)), L, h, mu_a, mu_s, sh, f, host(u))
    say(f"  iterations {its[1]} (two passes {its[0]}) oracle residual {e:.2e}")
    assert its[1] <= its[0] + 2
    assert e <= 1.2e-9
