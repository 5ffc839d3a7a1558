"""A mode vector is two real fields p + i q (p, q conjugate-symmetric modes; in 3D the real and imaginary
part), which the apply keeps apart: a real flux (q = 0) comes back exactly real, and a q of 1e-8 of p's
size keeps the accuracy it has alone.  Every padded x-length, odd rows, both row counts per block, one
mode, split pass B (L = 17) and 3D slabs.  Tolerance of the small part: the FP32 apply's 1e-6; reading it out
of a sum with p in double costs 1e-8 (1e-16 of p)."""
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


def symmetric(rng, shape):
    """Modes of a real field: u_-k = conj u_k, u_0 real."""
    u = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    return 0.5 * (u + np.conj(u[::-1]))


def parts(u, dim):
    """p and q of u = p + i q."""
    if dim == 3:
        return u.real, u.imag
    v = np.conj(u[::-1])
    return 0.5 * (u + v), -0.5j * (u - v)


CASES = [((7, 5), 2), ((8, 3), 0), ((16, 17), 3), ((31, 18), 8), ((64, 65), 1), ((127, 20), 4), ((200, 136), 3),
         ((300, 9), 17), ((512, 33), 2), ((511, 300), 7), ((5, 9, 6), 1), ((33, 20, 3), 0), ((12, 40, 17), 2)]


@pytest.mark.parametrize("n,L", CASES)
@pytest.mark.parametrize("prec", [0, 1])
def test_parts_stay_apart(rte, n, L, prec):
    say("mode parts", n, L, prec)
    mu_a, mu_s, h = 0.2, 3.0, 1.0 / max(n)
    dim = len(n)
    sh = inputs.hg_sigma_hat(0.6, L)
    ctx = rte.Context(n, h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=prec)
    rng = np.random.default_rng(sum(n) + L)
    shape = tuple(ctx.mode_shape)
    field = (lambda: symmetric(rng, shape)) if dim == 2 else (lambda: rng.standard_normal(shape).astype(complex))
    p, q = field(), field()
    for op, name in ((rte.OP_A, "A"), (rte.OP_KT, "KT")):
        y = host(ctx.apply(dev(p), op=op)).reshape(shape)
        if dim == 2:
            assert np.array_equal(y, np.conj(y[::-1]))
        else:
            assert not y.imag.any()
        y = host(ctx.apply(dev(1j * p), op=op)).reshape(shape)
        if dim == 2:
            assert np.array_equal(y, -np.conj(y[::-1]))
        else:
            assert not y.real.any()
        if prec == rte.PREC_FP32:
            yp, yq = parts(host(ctx.apply(dev(p + 1e-8j * q), op=op)).reshape(shape), dim)
            if dim == 2:
                ref = [op2.apply_fft(v, L, h, mu_a + mu_s, mu_s, sh, name) for v in (p, q)]
            else:
                ref = [o3s.apply_fft(v.real, L, h, mu_a + mu_s, mu_s, sh, name) for v in (p, q)]
            e = [relerr(yp, ref[0]), relerr(1e8 * yq, ref[1])]
            say(f"  {name}: relerr of p {e[0]:.2e}, of a q 1e-8 of it {e[1]:.2e}")
            assert max(e) <= 1e-6
    ctx.close()
