"""The plain solver's step (Arnoldi on K with lazy factors, the Gram-Schmidt update fused with pass A):
row tiles with remainders, odd and unaligned rows, the smallest and the padded x-lengths 16..1024, the
split form's unpacked spectra (L = 17), 3D slabs, an FP32 basis, a short restart (many cycles) and a long
one (more than 16 vectors, two dot launches), no scattering at all (K = 0) and several right-hand
sides.  Checked by the oracle's residual |K~ f - A u| / |K~ f|: the solver stops at an FP64 residual of
1e-10 and its apply agrees with the oracle's to 1e-12 of the largest term, so 2e-10 bounds it."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, say
from oracle import operator2d as op2
from oracle import operator3d as op3
from oracle import operator3d_sh as o3s
from paper_1802_03061_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rte():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1802_03061_amd import rte as r
    r.load()
    return r


def residual(shape, L, h, mu_a, mu_s, sh, f, u):
    if len(shape) == 2:
        b = op2.rhs(f, L, h, mu_a + mu_s)
        r = b - op2.apply_fft(u, L, h, mu_a + mu_s, mu_s, sh, "A")
    elif L == 0:
        b = op3.apply_fft(f, h, mu_a + mu_s, mu_s, "KT")
        r = b - op3.apply_fft(u[0].real, h, mu_a + mu_s, mu_s, "A")
    else:
        b = o3s.rhs(f, L, h, mu_a + mu_s)
        r = b - o3s.apply_fft(u.real, L, h, mu_a + mu_s, mu_s, sh, "A")
    return float(np.linalg.norm(r) / np.linalg.norm(b))


CASES = [((3, 2), 1, {}), ((8, 7), 0, {}), ((9, 33), 3, {}), ((31, 18), 2, dict(restart=3, max_cycles=200)),
         ((64, 65), 0, {}), ((65, 30), 4, {}), ((127, 21), 2, dict(restart=40)), ((256, 9), 8, {}),
         ((301, 40), 1, {}), ((511, 6), 2, {}), ((512, 33), 0, {}), ((12, 10), 17, {}), ((7, 5, 6), 0, {}),
         ((9, 4, 11), 1, {}), ((20, 33, 17), 0, dict(restart=4, max_cycles=200)), ((33, 6, 5), 2, {})]


@pytest.mark.parametrize("n,L,opts,mu_s", [c + (6.0,) for c in CASES] +
                         [((9, 33), 3, {}, 0.0), ((7, 5, 6), 0, {}, 0.0)])
@pytest.mark.parametrize("prec,basis32", [(0, 0), (1, 0), (0, 1)])
def test_solve_residual(rte, n, L, opts, mu_s, prec, basis32):
    say("solve", n, L, opts, mu_s, prec, basis32)
    shape = tuple(reversed(n))
    mu_a, h = 0.1, 1.0 / max(n)
    sh = inputs.hg_sigma_hat(0.5, L)
    ctx = rte.Context(n, h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=prec)
    ctx.set_opts(use_pc=0, basis_fp32=basis32, **{"max_cycles": 40, **opts})
    rng = np.random.default_rng(sum(n) + L)
    f = rng.standard_normal(shape)
    u, info = ctx.solve(dev(f), tol=1e-10)
    e = residual(shape, L, h, mu_a, mu_s, sh, f, host(u))
    say(f"  iterations {info['iterations']} cycles {info['cycles']} oracle residual {e:.2e}")
    assert e <= 2e-10
    if len(n) == 2 and not basis32:
        fs = [rng.standard_normal(shape) for _ in range(3)]
        us, _, rc = ctx.solve_multi([dev(g) for g in fs], tol=1e-10)
        assert rc == rte.RTE_OK
        # the stacked system stops at 1e-10 of the stacked right-hand side: the smallest of the three
        # may carry sqrt(3) of that times the ratio of the norms, well under a factor of 3
        assert max(residual(shape, L, h, mu_a, mu_s, sh, g, host(v)) for g, v in zip(fs, us)) <= 6e-10
    ctx.close()
