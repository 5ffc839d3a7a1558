"""Restart lengths whose device Arnoldi state ends just below a page: the factors of the basis vectors are its
last block, so a state one block short would overlap the next allocation.  Several sources at once, which
allocate the state for the restart length itself, twice, then one source alone: the oracle's residual."""
import pytest

from gpu_util import dev, host, say
from paper_1802_03061_amd import inputs
from test_gpu_diffusive import residual, rte, source  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 20, 48, 57, 65, 96, 121, 128])
@pytest.mark.parametrize("prec", [0, 1])
def test_restart(rte, m, prec):  # noqa: F811
    n, L, mu_a, mu_s = (45, 16), 3, 0.1, 30.0
    h, sh = 0.02, inputs.hg_sigma_hat(0.5, 3)
    ctx = rte.Context(n, h=h, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=prec)
    ctx.set_opts(restart=m, max_cycles=400)
    fs = [source(n, k) for k in range(3)]
    out = []
    for _ in range(2):
        us, infos = ctx.solve_multi([dev(f) for f in fs], tol=1e-8)[:2]
        out += list(zip(fs, us))
    u, info = ctx.solve(dev(fs[0]), tol=1e-8)
    say(f"restart {m} prec {prec}: iterations alone {info['iterations']}")
    for f, v in out + [(fs[0], u)]:
        assert residual((n[1], n[0]), L, h, mu_a, mu_s, sh, f, host(v)) <= 1.2e-8
    ctx.close()
