"""The batched solver on diffusive media (see test_gpu_diffusive.py): each problem takes no more
iterations than alone with two Gram-Schmidt passes per step, but for one or two in each cycle."""
import pytest

from gpu_util import dev, host, say
from oracle import operator2d as op2  # noqa: F401  (the residual's operator)
from test_gpu_diffusive import residual, rte, source  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
def test_iterations(rte, prec):  # noqa: F811
    import numpy as np
    media = [(n, mu_s, mu_a) for n in (33, 64, 100) for mu_s in (100.0, 400.0) for mu_a in (0.01, 1.0)]
    ctxs = [rte.Context((n, n), h=1.0 / n, mu_a=a, mu_s=s, sigma_hat=[1.0], L=0, prec=prec) for n, s, a in media]
    fs = [source((n, n), k) for k, (n, _, _) in enumerate(media)]
    us, infos, rc = rte.solve_batched(ctxs, [dev(f) for f in fs], [1e-9] * len(ctxs))
    assert rc == rte.RTE_OK
    for (n, s, a), ctx, f, u, info in zip(media, ctxs, fs, us, infos):
        ctx.set_opts(reorth=2)
        _, alone = ctx.solve(dev(f), tol=1e-9)
        e = residual((n, n), 0, 1.0 / n, a, s, np.ones(1), f, host(u))
        say(f"batched diffusive {n} {s} {a} prec {prec}: {info['iterations']} ({alone['iterations']}) residual {e:.2e}")
        assert info["iterations"] <= alone["iterations"] + 2 * info["cycles"]
        assert e <= 1.2e-9
        ctx.close()
