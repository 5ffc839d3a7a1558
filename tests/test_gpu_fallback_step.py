"""The step that a solve goes on with after it has dropped its preconditioner (normalised basis vectors,
rescaled where their norm is off): with the rescaling at its tolerance and forced at every step, both basis
types, restarts shorter and longer than 16 vectors and a diffusive medium.  As many iterations as a plain
solve, one or two more allowed in each cycle, and the oracle's FP64 residual: the solver stops at 1e-9, its
apply agrees with the oracle's to 1e-12 of the largest term."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, say
from paper_1802_03061_amd import inputs
from test_gpu_diffusive import residual, rte, source  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("renorm", ["", "-1"])
@pytest.mark.parametrize("basis32", [0, 1])
@pytest.mark.parametrize("n,L,mu_s,restart", [(32, 1, 5.0, 64), (64, 0, 100.0, 20), (48, 2, 10.0, 7)])
def test_after_fallback(rte, monkeypatch, n, L, mu_s, restart, basis32, renorm):  # noqa: F811
    say("fallback step", n, L, mu_s, restart, basis32, renorm)
    if renorm:
        monkeypatch.setenv("RTE_RENORM_TOL", renorm)
    else:
        monkeypatch.delenv("RTE_RENORM_TOL", raising=False)
    mu_a, sh = 0.1, inputs.hg_sigma_hat(0.5, L)
    ctx = rte.Context((n, n), h=1.0 / n, mu_a=mu_a, mu_s=mu_s, sigma_hat=sh, L=L, prec=rte.PREC_FP32)
    opts = dict(restart=restart, max_cycles=100, basis_fp32=basis32)
    f = source((n, n), L)
    ctx.set_opts(**opts)
    _, plain = ctx.solve(dev(f), tol=1e-9)
    net = rte.Net(ctx.channels, 32, 5, seed=1)
    ctx.attach_pc(torch.full((net.nparam,), float("nan"), dtype=torch.float32, device="cuda"), factor=4)
    ctx.set_opts(**opts)
    u, info = ctx.solve(dev(f), tol=1e-9)
    e = residual((n, n), L, 1.0 / n, mu_a, mu_s, sh, f, host(u))
    say(f"  iterations {info['iterations']} (plain {plain['iterations']}) cycles {info['cycles']} residual {e:.2e}")
    assert plain["pc_used"] == 0 and info["pc_fallback"] == 1
    # the iterations of the dropped cycle (two at most are queued before the host sees the fault) count too
    assert abs(info["iterations"] - plain["iterations"]) <= 2 + 2 * info["cycles"]
    assert e <= 1.2e-9
    ctx.close()
    net.close()
