"""The network's forward and gradient at the edges of its tiles and of its launch rules: images of one
pixel, odd rows, whole 32-pixel tiles, the largest image whose activations stay in LDS between layers
(28^2) and the next one (a launch per layer, rows of 16 or 32), and a batch of so many tiles that the
weight gradients go layer by layer.  Against the FP64 oracle with the network tests' bars for BF16
operands through up to five layers: 3e-2 forward, 5e-2 gradients."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, relerr, say
from oracle import convnet as cn
from test_gpu_pc import pack, unpack

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("C,hidden,layers,B,H,W", [
    (1, 16, 2, 2, 1, 1), (3, 32, 3, 2, 5, 7), (17, 32, 5, 2, 16, 16), (9, 16, 4, 3, 8, 20), (5, 32, 5, 1, 28, 28),
    (5, 32, 3, 1, 29, 29), (3, 16, 3, 2, 2, 200), (7, 32, 3, 1, 300, 9), (17, 32, 3, 1, 40, 33), (3, 16, 3, 300, 4, 4)])
def test_forward_and_gradient_match_oracle(C, hidden, layers, B, H, W):
    from paper_1802_03061_amd import rte
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    rng = np.random.default_rng(C + 10 * H + W)
    net = rte.Net(C, hidden, layers, seed=C)
    params = [(Wt, 0.1 * rng.standard_normal(b.shape)) for Wt, b in unpack(host(net.params()), C, hidden, layers)]
    net.set_params(dev(pack(params)))
    x, t = (rng.standard_normal((B, C, H, W)).astype(np.float32) for _ in range(2))
    w = (rng.random(B) + 0.5).astype(np.float32)
    y, _ = cn.net_forward(x.astype(np.float64), params)
    e = relerr(host(net.forward(dev(x))), y)
    ref_loss, ref = cn.coarse_loss(x.astype(np.float64), t.astype(np.float64), w.astype(np.float64), params)
    gref = np.concatenate([np.concatenate([gW.reshape(-1), gb]) for gW, gb in ref])
    for _ in range(2):      # the second call reuses every buffer
        loss, g = net.loss_grad(dev(x), dev(t), dev(w), want_grad=True)
        eg = relerr(host(g), gref)
        say("nn tiles", C, hidden, layers, B, H, W, f"forward {e:.2e} gradient {eg:.2e} loss {loss:.6g} ({ref_loss:.6g})")
        assert e <= 3e-2 and eg <= 5e-2 and abs(loss - ref_loss) <= 2e-2 * abs(ref_loss)
    net.close()
