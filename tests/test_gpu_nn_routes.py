"""Forward and gradient on both sides of the rules that choose between one launch for all layers and a
launch per layer: one round of 32-pixel tiles (256 pixels) and one pixel row more, the last image of one
and a half rounds (384 pixels) and the next one, and batches whose layers have as many blocks as the chip has
units, and more.  Against the FP64 oracle with the network tests' bars for BF16 operands: 3e-2 forward, 5e-2
gradients."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, relerr, say
from oracle import convnet as cn
from test_gpu_pc import pack, unpack

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("B,H,W", [(1, 16, 16), (2, 17, 16), (1, 16, 24), (1, 24, 16), (1, 16, 25), (1, 19, 21),
                                   (51, 20, 20), (52, 20, 20), (85, 24, 24), (86, 24, 24)])
def test_forward_and_gradient_match_oracle(B, H, W):
    from paper_1802_03061_amd import rte
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    C, hidden, layers = 3, 16, 3
    rng = np.random.default_rng(B + 10 * H + W)
    net = rte.Net(C, hidden, layers, seed=C)
    params = [(Wt, 0.1 * rng.standard_normal(b.shape)) for Wt, b in unpack(host(net.params()), C, hidden, layers)]
    net.set_params(dev(pack(params)))
    x, t = (rng.standard_normal((B, C, H, W)).astype(np.float32) for _ in range(2))
    w = (rng.random(B) + 0.5).astype(np.float32)
    y, _ = cn.net_forward(x.astype(np.float64), params)
    e = relerr(host(net.forward(dev(x))), y)
    ref_loss, ref = cn.coarse_loss(x.astype(np.float64), t.astype(np.float64), w.astype(np.float64), params)
    gref = np.concatenate([np.concatenate([gW.reshape(-1), gb]) for gW, gb in ref])
    loss, g = net.loss_grad(dev(x), dev(t), dev(w), want_grad=True)
    eg = relerr(host(g), gref)
    say("nn routes", B, H, W, f"forward {e:.2e} gradient {eg:.2e} loss {loss:.6g} ({ref_loss:.6g})")
    assert e <= 3e-2 and eg <= 5e-2 and abs(loss - ref_loss) <= 2e-2 * abs(ref_loss)
    net.close()
