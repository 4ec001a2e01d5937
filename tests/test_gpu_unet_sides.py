"""U-Net kernels at the grid sides and channel counts where their tiling differs.

A periodic input of side 32 repeated k times has the repeated output, the same mean loss
and the same gradient, whatever tiles the levels of side 32 k are cut into.  Side 32 itself
is compared with the FP64 reference for each set of channels.  Bars as for side 32 (BF16
activations and weights, FP32 sums): 3e-2 for outputs, 6e-2 for gradients.
"""
import numpy as np
import pytest

from oracle import unet as R
from paper_1905_08890_amd import grmg
from test_gpu_unet import smooth_field

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# the last: concatenations of 80 channels, for which there is no backward pass
CHANNELS = [(16, 32, 64, 64), (16, 48, 48, 48), (16, 16, 16, 16), (16, 32, 32, 32), (16, 48, 32, 48)]


def _data(seed, cin, cout):
    rng = np.random.default_rng(seed)
    return smooth_field(rng, (cin, 32, 32, 32)), smooth_field(rng, (cout, 32, 32, 32))


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("ch", CHANNELS)
def test_side_32_matches_reference(ch):
    print(f"[gpu] unet {ch}", flush=True)
    x, t = _data(1, 5, 3)
    net = grmg.UNet(5, 3, ch, max_n=32)
    net.init(3)
    p = net.get_params().cpu().numpy().astype(np.float64)
    assert _rel(net.forward(x).cpu().numpy(), R.predict(p, x, ch, 3)) < 3e-2
    if ch[1] + ch[2] == 80:
        with pytest.raises(grmg.GrError):
            net.loss_grad(x, t)
        return
    _, g = net.loss_grad(x, t)
    _, ref = R.loss_and_grad(p, x, t, ch, 3)
    assert _rel(g.cpu().numpy().astype(np.float64), ref) < 6e-2


@pytest.mark.parametrize("ch", CHANNELS)
@pytest.mark.parametrize("k", [2, 3, 5])
def test_repeated_input_has_the_repeated_output(k, ch):
    """Sides 64, 96 and 160: levels of 8 to 160 cells, multiples of 16, 8 and only 4."""
    print(f"[gpu] unet n={32 * k} {ch}", flush=True)
    x, t = _data(2, 5, 3)
    small = grmg.UNet(5, 3, ch, max_n=32)
    small.init(5)
    y = small.forward(x).cpu().numpy()
    big = grmg.UNet(5, 3, ch, max_n=32 * k)
    big.set_params(small.get_params())
    rep = (1, k, k, k)
    Y = big.forward(np.tile(x, rep)).cpu().numpy()
    assert _rel(Y, np.tile(y, rep)) < 3e-2
    if ch[1] + ch[2] == 80:
        return
    loss, g = small.loss_grad(x, t)
    L, G = big.loss_grad(np.tile(x, rep), np.tile(t, rep))
    assert abs(L - loss) <= 3e-2 * loss
    assert _rel(G.cpu().numpy(), g.cpu().numpy()) < 6e-2
