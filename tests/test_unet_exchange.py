"""The driver's exchanges: which call does them."""
import pytest
import torch

from paper_1909_03108_amd import sp3d, synth
from paper_1909_03108_amd import unet as PU
from gpu_util import to_dev


def test_an_exchange_that_fails_leaves_the_driver_as_it_was():
    """_exchange is where a program can put its own delivery; after one that raised the next direct call has to exchange."""
    net = PU.UNet.__new__(PU.UNet)
    net.dt = sp3d.SP_BF16
    g = sp3d.Geom(1, (8, 8, 8), (2, 2, 1))

    def lost(P, g, c):
        raise OSError("peer is gone")
    net._exchange = lost
    before = dict(vars(net))
    with pytest.raises(OSError):
        net._with_exchange(g, (None, 32))
    assert vars(net) == before


@pytest.mark.gpu
@pytest.mark.parametrize("gather", [False, True])
def test_every_exchange_is_a_flag_of_a_convolution(gather, monkeypatch):
    """What passes through _exchange is what the convolutions are called to fill: the same tensors, in the same order."""
    channels, in_ch, classes, convs = (32, 64, 128), 1, 3, 2
    n, dhw, grid = 1, (16, 32, 64), (2, 2, 1)
    w = {name: to_dev(synth.weights(shape[3], shape[4], 100 + k, "bf16", taps=shape[:3]))
         for k, (name, shape) in enumerate(PU.layer_plan(channels, in_ch, classes, convs))}
    net = PU.UNet(n, dhw, grid, w, channels, in_ch, classes, convs=convs, gather=gather)
    asked, flagged = [], []
    inner = net._exchange

    def hook(P, g, c):
        asked.append(P.data_ptr())
        inner(P, g, c)
    net._exchange = hook

    def watch(name, inputs):
        call = getattr(sp3d, name)

        def watched(*a, **k):
            g = next(x for x in a if isinstance(x, sp3d.Geom))
            if g.opts & sp3d.SP_HALO_EXCHANGE:
                flagged.extend(a[i].data_ptr() for i in inputs)
            return call(*a, **k)
        monkeypatch.setattr(sp3d, name, watched)
    for name in ("conv3d_fwd", "conv3d_fwd_bits", "conv3d_dgrad", "conv3d_dgrad_relu", "conv3d_dgrad_bits", "conv3d_dgrad2"):
        watch(name, (0,))
    for name in ("conv3d_fwd2", "conv3d_fwd2_bits"):
        watch(name, (0, 2))
    monkeypatch.setattr(sp3d, "sp_halo_exchange", lambda *a, **k: pytest.fail("an exchange in a launch of its own"))
    x = to_dev(synth.ct_like_volume((n,) + dhw + (in_ch,), 9130, "bf16"))
    logits = net.forward(x)
    net.backward(torch.ones_like(logits))
    assert asked and asked == flagged
