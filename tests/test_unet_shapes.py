"""The layer shapes of the network that one native call runs (CPU)."""
from paper_1511_04633_amd import unet


def test_native_shapes_are_those_of_the_network():
    assert unet.native_shapes(unet.UNet.LEVELS) == [(ci, co) for ci, co, _, _ in unet.conv_layers()]
    assert unet.native_shapes((16,)) == [(16, 16), (16, 16), (16, 16)]
    assert len(unet.native_shapes((16,) * 8)) == 31 and unet.native_shapes((16,) * 9) is None
