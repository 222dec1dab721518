"""Float frames beyond 2^31 bytes whose strips are not, on the GPU: the bits of the same frame in compact memory, at
the time per pixel of a frame below that size."""
import pytest
import torch

import synth
from test_kernel_choice_gpu import least_us

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("h,pitch,channel", [(170, 16_000_000, 60), (170, 60, 1 << 30), (170, 32_000_000, 1_000_000), (33, 33_000_000, 60),
                                             (33, 35_000_000, 60)])  # in bytes / 4; the last: 63 rows pass 2^31 bytes
@pytest.mark.parametrize("cap", [1.0, 16.3])
def test_bits(fov, dev, dtype, h, pitch, channel, cap):
    size = torch.empty(0, dtype=dtype).element_size()
    pitch, channel = max(pitch * 4 // size, 60), max(channel * 4 // size, 60)  # rows do not overlap
    if channel < h * pitch and pitch < 2 * channel:
        pitch = max(pitch, 2 * channel)  # the channels of a row side by side
    g = torch.Generator(device=dev).manual_seed(h)
    near = torch.rand((2, h, 60), device=dev, generator=g, dtype=dtype)
    far = torch.zeros(h * pitch + 2 * channel, device=dev, dtype=dtype).as_strided((2, h, 60), (channel, pitch, 1))
    far.copy_(near)
    for x_in, y_out in ((far, torch.empty_like(near)), (near, far)):
        p = synth.params_dict(12.0, 9.0, 0.0, 0.6, cap, 32, 0, -4)
        want = fov.forward(near, p, layout="CHW")
        fov.forward(x_in, p, layout="CHW", out=y_out)
        assert torch.equal(y_out, want)


def test_time_per_pixel(fov, dev):
    def per_pixel(side):
        x = torch.rand((1, side, side), device=dev)
        y = torch.empty_like(x)
        p = synth.params_dict(0.4 * side, 0.6 * side, 32.0, 0.03, 7.9)
        return least_us(lambda: fov.forward(x, p, out=y, layout="CHW"), 2, 3) / side ** 2

    below, above = per_pixel(22000), per_pixel(24000)  # 1.9 and 2.3 GB
    assert above < 1.35 * below, (below, above)  # 1.8 times when such frames were loaded without prefetching
