"""The FP32 kernel on 8-bit frames under every launch configuration (8-bit output of up to radius 48 with three channels runs on the
8-bit kernel, for which most configurations are one launch), and both kernels at work item counts around whole rounds of 64,
which are dealt to the dies in another order than a last, shorter round."""
import pytest
import torch

import synth
from test_tuning_gpu import run_all_configs

pytestmark = pytest.mark.gpu


# channels, block, largest radius, output: gray frames that the FP32 kernel takes by rule, float output, radii from 49 on;
# fragments that reach past the frame, odd numbers of rows
@pytest.mark.parametrize("c,block,radius,out", [(1, 24, 24, "u8"), (1, 16, 40, "u8"), (1, 5, 3, "u8"), (3, 32, 16, "f32"), (3, 24, 40, "f32"),
                                                (3, 32, 49, "u8"), (1, 31, 70, "u8"), (2, 48, 60, "u8"), (3, 8, 8, "u8")])
def test_every_config_8_bit_input(fov, dev, c, block, radius, out):
    g = torch.Generator(device=dev).manual_seed(block + radius)
    h, w = 5 * block + 3, 9 * block - 2
    x = torch.randint(0, 256, (h, w, c), dtype=torch.uint8, device=dev, generator=g)
    p = synth.params_dict(0.3 * w, 0.7 * h, block / 2, 4.0 / block, (radius - 0.5) / 3.0, block)
    o = torch.float32 if out == "f32" else torch.uint8
    base = run_all_configs(fov, lambda: fov.forward(x, p, layout="HWC", out_dtype=o))
    f = fov.forward(x, p, layout="HWC", out_dtype=torch.float32)
    assert torch.equal(base, f if out == "f32" else f.round().clamp(0, 255).to(torch.uint8))


@pytest.mark.parametrize("n", [1, 7, 63, 64, 65, 127, 128, 129])
def test_item_counts(fov, dev, orc, n):
    # n fragments: n items of the 8-bit kernel and of the FP32 kernel with one channel; with three channels it has 3 n by
    # default and n where the configuration says so
    g = torch.Generator(device=dev).manual_seed(n)
    x = torch.randint(0, 256, (17, 24 * n - 5, 3), dtype=torch.uint8, device=dev, generator=g)
    p = synth.params_dict(10.0 * n, 8.0, 6.0, 0.2, 3.9, 24)
    want = torch.from_numpy(orc.forward(x.double().cpu().numpy().transpose(2, 0, 1), p).transpose(1, 2, 0)).to(dev)
    f = fov.forward(x, p, layout="HWC", out_dtype=torch.float32)
    assert (f.double() - want).abs().max() <= 255 * 2e-5
    assert torch.equal(fov.forward(x, p, layout="HWC"), f.round().clamp(0, 255).to(torch.uint8))
    one = fov.forward(x[:, :, :1].contiguous(), p, layout="HWC", out_dtype=torch.float32)
    assert torch.equal(one, f[:, :, :1])
    fov.tuning_force(1, 64, 0, 0, 0)
    try:
        assert torch.equal(fov.forward(x, p, layout="HWC", out_dtype=torch.float32), f)
    finally:
        fov.tuning_force(None)


@pytest.mark.parametrize("radius", [3, 8, 9, 16, 17])
@pytest.mark.parametrize("w", [1365, 1366])  # 3 x 1024 x w bytes: below and above 4 MiB, from which rows are taken up to radius 16
def test_order_of_small_radii(fov, dev, radius, w):
    g = torch.Generator(device=dev).manual_seed(radius)
    x = torch.randint(0, 256, (3, 1024, w), dtype=torch.uint8, device=dev, generator=g)
    p = synth.params_dict(0.3 * w, 700.0, 32.0, 0.02, (radius - 0.5) / 3.0, 32)
    f = fov.forward(x, p, layout="CHW", out_dtype=torch.float32)
    assert torch.equal(fov.forward(x, p, layout="CHW"), f.round().clamp(0, 255).to(torch.uint8))
