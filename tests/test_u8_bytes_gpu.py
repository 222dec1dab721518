"""The bytes of the matrix-core kernel of 8-bit output (radii 1 .. 48) on the GPU.

It computes each pixel in fixed point with an error bound and runs the FP32 sum
only where the bound leaves the byte open, so its bytes must be those of the
FP32 kernel: exactly the rounded values of the 8-bit to float output, which
runs the FP32 passes for every pixel.  Cases: every radius (each number of
32-wide blocks and tap tails), sigmas below one pixel, fragment sides around
the 32-pixel tile, every staging layout, windows over the frame's edges and
frames narrower than them, and images of exact half-integer means, whose tiles
are left to the FP32 passes.
"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def check(fov, x, p, layout):
    y = fov.forward(x, p, layout=layout)
    f = fov.forward(x, p, layout=layout, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = f.round().clamp(0, 255).to(torch.uint8)
    assert torch.equal(y, ref), (tuple(x.shape), p, int((y != ref).sum()))


def grating(dev, h=150, w=260, c=3, seed=4):
    return torch.from_numpy(synth.grating_frame(h, w, c, seed=seed)).to(dev)


@pytest.mark.parametrize("r0", range(0, 50, 10))
def test_every_radius(fov, dev, r0):
    x = grating(dev)
    for r in range(max(r0, 1), r0 + 10):  # 49 runs the FP32 kernel
        check(fov, x, synth.params_dict(37.25, 20.5, 0.0, 100.0, (r - 0.5) / 3.0, 32, -5, -9), "HWC")


@pytest.mark.parametrize("sigma", [1e-3, 0.05, 0.2, 0.3, 0.45, 0.6, 0.9, 1.0, 1.0 / 3.0, 16.0])
def test_small_and_limit_sigmas(fov, dev, sigma):
    check(fov, grating(dev), synth.params_dict(37.25, 20.5, 0.0, 1e4, sigma, 32, -5, -9), "HWC")


@pytest.mark.parametrize("block", [1, 3, 5, 16, 24, 31, 32, 33, 64])
def test_fragment_sides(fov, dev, block):
    p = synth.params_dict(100.0, 70.0, 10.0, 0.1, 16.0, block, -(block // 2), 0)
    check(fov, grating(dev)[:, :, 0].contiguous(), p, "HW")


@pytest.mark.parametrize("form", ["CHW", "HWC4", "CHW7", "strided", "CHW2", "planes of HWC"])
def test_layouts(fov, dev, form):
    g = torch.Generator(device=dev).manual_seed(5)
    rnd = lambda *s: torch.randint(0, 256, s, dtype=torch.uint8, device=dev, generator=g)  # noqa: E731
    p = synth.params_dict(50.0, 40.0, 10.0, 0.1, 16.0)
    x, layout = {"CHW": lambda: (rnd(3, 151, 263), "CHW"), "HWC4": lambda: (rnd(90, 131, 4), "HWC"),
                 "CHW7": lambda: (rnd(7, 90, 131), "CHW"), "strided": lambda: (rnd(64, 192, 3)[:, ::2], "HWC"),
                 "CHW2": lambda: (rnd(2, 150, 200), "CHW"),
                 "planes of HWC": lambda: (rnd(150, 200, 3).permute(2, 0, 1), "CHW")}[form]()
    check(fov, x, p, layout)


@pytest.mark.parametrize("shape", [(1, 1, 3), (2, 3, 3), (5, 2, 3), (40, 1, 3), (1, 70, 3), (3, 4, 3), (4, 5, 1), (33, 15, 3)])
def test_frames_smaller_than_a_window(fov, dev, shape):
    g = torch.Generator(device=dev).manual_seed(sum(shape))
    x = torch.randint(0, 256, shape, dtype=torch.uint8, device=dev, generator=g)
    check(fov, x, synth.params_dict(0, 0, 0, 1.0, 9.0, 32), "HWC")


@pytest.mark.parametrize("image", ["checker 0/1", "checker 0/255", "stripes", "201", "255", "0", "ramp", "edge"])
def test_images_with_ties(fov, dev, image):
    y, x = torch.meshgrid(torch.arange(200, device=dev), torch.arange(333, device=dev), indexing="ij")
    im = {"checker 0/1": (x + y) % 2, "checker 0/255": (x + y) % 2 * 255, "stripes": x % 2 * 255, "201": 0 * x + 201,
          "255": 0 * x + 255, "0": 0 * x, "ramp": x // 2 % 256, "edge": (x > 100) * 255}[image]
    im = im.to(torch.uint8)[:, :, None].expand(-1, -1, 3).contiguous()
    im[:, :, 2] = grating(dev, 200, 333, 1)[:, :, 0]  # one channel of the tile without ties
    check(fov, im, synth.params_dict(60, 60, 5, 0.2, 16.0), "HWC")


def test_forced_configurations(fov, dev):
    x, p = grating(dev, 200, 333), synth.params_dict(60, 60, 5, 0.1, 16.0, 64)
    ref = fov.forward(x, p, layout="HWC")
    for cfg in ((1, 64, 0, 1, 0), (1, 64, 0, 0, 1), (2, 64, 0, 0, 0), (4, 16, 1, 0, 0)):
        fov.tuning_force(*cfg)
        try:
            y = fov.forward(x, p, layout="HWC")
        finally:
            fov.tuning_force(None)
        assert torch.equal(y, ref), cfg


def test_1080p(fov, dev):
    check(fov, grating(dev, 1080, 1920, 3, 1), synth.params_cfg2(np.random.default_rng(9)), "HWC")
