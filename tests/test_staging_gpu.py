"""Staging of float frames on the GPU: frames whose bytes pass 31 bits, which are not read with buffer loads,
give the bits of the same frame in compact memory; tiles on both sides of the 64- and 128-column chunks."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("cap", [5.2, 5.5, 15.9, 16.3])  # radii 16, 17, 48, 49
def test_far_rows(fov, orc, dev, dtype, cap):
    h, w, pitch = 33, 60, 17_000_000
    x = np.random.default_rng(2).random((1, h, w))
    p = synth.params_dict(12.0, 9.0, 0.0, 0.6, cap, 32, 0, -4)
    near = torch.from_numpy(x).to(dev, dtype)
    far = torch.zeros(h * pitch, device=dev, dtype=dtype).as_strided((1, h, w), (h * pitch, pitch, 1))
    far.copy_(near)
    assert far.element_size() * (h - 1) * pitch > 2**31
    a = fov.forward(near, p, layout="CHW")
    b = fov.forward(far, p, layout="CHW", out=torch.empty_like(near))
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    # two FP32 sums of at most 99 terms with weights of sum 1: below 200 roundings of 2^-24
    bound = 1.2e-5 if dtype == torch.float32 else 1e-12
    assert np.max(np.abs(a.cpu().numpy() - orc.forward(near.cpu().numpy().astype(np.float64), p))) <= bound
