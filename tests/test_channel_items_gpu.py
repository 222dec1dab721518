"""Calls on both sides of the fragment count from which a work item holds all channels of its fragment: the bits
of each channel's own call."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,out_dtype", [(torch.float32, torch.float32), (torch.uint8, torch.float32),
                                             (torch.float64, torch.float64)])
@pytest.mark.parametrize("w", [7 * 329 - 3, 7 * 330 - 3, 7 * 400 - 3])  # 2303, 2310, 2800 fragments; 9 x 256 is the line
def test_channels(fov, dev, dtype, out_dtype, w):
    g = torch.Generator(device=dev).manual_seed(w)
    x = torch.randint(0, 256, (1, 3, 45, w), device=dev, generator=g).to(dtype)
    p = synth.params_dict(w * 0.3, 20.0, 4.0, 0.02, 6.0, 7, -3, -2)
    nby, nbx = fov.grid(45, w, p)
    assert (nby, nbx) == (7, -(-(w + 3) // 7))
    y = fov.forward(x, p, out_dtype=out_dtype)
    for c in range(3):
        assert torch.equal(y[:, c:c + 1], fov.forward(x[:, c:c + 1].contiguous(), p, out_dtype=out_dtype)), c
