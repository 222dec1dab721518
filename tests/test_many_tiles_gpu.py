"""8-bit fragments of more than one tile in numbers around what one launch holds with an item per tile."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fragments", [(1 << 22) - 1, 1 << 22])  # four items each: just below 2^24, and as many
def test_one_row_of_fragments(fov, dev, fragments):
    w = 33 * fragments
    g = torch.Generator(device=dev).manual_seed(1)
    x = torch.randint(0, 256, (3, 1, w), dtype=torch.uint8, device=dev, generator=g)
    p = synth.params_dict(w / 3.0, 0.0, 100.0, 0.5, 15.9, 33)
    assert fov.grid(1, w, p) == (1, fragments)
    y = fov.forward(x, p, layout="CHW")
    f = fov.forward(x, p, layout="CHW", out_dtype=torch.float32)
    torch.cuda.synchronize()
    for a, b in zip(y.view(-1).split(1 << 27), f.view(-1).split(1 << 27)):
        assert torch.equal(a, b.round_().clamp_(0, 255).to(torch.uint8))
