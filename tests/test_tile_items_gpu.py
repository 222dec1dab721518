"""8-bit fragments of more than one 32-pixel tile, a work item each: alone, in batches with and without smaller
fragments, and served, byte for byte the rounded values of the 8-bit to float output."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def frames(dev, blocks):
    g = torch.Generator(device=dev).manual_seed(sum(blocks))
    xs = [torch.randint(0, 256, (70 + 9 * (i % 7), 150 - 11 * (i % 7), 3), dtype=torch.uint8, device=dev, generator=g)
          for i in range(len(blocks))]
    ps = [synth.params_dict(40.0 + 7 * i, 30.0, 6.0, 0.15, 16.0, b, -(b // 3), -(b - 1)) for i, b in enumerate(blocks)]
    return xs, ps


def expect(fov, x, p):
    return fov.forward(x, p, layout="HWC", out_dtype=torch.float32).round().clamp(0, 255).to(torch.uint8)


@pytest.mark.parametrize("blocks", [(33,), (63,), (64,), (64, 33, 48), (64, 32, 16), (40,) * 17])
def test_batches(fov, dev, blocks):
    xs, ps = frames(dev, blocks)
    outs = fov.forward_batch(xs, ps)
    for x, p, y in zip(xs[:4], ps, outs):
        assert torch.equal(y, expect(fov, x, p)), p["block"]


@pytest.mark.parametrize("blocks", [(64, 48), (64, 20)])
def test_served(fov, dev, blocks):
    xs, ps = frames(dev, blocks)
    outs = [torch.zeros_like(x) for x in xs]
    with fov.Server(hbm_budget_bytes=64 << 20, max_batch_frames=4, max_inflight_batches=2, max_fragments=4096,
                    max_block=64, max_sigma=16.0) as server:
        for _ in range(3):  # replays
            tickets = [server.submit(x, o, p) for x, o, p in zip(xs, outs, ps)]
            server.drain()
            assert all(server.poll(t)[0] for t in tickets)
    torch.cuda.synchronize()
    for x, p, y in zip(xs, ps, outs):
        assert torch.equal(y, expect(fov, x, p)), p["block"]


@pytest.mark.parametrize("c", [1, 3])  # one channel of at most 16 px: the FP32 kernel
@pytest.mark.parametrize("block", [1, 5, 15, 16, 17])
def test_small_sides(fov, dev, block, c):
    g = torch.Generator(device=dev).manual_seed(block)
    x = torch.randint(0, 256, (61, 83, c), dtype=torch.uint8, device=dev, generator=g)
    p = synth.params_dict(30.0, 20.0, 5.0, 0.2, 16.0, block, -(block // 3), -(block // 2))
    assert torch.equal(fov.forward(x, p, layout="HWC"), expect(fov, x, p))


@pytest.mark.parametrize("cap", [10.6, 10.7])  # radii 32 and 33: gray frames of many such fragments change kernels
@pytest.mark.parametrize("n", [15, 16])  # 255 and 272 fragments
def test_many_large_gray(fov, dev, n, cap):
    g = torch.Generator(device=dev).manual_seed(n)
    x = torch.randint(0, 256, (17 * 33 - 4, n * 33 - 7, 1), dtype=torch.uint8, device=dev, generator=g)
    p = synth.params_dict(90.0, 200.0, 5.0, 0.08, cap, 33)
    assert fov.grid(x.shape[0], x.shape[1], p) == (17, n)
    assert torch.equal(fov.forward(x, p, layout="HWC"), expect(fov, x, p))
