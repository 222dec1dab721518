"""Which kernel 8-bit output runs on: the same bytes on both sides of the rule's lines, and not a multiple of the FP32
kernel's time for layouts that the 8-bit kernel reads byte by byte, nor for served gray frames of small fragments."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def least_us(fn, n=6, rounds=5):
    fn()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / n)
    return best


# channels, block, fragment columns, and radii on both sides of a line (256 compute units)
LINES = [(1, 17, 40, (24, 25)), (1, 17, 144, (36, 37)), (1, 20, 384, (40, 41)), (1, 33, 16, (32, 33)), (1, 33, 80, (40, 41)), (1, 49, 17, (32, 33)),
         (3, 16, 16, (8, 9)), (3, 5, 448, (24, 25)), (2, 5, 192, (24, 25)), (2, 5, 448, (40, 41)), (3, 28, 144, (8, 9)), (2, 32, 8, (8, 9)),
         (3, 33, 32, (24, 25)), (3, 49, 16, (4, 5)), (2, 40, 144, (36, 37))]


@pytest.mark.parametrize("c,block,cols,radii", LINES)
def test_bytes_on_both_sides(fov, dev, c, block, cols, radii):
    g = torch.Generator(device=dev).manual_seed(block)
    for nx in (cols - 1, cols):  # 16 rows of them: 256 is one a compute unit
        x = torch.randint(0, 256, (16 * block - 3, nx * block - 1, c), dtype=torch.uint8, device=dev, generator=g)
        x = x.permute(2, 0, 1).contiguous()
        for r in radii:
            p = synth.params_dict(30.0, 20.0, 4.0, 0.3, (r - 0.5) / 3.0, block)
            y = fov.forward(x, p, layout="CHW")
            f = fov.forward(x, p, layout="CHW", out_dtype=torch.float32)
            assert torch.equal(y, f.round().clamp(0, 255).to(torch.uint8)), (nx, r)


@pytest.mark.parametrize("form", ["RGBA", "RGB of RGBA", "every second column"])
def test_bytewise_layouts(fov, dev, form):
    p = synth.params_dict(700.0, 600.0, 32.0, 0.05, 15.9)
    x = torch.randint(0, 256, (1080, 1920, 4), dtype=torch.uint8, device=dev)
    if form != "RGBA":
        x = x[:, :, :3] if form == "RGB of RGBA" else x.view(1080, 3840, 2)[:, ::2, :1]
    y, f = torch.empty(x.shape, dtype=torch.uint8, device=dev), torch.empty(x.shape, device=dev)
    u8 = least_us(lambda: fov.forward(x, p, out=y, layout="HWC"))
    f32 = least_us(lambda: fov.forward(x, p, out=f, layout="HWC"))  # the FP32 kernel
    assert torch.equal(y, f.round().clamp(0, 255).to(torch.uint8))
    assert u8 < 1.3 * f32, (u8, f32)  # 2 to 3 times as long on the 8-bit kernel


def test_served_gray(fov, dev):
    p = synth.params_dict(1500.0, 1200.0, 32.0, 0.03, 7.9, 16)
    x = [torch.randint(0, 256, (2160, 3840, 1), dtype=torch.uint8, device=dev) for _ in range(4)]
    y = [torch.empty_like(t) for t in x]
    want = fov.forward(x[0], p, layout="HWC")
    plain = least_us(lambda: [fov.forward(a, p, out=b, layout="HWC") for a, b in zip(x, y)], 2)
    with fov.Server(hbm_budget_bytes=1 << 30, max_batch_frames=4, max_inflight_batches=1, max_fragments=1 << 18, max_sigma=16.0) as server:
        def served():
            tickets = [server.submit(a, b, p) for a, b in zip(x, y)]
            server.drain()
            for t in tickets:
                server.poll(t)
        took = least_us(served, 2)
    assert torch.equal(y[0], want)
    assert took < 1.25 * plain + 200.0, (took, plain)  # 1.8 times plain and more on the 8-bit kernel
