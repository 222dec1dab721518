"""Merged vertical pairs of fragments on the GPU: the bits of the launch without them, every pixel written, for frames
of all forms; and frames of an even number of fragment rows take no longer than a row more would."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def forced(fov, merge, chan, fn):
    fov.tuning_force(1, 64, 0, merge, chan)
    try:
        return fn()
    finally:
        fov.tuning_force(None)


# h, w, block, origin x and y, fixation x and y, e0, slope, cap: wide, tall, one row, one column, odd and even rows,
# shifted; gaze at the ends, far outside; nearly all at the cap, nearly none, sigma(0) > 0
FRAMES = [(200, 333, 32, 0, 0, 100.0, 80.0, 20.0, 0.3, 6.0), (333, 200, 32, -5, -9, 20.0, 300.0, 20.0, 0.3, 6.0),
          (97, 140, 16, 0, -3, 139.0, 1.0, 4.0, 0.2, 4.0), (140, 97, 16, -15, -15, 0.0, 60.0, 4.0, 0.2, 4.0),
          (9, 200, 10, 0, 0, 50.0, 3.0, 4.0, 0.2, 4.0), (200, 9, 10, 0, 0, 3.0, 50.0, 4.0, 0.2, 4.0),
          (64, 64, 64, 0, 0, 10.0, 10.0, 1.0, 1.0, 3.0), (65, 64, 64, 0, -63, 10.0, 10.0, 1.0, 1.0, 3.0),
          (120, 131, 8, 0, 0, -900.0, 4000.0, 10.0, 0.3, 3.0), (120, 131, 8, 0, 0, 60.0, 60.0, -50.0, 0.1, 6.0),
          (120, 131, 8, -1, -7, 60.0, 60.0, 0.0, 0.01, 6.0), (120, 131, 8, 0, 0, 60.0, 60.0, 30.0, 50.0, 0.2)]


@pytest.mark.parametrize("frame", FRAMES)
@pytest.mark.parametrize("dtype,out_dtype", [(torch.uint8, torch.float32), (torch.float32, torch.float32), (torch.float64, torch.float64)])
def test_frames(fov, dev, frame, dtype, out_dtype):
    h, w, block, ox, oy, fx, fy, e0, slope, cap = frame
    g = torch.Generator(device=dev).manual_seed(h * w)
    x = torch.randint(0, 256, (2, 2, h, w), device=dev, generator=g).to(dtype)
    p = synth.params_dict(fx, fy, e0, slope, cap, block, ox, oy)
    nby, nbx = fov.grid(h, w, p)
    smap = (torch.rand((nby, nbx), device=dev, generator=g) * 3 * cap).contiguous()  # two in three at the cap
    other = dict(p, fix_x=w - fx, fix_y=0.7 * fy)
    for params in (p, [p, other], [p, dict(other, sigma_map=smap)], dict(p, sigma_map=torch.full_like(smap, cap))):
        for chan in (0, 1):
            run = lambda: fov.forward(x, params, out=torch.full_like(x, float("nan"), dtype=out_dtype))  # noqa: E731
            a, b = forced(fov, 1, chan, run), forced(fov, 0, chan, run)
            assert torch.equal(a, b), (params, chan)


@pytest.mark.parametrize("n", [16, 17])  # descriptors in the kernel's arguments and in a table
@pytest.mark.parametrize("one_grid", [False, True])
def test_batches(fov, dev, n, one_grid):
    g = torch.Generator(device=dev).manual_seed(n)
    xs, ps = [], []
    for i in range(n):
        h, w, block, ox, oy, fx, fy, e0, slope, cap = FRAMES[0 if one_grid else i % len(FRAMES)]
        xs.append(torch.rand((h, w, 1), device=dev, generator=g))
        ps.append(synth.params_dict((i + 1) / n * w if one_grid else fx, fy, e0, slope, cap, block, ox, oy))
    run = lambda: fov.forward_batch(xs, ps, [torch.full_like(t, float("nan")) for t in xs])  # noqa: E731
    for a, b in zip(forced(fov, 1, 0, run), forced(fov, 0, 0, run)):
        assert torch.equal(a, b)


def test_served(fov, dev):
    g = torch.Generator(device=dev).manual_seed(3)
    xs = [torch.rand((f[0], f[1], 2), device=dev, generator=g) for f in FRAMES]
    ps = [synth.params_dict(*f[5:10], *f[2:5]) for f in FRAMES]
    outs = [torch.full_like(t, float("nan")) for t in xs]
    with fov.Server(hbm_budget_bytes=64 << 20, max_batch_frames=4, max_inflight_batches=2, max_fragments=4096, max_block=64,
                    max_sigma=6.0, in_dtype="f32", out_dtype="f32") as server:
        tickets = [server.submit(x, o, p) for x, o, p in zip(xs, outs, ps)]
        server.drain()
        assert all(server.poll(t)[0] for t in tickets)
    for x, o, p in zip(xs, outs, ps):
        assert torch.equal(o, forced(fov, 0, 0, lambda: fov.forward(x, p, layout="HWC")))


def test_even_rows_cost_no_more(fov, dev):
    # 68 and 69 rows of fragments, nearly all in merged pairs.  With an empty item after every full one the even
    # number took 1.6 times as long.
    def us(h):
        x = torch.randint(0, 256, (3, h, 3840), dtype=torch.uint8, device=dev)
        y = torch.empty((3, h, 3840), device=dev)
        p = synth.params_dict(1500.0, 1200.0, 32.0, 0.1, 15.9)
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(8):
                fov.forward(x, p, out=y, layout="CHW")
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) / 8)
        return best

    even, odd = us(68 * 32), us(69 * 32)
    assert even < 1.25 * odd, (even, odd)
