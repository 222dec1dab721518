"""8-bit output whose rows lie far apart on the GPU: the bytes of the same frame in compact memory, and none written in
between, plain, with a forced configuration and served.  The 8-bit kernel forms a tile's offsets in 32 bits, so from
31 rows of 2^32 / 31 bytes on such frames are the FP32 kernel's."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,pitch,block", [(32, 138_547_332, 32), (32, 138_547_333, 32), (40, 140_000_000, 32), (20, 1 << 28, 32),
                                              (3, (1 << 32) + 5, 32), (40, 140_000_000, 16), (40, 140_000_000, 64)])
def test_output(fov, dev, rows, pitch, block):
    g = torch.Generator(device=dev).manual_seed(rows)
    x = torch.randint(0, 256, (rows, 60, 3), dtype=torch.uint8, device=dev, generator=g)
    p = synth.params_dict(12.0, 9.0, 3.0, 0.6, 9.0, block)
    buf = torch.full((rows * pitch,), 7, dtype=torch.uint8, device=dev)
    far = buf.as_strided((rows, 60, 3), (pitch, 3, 1))
    near = fov.forward(x, p, layout="HWC")
    f32 = fov.forward(x, p, layout="HWC", out_dtype=torch.float32)
    assert torch.equal(near, f32.round().clamp(0, 255).to(torch.uint8))

    def check(what):
        torch.cuda.synchronize()
        assert torch.equal(far, near), what
        far.fill_(7)
        assert all(bool((c == 7).all()) for c in buf.split(1 << 30)), what

    fov.forward(x, p, layout="HWC", out=far)
    check("forward")
    fov.forward_batch([x], [p], [far], layout="HWC")
    check("batch")
    fov.tuning_force(1, 64, 0, 0, 0)
    try:
        fov.forward(x, p, layout="HWC", out=far)
    finally:
        fov.tuning_force(None)
    check("forced")
    with fov.Server(hbm_budget_bytes=1 << 20, max_batch_frames=4, max_inflight_batches=1, max_fragments=4096, max_block=64,
                    max_sigma=9.0) as server:
        server.submit(x, far, p)
        server.drain()
    check("served")
