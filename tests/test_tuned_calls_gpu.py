"""Tuned 8-bit calls on the GPU: no slower than untuned ones, and a tuned frame leaves calls of the other kernel alone."""
import pytest
import torch

import synth
from test_kernel_choice_gpu import least_us

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def clear(fov):
    fov.tuning_clear()
    yield
    fov.tuning_clear()


@pytest.mark.parametrize("h,w,c,block", [(2160, 3840, 1, 16), (2160, 3840, 1, 24), (4800, 3840, 1, 64), (1080, 1920, 3, 32), (480, 640, 3, 64)])
def test_no_slower(fov, dev, tmp_path, h, w, c, block):
    x = torch.randint(0, 256, (h, w, c), dtype=torch.uint8, device=dev)
    p = synth.params_dict(0.4 * w, 0.6 * h, 32.0, 0.03, 15.9, block)
    y = torch.empty_like(x)
    call = lambda: fov.forward(x, p, out=y, layout="HWC")  # noqa: E731
    plain, want = least_us(call), y.clone()
    best = fov.autotune(x, p, out=y, layout="HWC", reps=9)
    assert torch.equal(y, want)
    assert best["split"] in (1, 2, 4) and best["merge"] in (0, 1) and best["chan_split"] in (0, 1) and fov.tuning_count() == 1
    assert least_us(call) < 1.15 * plain, best
    path = str(tmp_path / "t.txt")
    fov.tuning_save(path)
    fov.tuning_clear()
    fov.tuning_load(path)
    assert fov.tuning_count() == 1
    assert least_us(call) < 1.15 * plain, best
    assert torch.equal(y, want)


def test_other_kernel_and_sides_untouched(fov, dev, tmp_path):
    # a split that the file forces on RGB frames of 32 px: not taken for the same shape in RGBA memory (the FP32 kernel), nor for a
    # batch with smaller fragments, and a version-3 entry for none of them
    arch = torch.cuda.get_device_properties(0).gcnArchName
    x4 = torch.randint(0, 256, (1080, 1920, 4), dtype=torch.uint8, device=dev)
    x, y = x4[:, :, :3].contiguous(), torch.empty((1080, 1920, 3), dtype=torch.uint8, device=dev)
    p = synth.params_dict(700.0, 600.0, 32.0, 0.05, 15.9)
    calls = [lambda: fov.forward(x, p, out=y, layout="HWC"), lambda: fov.forward(x4[:, :, :3], p, out=y, layout="HWC")]
    want = calls[0]().clone()
    plain = [least_us(c) for c in calls]
    f = tmp_path / "t.txt"
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    f.write_text("fov-tune-v3 %s %d 0 0 3 32 6 11 0 : 4 16 0 0 0 9.0\n" % (arch, cus))
    fov.tuning_load(str(f))
    now = [least_us(c) for c in calls]
    assert now[0] < 1.15 * plain[0], (now, plain)
    assert now[1] > 1.3 * plain[1], (now, plain)  # the FP32 kernel, for which it was made
    fov.tuning_clear()
    f.write_text("fov-tune-v4 %s %d 0 0 3 32 6 11 0 32 : 4 64 0 0 0 9.0\n" % (arch, cus))
    fov.tuning_load(str(f))
    now = [least_us(c) for c in calls]
    assert now[0] > 1.3 * plain[0], (now, plain)
    assert now[1] < 1.15 * plain[1], (now, plain)
    for c in calls:
        y.zero_()
        assert torch.equal(c(), want)
