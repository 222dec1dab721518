"""The matrix-core gather of the 32-bit adjoint (fragment sides 16 and 28 .. 32) on the GPU, at the edges of its
32-pixel tiles, against the oracle's transpose.

An output is a sum over the fragments that reach it of two nested products of at most 32 terms each, in
FP32: below 100 roundings of 2^-24 on sums of non-negative terms, 6e-6 of the value; the bound is that of
the other 32-bit adjoint tests, 2e-5 of the largest output (1 if that is smaller)."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def check(got, ref, what):
    assert np.max(np.abs(got.cpu().numpy() - ref)) <= 2e-5 * max(1.0, np.abs(ref).max()), what


# radii ceil(3 cap): 1, around 16 and 32 (the reach of one and two fragments of 16, of one of 32) and beyond
@pytest.mark.parametrize("cap", [0.2, 5.2, 5.5, 10.6, 11.0, 16.0])
@pytest.mark.parametrize("block", [15, 16, 17, 27, 28, 31, 32, 33])  # 16 and 28 .. 32 are gathered
def test_blocks_and_radii(fov, orc, dev, block, cap):
    rng = np.random.default_rng(block)
    h, w = 3 * block + 5, 4 * block - 1
    p = synth.params_dict(w * 0.4, h * 0.6, 3.0, 0.5, cap, block, -(block // 3), -(block - 1))
    g = rng.random((2, h, w)).astype(np.float32)
    got = fov.backward(torch.from_numpy(g).to(dev), p, layout="CHW")
    check(got, orc.adjoint(g.astype(np.float64), p), (block, cap))


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 40), (5, 33, 1), (3, 2, 17), (1, 32, 32), (2, 16, 64)])
@pytest.mark.parametrize("block", [16, 32])
def test_small_frames(fov, orc, dev, shape, block):
    g = np.random.default_rng(3).random(shape).astype(np.float32)
    p = synth.params_dict(0.0, 0.0, 0.0, 1.0, 12.0, block, -7, -2)
    got = fov.backward(torch.from_numpy(g).to(dev), p, layout="CHW")
    check(got, orc.adjoint(g.astype(np.float64), p), (shape, block))


def test_strides_and_sigma_map(fov, orc, dev):
    rng = np.random.default_rng(4)
    h, w, B = 70, 101, 16
    p = synth.params_dict(0, 0, 0, 0, 9.0, B, -5, -11)
    smap = rng.uniform(-1, 11, size=orc.grid(h, w, p)).astype(np.float32)
    smap[0, 0] = np.nan
    pd = dict(p, sigma_map=torch.from_numpy(smap.reshape(-1)).to(dev))
    g = rng.random((h, 2 * w, 3)).astype(np.float32)
    for cols in (slice(None, None, 2), slice(0, w)):  # every second pixel; rows of a wider frame
        ref = orc.adjoint(g[:, cols].transpose(2, 0, 1).astype(np.float64), p, sigma_map=smap.astype(np.float64))
        x = torch.from_numpy(g).to(dev)[:, cols].permute(2, 0, 1)
        check(fov.backward(x, pd, layout="CHW"), ref, cols)


def test_rows_far_apart(fov, orc, dev):
    # rows of a fragment that span more than 2^31 bytes
    g = np.random.default_rng(7).random((1, 33, 40)).astype(np.float32)
    p = synth.params_dict(12.0, 9.0, 2.0, 0.3, 6.0, 32, 0, -4)
    x = torch.zeros(33 * 18_000_000, device=dev).as_strided((1, 33, 40), (1, 18_000_000, 1))
    x.copy_(torch.from_numpy(g).to(dev))
    got = fov.backward(x, p, layout="CHW", grad_in=torch.empty(1, 33, 40, device=dev))
    check(got, orc.adjoint(g.astype(np.float64), p), "far")


@pytest.mark.parametrize("n", [5, 18])
def test_frame_table_of_mixed_blocks(fov, orc, dev, n):
    # frames that travel in the kernel arguments and more than do, one or two fragments per tile side
    rng = np.random.default_rng(5)
    c, h, w = 2, 60, 75
    ps = [synth.params_dict(rng.uniform(0, w - 1), rng.uniform(0, h - 1), 2.0, 0.3, rng.uniform(1, 12),
                            (16, 32, 29)[i % 3], -int(rng.integers(0, 16)), -int(rng.integers(0, 16))) for i in range(n)]
    g = rng.random((n, c, h, w)).astype(np.float32)
    got = fov.backward(torch.from_numpy(g).to(dev), ps)
    for i in range(n):
        check(got[i], orc.adjoint(g[i].astype(np.float64), ps[i]), i)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("block", [16, 32])
def test_non_finite_gradients_stay_local(fov, orc, dev, block, bad):
    rng = np.random.default_rng(6)
    h, w = 90, 110
    p = synth.params_dict(40.0, 30.0, 4.0, 0.2, 7.0, block, -3, -9)
    g = rng.random((1, h, w)).astype(np.float32)
    at = (0, 52, 71)
    one = np.zeros((1, h, w))
    one[at] = 1.0
    reached = orc.adjoint(one, p) != 0.0
    g[at] = 0.0
    ref = orc.adjoint(g.astype(np.float64), p)
    g[at] = bad
    got = fov.backward(torch.from_numpy(g).to(dev), p, layout="CHW").cpu().numpy()
    assert np.array_equal(~np.isfinite(got), reached)
    assert np.max(np.abs(got[~reached] - ref[~reached])) <= 2e-5 * max(1.0, np.abs(ref).max())
