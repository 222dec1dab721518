"""Sigma maps that lie in an output buffer on the GPU: read as they were before the call, plain, in batches, through
the server, by the call that allocates nothing, also captured."""
import pytest
import torch

import synth
from paper_2012_08655_amd import api

pytestmark = pytest.mark.gpu

H, W, B = 1024, 1024, 8  # 128 x 128 fragments: 64 KiB of map


def make(dev, seed, dtype):
    g = torch.Generator(device=dev).manual_seed(seed)
    x = (torch.rand((1, H, W), device=dev, generator=g) * 255).to(dtype)
    m = torch.rand((H // B, W // B), device=dev, generator=g) * 5.0
    out = torch.zeros((1, H, W), device=dev, dtype=dtype)
    inside = out.view(-1).view(torch.float32)[4096:4096 + m.numel()]
    return x, m, out, inside, synth.params_dict(0.0, 0.0, 0.0, 0.0, 4.0, B)


@pytest.mark.parametrize("dtype", [torch.uint8, torch.float32])
def test_plain_and_tables(fov, dev, dtype):
    for n in (1, 3, 17):
        cases = [make(dev, n + i, dtype) for i in range(n)]
        want = [fov.forward(x, dict(p, sigma_map=m.view(-1)), layout="CHW") for x, m, _, _, p in cases]
        for which in (0, n - 1):  # the map in its own output or in another's
            for i, (_, m, out, inside, _) in enumerate(cases):
                cases[(i + which) % n][3].copy_(m.view(-1))
            ps = [dict(c[4], sigma_map=cases[(i + which) % n][3]) for i, c in enumerate(cases)]
            outs = [c[2] for c in cases]
            if n == 1:
                fov.forward(cases[0][0], ps[0], out=outs[0], layout="CHW")
            else:
                fov.forward_batch([c[0] for c in cases], ps, outs, layout="CHW")
            for i, y in enumerate(outs):
                assert torch.equal(y, want[i]), (n, which, i)


@pytest.mark.parametrize("use_graph", [True, False])
def test_served(fov, dev, use_graph):
    x, m, out, inside, p = make(dev, 5, torch.uint8)
    want = fov.forward(x, dict(p, sigma_map=m.view(-1)), layout="CHW")
    with fov.Server(hbm_budget_bytes=64 << 20, max_batch_frames=4, max_inflight_batches=2, max_fragments=1 << 15, max_block=32,
                    max_sigma=4.0, use_graph=use_graph) as server:
        for _ in range(3):
            inside.copy_(m.view(-1))
            t = server.submit(x, out, dict(p, sigma_map=inside), layout="CHW")
            server.drain()
            assert server.poll(t)[0]
            assert torch.equal(out, want)
            # and a map of its own, by the replayed step
            t = server.submit(x, out, dict(p, sigma_map=m.view(-1)), layout="CHW")
            server.drain()
            assert server.poll(t)[0]
            assert torch.equal(out, want)


@pytest.mark.parametrize("dtype", [torch.uint8, torch.float32])
def test_noalloc(fov, dev, dtype):
    cases = [make(dev, 60 + i, dtype) for i in range(6)]
    want = [fov.forward(x, dict(p, sigma_map=m.view(-1)), layout="CHW") for x, m, _, _, p in cases]
    for streams in (1, 3):  # in order on one stream; on several, where calls wait for each other
        for _, m, out, inside, _ in cases:
            inside.copy_(m.view(-1))
        torch.cuda.synchronize()
        s = [torch.cuda.Stream() for _ in range(streams)]
        for i, (x, m, out, inside, p) in enumerate(cases):
            api.forward_noalloc(x, dict(p, sigma_map=inside), out, layout="CHW", stream=s[i % streams])
        torch.cuda.synchronize()
        for (_, _, out, _, _), y in zip(cases, want):
            assert torch.equal(out, y), streams


def test_noalloc_captured(fov, dev):
    x, m, out, inside, p = make(dev, 70, torch.float32)
    want = fov.forward(x, dict(p, sigma_map=m.view(-1)), layout="CHW")
    api.forward_noalloc(x, dict(p, sigma_map=m.view(-1)), out, layout="CHW")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        inside.copy_(m.view(-1))
        api.forward_noalloc(x, dict(p, sigma_map=inside), out, layout="CHW")
    for k in range(4):
        out.fill_(float(k))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), k
