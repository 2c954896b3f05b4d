"""The native ray batch of a mapping iteration where it counts in several launches
(more than 8,192 rays), against torch's indexing, bit for bit, and in a graph."""
import pytest

from paper_2307_03404_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _loop(n, counts):
    from paper_2307_03404_amd import pxm
    from paper_2307_03404_amd.batch import MappingLoop
    gen = torch.Generator(device="cuda").manual_seed(n)
    total, F = sum(counts), len(counts)
    off = torch.tensor([0] + list(counts), dtype=torch.int32).cumsum(0).to(torch.int32).cuda()
    pix = torch.randint(0, 640, (total, 2), dtype=torch.int32, device="cuda", generator=gen)
    rgb = torch.rand(total, 3, device="cuda", generator=gen)
    depth = torch.randn(total, device="cuda", generator=gen)
    depth[::7] = float("nan")
    depth[1::7] = float("inf")
    kf = pxm.DeviceRays(torch.zeros(F, 3, 4, device="cuda"), torch.ones(F, 4, device="cuda"), off, pix)
    return MappingLoop(pxm.grid_to_device(synth.sphere_grid(1, 8)[0]), kf, rgb, depth, synth.Opts(), n, 0.1, 0.1, seed=n)


def _same(a, b):
    for x, y in ((a[0], b[0]), (a[1].frame_offsets, b[1].frame_offsets), (a[1].pix, b[1].pix), (a[2], b[2]), (a[4], b[4])):
        assert x.dtype == y.dtype and torch.equal(x, y)
    assert torch.equal(a[3].isnan(), b[3].isnan()) and torch.equal(a[3].nan_to_num(), b[3].nan_to_num())


@pytest.mark.parametrize("n", [8191, 8192, 8193, 9216, 9217, 300_001])
@pytest.mark.parametrize("counts", [(70_000,), (0, 3, 0, 90_000, 1, 0)])
def test_against_torch_indexing(n, counts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    loop = _loop(n, counts)
    print(f"[gpu] gather {n} rays of {counts}", flush=True)
    got = loop.sample()
    _same(got, loop.sample(got[0]))                             # given indices go through torch


def test_without_a_valid_depth():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    loop = _loop(20_000, (500, 500))
    loop.tgt_depth.zero_()
    print("[gpu] gather without a valid depth", flush=True)
    assert loop.sample()[4].tolist() == [1.0, 1.0]


def test_replayed_in_a_graph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    loop = _loop(20_000, (30_000, 4_000))
    idx = torch.sort(torch.randint(0, 34_000, (20_000,), device="cuda")).values
    call = lambda: pxm.gather_rays(idx, loop.kf, loop.tgt_rgb, loop.tgt_depth)             # noqa: E731
    call()
    print("[gpu] gather in a graph", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    for k in range(3):
        idx.copy_(torch.sort(torch.randint(0, 34_000, (20_000,), device="cuda")).values)
        loop.tgt_depth.mul_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        _same((idx, *out), loop.sample(idx))


@pytest.mark.parametrize("which", ["tgt_rgb", "tgt_depth"])
def test_targets_under_autograd_keep_their_graph(which):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    loop = _loop(100, (300, 40))
    getattr(loop, which).requires_grad_(True)
    print(f"[gpu] a batch of {which} that requires a gradient", flush=True)
    idx, _, rgb, depth, _ = loop.sample()
    out = rgb if which == "tgt_rgb" else depth
    assert out.requires_grad
    out[torch.isfinite(out)].sum().backward()
    counts = torch.bincount(idx, minlength=340).float()
    got = getattr(loop, which).grad.reshape(340, -1)[:, 0]
    ok = torch.isfinite(getattr(loop, which).detach()).reshape(340, -1)[:, 0]
    assert torch.equal(got[ok], counts[ok])
