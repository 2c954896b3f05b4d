"""The native ray batch of a mapping iteration against torch's indexing, bit for
bit: repeats, empty frames, batch sizes around a workgroup, invalid depths."""
import pytest

from paper_2307_03404_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 63, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("counts", [(700,), (0, 3, 0, 900, 1, 0)])
def test_against_torch_indexing(n, counts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
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
    grid = pxm.grid_to_device(synth.sphere_grid(1, 8)[0])
    loop = MappingLoop(grid, kf, rgb, depth, synth.Opts(), n, 0.1, 0.1, seed=n)
    print(f"[gpu] gather {n} rays of {counts}", flush=True)
    idx, rays, c, d, w = loop.sample()
    ref_idx, ref, ref_c, ref_d, ref_w = loop.sample(idx)        # given indices go through torch
    for a, b in ((idx, ref_idx), (rays.frame_offsets, ref.frame_offsets), (rays.pix, ref.pix), (c, ref_c), (w, ref_w)):
        assert a.dtype == b.dtype and torch.equal(a, b)
    assert torch.equal(d.isnan(), ref_d.isnan()) and torch.equal(d.nan_to_num(), ref_d.nan_to_num())


def test_indices_outside_the_keyframes_stay_inside():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    pix = torch.arange(20, dtype=torch.int32, device="cuda").reshape(10, 2)
    kf = pxm.DeviceRays(torch.zeros(1, 3, 4, device="cuda"), torch.ones(1, 4, device="cuda"),
                        torch.tensor([0, 10], dtype=torch.int32, device="cuda"), pix)
    idx = torch.tensor([-5, 0, 9, 400], device="cuda")
    rays, _, depth, w = pxm.gather_rays(idx, kf, torch.rand(10, 3, device="cuda"), torch.ones(10, device="cuda"))
    assert rays.pix.tolist() == [[0, 1], [0, 1], [18, 19], [18, 19]]
    assert rays.frame_offsets.tolist() == [0, 4] and w.tolist() == [0.25]
