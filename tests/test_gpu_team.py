"""GPU parity of the kernels with a team of lanes per ray, at the batch sizes on
either side of each change of team width (the rule of team_lanes_log2: 64 lanes
up to 2,700 rays, 32 up to 5,400, then 16, 8, 4, 2 at sizes that differ between
the pose and the grid gradient), on rays of many frames so that a wave and a
workgroup hold rays of several; and on long rays whose lit samples overflow
the windows that the march keeps for the grid gradient.  Against the FP64
oracle, with the tolerances of every other kernel."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2307_03404_amd import synth
from tests._parity import TAU_FWD, TAU_GRAD, assert_pose, assert_r28, reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(wl, nsamp_off=1e-3):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    wl, ref = reference(wl)
    n, F = wl.rays.n_rays, wl.rays.n_frames
    print(f"[gpu] team: {wl.name}, {n} rays, {F} frames", flush=True)
    g, r = pxm.grid_to_device(wl.grid), pxm.rays_to_device(wl.rays)
    dev = lambda x, t=torch.float32: torch.from_numpy(np.ascontiguousarray(x)).to("cuda", t)  # noqa: E731
    tgt = [dev(x) for x in (wl.targets.rgb, wl.targets.depth, wl.targets.frame_weight)]
    host = lambda t: t.detach().cpu().numpy()                                              # noqa: E731

    rgb, depth, ns = pxm.render_forward(g, r, wl.opts)
    assert_r28(host(rgb), ref["rgb"], TAU_FWD, "rgb")
    assert_r28(host(depth), ref["depth"], TAU_FWD, "depth")
    assert np.mean(host(ns) != ref["nsamp"]) <= nsamp_off

    for want in (pxm.WANT_GRID, pxm.WANT_POSE, pxm.WANT_GRID | pxm.WANT_POSE):
        grad = torch.zeros_like(g.data)
        pose = torch.zeros(F, 6, dtype=torch.float64, device="cuda")
        loss = torch.zeros(F, dtype=torch.float64, device="cuda")
        out = pxm.render_fused(g, r, wl.opts, *tgt, want, rgb=torch.empty_like(rgb), depth=torch.empty_like(depth),
                               loss=loss, grad_data=grad, grad_pose=pose)
        assert_r28(host(out["rgb"]), ref["rgb"], TAU_FWD, f"want {want} rgb")
        assert_r28(host(loss), ref["loss"], TAU_FWD, f"want {want} loss")
        if want & pxm.WANT_GRID:
            assert_r28(host(grad), ref["grad_data"], TAU_GRAD, f"want {want} grad_data")
        if want & pxm.WANT_POSE:
            assert_pose(host(pose), ref["grad_pose"], TAU_GRAD, f"want {want} grad_pose")

    up = dev(ref["g_rgb"]), dev(ref["g_depth"])
    grad = pxm.render_backward_grid(g, r, wl.opts, rgb, depth, ns, *up)
    assert_r28(host(grad), ref["grad_data"], TAU_GRAD, "backward grad_data")
    pose = pxm.render_backward_pose(g, r, wl.opts, rgb, depth, ns, *up)
    assert_pose(host(pose), ref["grad_pose"], TAU_GRAD, "backward grad_pose")

    gn = pxm.render_gn(g, r, wl.opts, *tgt)
    H, grad6, E = (host(x) for x in pxm.gn_unpack(gn))
    rH, rg, rE = oracle.gn_system(wl.grid, wl.rays, wl.targets, wl.opts)
    for a, b in ((slice(0, 3), slice(0, 3)), (slice(3, 6), slice(3, 6)), (slice(0, 3), slice(3, 6))):
        assert_r28(H[:, a, b], rH[:, a, b], TAU_GRAD, f"H {a} {b}")
    assert_r28(grad6[:, :3], rg[:, :3], TAU_GRAD, "J^T W e rho")
    assert_r28(grad6[:, 3:], rg[:, 3:], TAU_GRAD, "J^T W e phi")
    assert_r28(E, rE, TAU_GRAD, "E")


# either side of the widths' limits; 1 and 65: a lone ray, a wave and a ray
@pytest.mark.parametrize("n", [1, 65, 2700, 2701, 5401, 10801, 21201, 42401, 84801])
def test_team_widths_on_many_frames(n):
    _check(synth.subset_rays(synth.config3(), n, seed=n))


@pytest.mark.parametrize("n", [40, 3000, 12000])
def test_more_lit_windows_than_are_kept(n):
    # a thin fog in every cell and samples a tenth of a voxel apart: hundreds of
    # lit samples on a ray, in more than six windows of any team
    wl = synth.subset_rays(synth.config3(), n, seed=5)
    rng = np.random.default_rng(6)
    data = wl.grid.data.copy()
    data[:, 0] = rng.uniform(0.01, 0.2, size=data.shape[0])
    opts = dataclasses.replace(wl.opts, step_vox=synth.f32(0.05 if n == 40 else 0.1), max_samples=2 ** 31 - 1)
    _check(wl.replace(grid=dataclasses.replace(wl.grid, data=data), opts=opts))


# the pose alone: two lanes per ray up to 400,000 rays; on a map that is mostly
# allocated (this one) one lane from 200,001 on
@pytest.mark.parametrize("n", [200000, 200001])
def test_pose_alone_of_many_rays_on_a_dense_map(n):
    _check(synth.subset_rays(synth.config3(), n, seed=n))
