"""The launches that a call without statistics takes at the default tuning, where the
other tests' helper asks for statistics or another variant: the forms of the team
kernel (view-direction term, SH degrees, loss alone), the one-lane kernels on whole
frames of a sparse map and at the lower degrees, with and without the bitfield, and
work masks that overflow.  Against the FP64 oracle, with the tolerances of every other
kernel."""
import dataclasses
import functools

import numpy as np
import pytest

import oracle
from paper_2307_03404_amd import synth
from tests._parity import TAU_FWD, TAU_GRAD, assert_pose, assert_r28, r28_ratio, reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pxm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    return pxm


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()


def _host(t):
    return t.detach().cpu().numpy()


def _fused(wl, ref, want, occupancy=True, stats=False, tuning=(256, 0)):
    pxm = _pxm()
    n, F = wl.rays.n_rays, wl.rays.n_frames
    what = f"{wl.name}, {n} rays, degree {wl.grid.sh_degree}, flags {wl.opts.flags}, want {want}, occupancy {occupancy}, tuning {tuning}"
    print(f"[gpu] default launch: {what}", flush=True)
    g, r = pxm.grid_to_device(wl.grid, occupancy=occupancy), pxm.rays_to_device(wl.rays)
    rgb, depth = torch.empty(n, 3, device="cuda"), torch.empty(n, device="cuda")
    loss = torch.zeros(F, dtype=torch.float64, device="cuda")
    grad = torch.zeros_like(g.data) if want & pxm.WANT_GRID else None
    pose = torch.zeros(F, 6, dtype=torch.float64, device="cuda") if want & pxm.WANT_POSE else None
    counts = torch.zeros(4, dtype=torch.int64, device="cuda") if stats else None
    old = pxm.get_tuning()
    pxm.set_tuning(*tuning)
    try:
        pxm.render_fused(g, r, wl.opts, _dev(wl.targets.rgb), _dev(wl.targets.depth), _dev(wl.targets.frame_weight),
                         want | (pxm.WANT_STATS if stats else 0), rgb=rgb, depth=depth, loss=loss, grad_data=grad,
                         grad_pose=pose, stats=counts)
    finally:
        pxm.set_tuning(*old)
    assert_r28(_host(rgb), ref["rgb"], TAU_FWD, what + " rgb")
    assert_r28(_host(depth), ref["depth"], TAU_FWD, what + " depth")
    assert_r28(_host(loss), ref["loss"], TAU_FWD, what + " loss")
    if grad is not None:
        used = oracle.used_fields(wl.grid.sh_degree)
        assert np.all(_host(grad)[:, used:] == 0)
        assert_r28(_host(grad)[:, 0], ref["grad_data"][:, 0], TAU_GRAD, what + " grad density")
        assert_r28(_host(grad)[:, 1:used], ref["grad_data"][:, 1:used], TAU_GRAD, what + " grad sh")
    if pose is not None:
        assert_pose(_host(pose), ref["grad_pose"], TAU_GRAD, what + " pose")


@functools.lru_cache(maxsize=1)
def _room():
    return synth.config2()


# 70 to 150,000 rays: sixty-four to two lanes per ray
@pytest.mark.parametrize("deg", [0, 1, 2])
@pytest.mark.parametrize("n", [70, 3000, 9000, 30000, 150000])
def test_teams_with_the_view_term(n, deg):
    wl = synth.subset_rays(synth.config3(), n, seed=n)
    wl = wl.replace(grid=synth.with_sh_degree(wl.grid, deg), opts=dataclasses.replace(wl.opts, flags=synth.FLAG_POSE_VIEWDIR))
    wl, ref = reference(wl)
    plain = oracle.fused(wl.grid, wl.rays, wl.targets, dataclasses.replace(wl.opts, flags=0), want_grid=False)
    if deg:                             # a constant basis has no direction
        assert r28_ratio(plain["grad_pose"][:, 3:], ref["grad_pose"][:, 3:]) > 10 * TAU_GRAD
    _fused(wl, ref, 2)
    _fused(wl, ref, 3)


# the limits of the forward's and the loss's teams, and of the grid gradient's, that
# test_gpu_team.py does not have; degree and map in turn
@pytest.mark.parametrize("n,deg", [(5300, 0), (5301, 1), (10600, 2), (10601, 0), (42400, 1), (169600, 2), (169601, 0)])
def test_loss_alone_and_grid_alone(n, deg):
    wl = synth.subset_rays(_room() if n % 2 else synth.config3(), n, seed=n)
    wl, ref = reference(wl.replace(grid=synth.with_sh_degree(wl.grid, deg)))
    _fused(wl, ref, 0)
    _fused(wl, ref, 1)
    pxm = _pxm()
    rgb, depth, ns = pxm.render_forward(pxm.grid_to_device(wl.grid), pxm.rays_to_device(wl.rays), wl.opts)
    assert_r28(_host(rgb), ref["rgb"], TAU_FWD, "forward rgb")
    assert_r28(_host(depth), ref["depth"], TAU_FWD, "forward depth")
    assert np.mean(_host(ns) != ref["nsamp"]) <= 1e-3


@functools.lru_cache(maxsize=1)
def _room_frame():
    return reference(_room())


@pytest.mark.parametrize("want", [1, 3])
@pytest.mark.parametrize("occupancy", [True, False])
def test_whole_frame_of_the_room(want, occupancy):
    wl, ref = _room_frame()
    _fused(wl, ref, want, occupancy)


@pytest.mark.parametrize("deg", [0, 1, 2])
@pytest.mark.parametrize("occupancy", [True, False])
def test_one_lane_forward_and_backward(deg, occupancy):
    pxm = _pxm()
    wl = synth.subset_rays(_room(), 175_000, seed=deg)
    wl, ref = reference(wl.replace(grid=synth.with_sh_degree(wl.grid, deg)))
    print(f"[gpu] one lane per ray: {wl.name}, degree {deg}, occupancy {occupancy}", flush=True)
    g, r = pxm.grid_to_device(wl.grid, occupancy=occupancy), pxm.rays_to_device(wl.rays)
    rgb, depth, ns = pxm.render_forward(g, r, wl.opts)
    assert_r28(_host(rgb), ref["rgb"], TAU_FWD, "rgb")
    assert_r28(_host(depth), ref["depth"], TAU_FWD, "depth")
    assert np.mean(_host(ns) != ref["nsamp"]) <= 1e-3
    grad = _host(pxm.render_backward_grid(g, r, wl.opts, rgb, depth, ns, _dev(ref["g_rgb"]), _dev(ref["g_depth"])))
    used = oracle.used_fields(deg)
    assert np.all(grad[:, used:] == 0)
    assert_r28(grad[:, 0], ref["grad_data"][:, 0], TAU_GRAD, "grad density")
    assert_r28(grad[:, 1:used], ref["grad_data"][:, 1:used], TAU_GRAD, "grad sh")


def _long_rays(dense):
    """Rays down a nearly transparent column of 600 voxels (more than 1024 lit samples) and
    across it; `dense`: the map allocates its whole lattice, else less than half of it."""
    rng = np.random.default_rng(66)
    R = (6, 6 if dense else 13, 600)
    mask = np.zeros(R, bool)
    mask[:, :6] = True
    grid = synth.grid_from_mask(R, (0.0, 0.0, 0.0), 0.01, mask.ravel(), rng.uniform(0.001, 0.003, int(mask.sum())), rng)
    along, across = np.zeros((3, 4)), np.zeros((3, 4))
    along[:, :3], along[:, 3] = np.eye(3), [0.025, 0.025, -0.3]
    across[:, :3], across[:, 3] = np.array([[0, 0, 1], [0, 1, 0], [-1, 0, 0]], float).T, [0.3, 0.025, 3.0]
    intr = np.array([[2000.0, 2000.0, 8.0, 8.0], [40.0, 40.0, 8.0, 8.0]], np.float32)
    u, v = np.meshgrid(np.arange(4, 12), np.arange(4, 12))
    pix = np.stack([u.ravel(), v.ravel()], 1).astype(np.int32)
    rays = synth.Rays(np.stack([along, across]).astype(np.float32), intr, np.array([0, 64, 128], np.int32),
                      np.concatenate([pix, pix]))
    opts = synth.Opts(step_vox=0.5, depth_loss=synth.DEPTH_L2)
    rgb, depth, nsamp, _ = oracle.render(grid, rays, opts)
    assert nsamp[:64].max() > 1100
    tg = synth.Targets((rgb + 0.05).astype(np.float32), (depth * 1.01).astype(np.float32),
                       synth.frame_weights(depth * 1.01, rays.frame_offsets, True))
    return reference(synth.Workload("long", grid, rays, tg, opts))


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("occupancy", [True, False])
def test_work_masks_that_overflow(dense, occupancy):
    """The pose alone marches lane by lane: past the end of its mask a lane searches
    again, in the persistent and two-launch forms and in the plain one that keeps
    statistics; a call without goes to a team, which has no mask."""
    wl, ref = _long_rays(dense)
    for want in (2, 3):
        for tuning in ((64, 1), (256, 1), (64, 2), (256, 0)):
            _fused(wl, ref, want, occupancy, False, tuning)
        _fused(wl, ref, want, occupancy, True)
