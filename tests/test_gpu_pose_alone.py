"""The pose gradient alone of large batches, fused and as a backward of its own, on
either side of the rules between a team of lanes per ray and one lane: sparse and
mostly allocated maps, the SH degrees, the view-direction term.  Without statistics,
whose counters another kernel keeps.  Against the FP64 oracle, with the tolerances of
every other kernel."""
import dataclasses
import functools

import numpy as np
import pytest

from paper_2307_03404_amd import synth
from tests._parity import TAU_FWD, TAU_GRAD, assert_pose, assert_r28, reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=1)
def _room():
    return synth.config2()


def _workload(scene, n, deg, view):
    wl = _room() if scene == "room" else synth.config3()
    wl = synth.subset_rays(wl, n, seed=n) if n < wl.rays.n_rays else wl
    return wl.replace(grid=synth.with_sh_degree(wl.grid, deg),
                      opts=dataclasses.replace(wl.opts, flags=synth.FLAG_POSE_VIEWDIR if view else 0))


def _check(wl, fused, backward):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    wl, ref = reference(wl, want_grid=False)
    F = wl.rays.n_frames
    print(f"[gpu] pose alone: {wl.name}, {wl.rays.n_rays} rays, degree {wl.grid.sh_degree}, flags {wl.opts.flags}", flush=True)
    g, r = pxm.grid_to_device(wl.grid), pxm.rays_to_device(wl.rays)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()           # noqa: E731
    host = lambda t: t.cpu().numpy()                                                       # noqa: E731
    if fused:
        pose = torch.zeros(F, 6, dtype=torch.float64, device="cuda")
        loss = torch.zeros(F, dtype=torch.float64, device="cuda")
        rgb, depth = torch.empty(wl.rays.n_rays, 3, device="cuda"), torch.empty(wl.rays.n_rays, device="cuda")
        pxm.render_fused(g, r, wl.opts, dev(wl.targets.rgb), dev(wl.targets.depth), dev(wl.targets.frame_weight),
                         pxm.WANT_POSE, rgb=rgb, depth=depth, loss=loss, grad_pose=pose)
        assert_r28(host(rgb), ref["rgb"], TAU_FWD, "rgb")
        assert_r28(host(depth), ref["depth"], TAU_FWD, "depth")
        assert_r28(host(loss), ref["loss"], TAU_FWD, "loss")
        assert_pose(host(pose), ref["grad_pose"], TAU_GRAD, "fused pose")
    if backward:
        rgb, depth, ns = pxm.render_forward(g, r, wl.opts)
        pose = pxm.render_backward_pose(g, r, wl.opts, rgb, depth, ns, dev(ref["g_rgb"]), dev(ref["g_depth"]))
        assert_pose(host(pose), ref["grad_pose"], TAU_GRAD, "backward pose")


@pytest.mark.parametrize("scene,n,deg,view", [
    ("room", 150000, 2, True), ("room", 150001, 2, True), ("ball", 120000, 2, True), ("ball", 120001, 2, True),
    ("room", 250000, 0, False), ("room", 250001, 0, False), ("room", 250001, 1, False), ("room", 150001, 1, True),
    ("ball", 200001, 1, False), ("ball", 120001, 0, True),
    ("room", 400000, 2, False), ("room", 400001, 2, False)])
def test_fused(scene, n, deg, view):
    _check(_workload(scene, n, deg, view), True, False)


@pytest.mark.parametrize("scene,n,deg,view", [
    ("room", 220000, 2, False), ("room", 220001, 2, False), ("room", 220001, 2, True), ("ball", 220001, 2, False),
    ("ball", 220001, 1, True), ("room", 220001, 0, False), ("room", 220001, 1, False), ("ball", 220001, 0, True)])
def test_backward(scene, n, deg, view):
    _check(_workload(scene, n, deg, view), False, True)


def test_whole_frame():
    _check(_workload("room", 816000, 2, False), True, True)


# the widths' own limits: four lanes per ray up to 43,200 rays, sixteen up to 10,800
@pytest.mark.parametrize("n", [10800, 10801, 21600, 21601, 43200, 43201])
def test_widths(n):
    _check(_workload("ball", n, 2, n % 2 == 1), True, True)
