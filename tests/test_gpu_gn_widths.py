"""Gauss-Newton normal equations at every team width, with the view-direction term, on
rays of frames that share waves, and on rays whose lit windows overflow what a team
keeps.  Against the FP64 oracle, with the tolerances of every other kernel."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2307_03404_amd import synth
from tests._parity import TAU_GRAD, assert_r28

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(wl):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    print(f"[gpu] Gauss-Newton: {wl.name}, {wl.rays.n_rays} rays, degree {wl.grid.sh_degree}, flags {wl.opts.flags}", flush=True)
    g, r = pxm.grid_to_device(wl.grid), pxm.rays_to_device(wl.rays)
    tgt = [torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()
           for x in (wl.targets.rgb, wl.targets.depth, wl.targets.frame_weight)]
    H, grad, E = (x.cpu().numpy() for x in pxm.gn_unpack(pxm.render_gn(g, r, wl.opts, *tgt)))
    rH, rg, rE = oracle.gn_system(wl.grid, wl.rays, wl.targets, wl.opts)
    for a, b in ((slice(0, 3), slice(0, 3)), (slice(3, 6), slice(3, 6)), (slice(0, 3), slice(3, 6))):
        assert_r28(H[:, a, b], rH[:, a, b], TAU_GRAD, f"H {a} {b}")
    assert_r28(grad[:, :3], rg[:, :3], TAU_GRAD, "J^T W e rho")
    assert_r28(grad[:, 3:], rg[:, 3:], TAU_GRAD, "J^T W e phi")
    assert_r28(E, rE, TAU_GRAD, "E")


def _repeat(wl, n):
    """A workload of n rays: c3's, frame by frame, some of them more than once."""
    off = wl.rays.frame_offsets
    times = -(-n // wl.rays.n_rays)
    idx = np.sort(np.concatenate([np.arange(off[-1])] * times)[:n])
    new = np.searchsorted(idx, off).astype(np.int32)
    new[-1] = n
    rays = dataclasses.replace(wl.rays, pix=np.ascontiguousarray(wl.rays.pix[idx]), frame_offsets=new)
    tg = dataclasses.replace(wl.targets, rgb=wl.targets.rgb[idx], depth=wl.targets.depth[idx])
    return wl.replace(rays=rays, targets=tg)


# sixteen lanes per ray up to 21,200 rays, four up to 84,800, two up to 620,000, then one
@pytest.mark.parametrize("n,view", [(70, False), (21200, False), (21201, False), (84800, False), (84801, False), (620000, False),
                                    (620001, False), (70, True), (21201, True), (84801, True), (620001, True)])
def test_widths(n, view):
    wl = synth.config3()
    wl = synth.subset_rays(wl, n, seed=n) if n <= wl.rays.n_rays else _repeat(wl, n)
    _check(wl.replace(opts=dataclasses.replace(wl.opts, flags=synth.FLAG_POSE_VIEWDIR if view else 0)))


@pytest.mark.parametrize("deg", [0, 1])
@pytest.mark.parametrize("n", [3000, 50000, 150000])
def test_lower_degrees_with_the_view_term(deg, n):
    wl = synth.subset_rays(synth.config3(), n, seed=n)
    _check(wl.replace(grid=synth.with_sh_degree(wl.grid, deg), opts=dataclasses.replace(wl.opts, flags=synth.FLAG_POSE_VIEWDIR)))


# a thin fog in every cell and fine samples: some teams keep more windows than there is
# room for, others none (frames of rays that miss are among them)
@pytest.mark.parametrize("n,step", [(200, 0.02), (30000, 0.1), (90000, 0.1)])
def test_more_lit_windows_than_a_team_keeps(n, step):
    wl = synth.subset_rays(synth.config3(), n, seed=5)
    rng = np.random.default_rng(6)
    data = wl.grid.data.copy()
    data[:, 0] = rng.uniform(0.01, 0.2, size=data.shape[0])
    opts = dataclasses.replace(wl.opts, step_vox=synth.f32(step), max_samples=2 ** 31 - 1)
    _check(wl.replace(grid=dataclasses.replace(wl.grid, data=data), opts=opts))
