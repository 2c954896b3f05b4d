"""Maps that allocate their whole lattice and are lit in part or throughout, where a march
reads a sample's density before its colours only until the samples around it have
light: forward, fused and both backward passes, in teams and with one lane per ray,
against the FP64 oracle, with the tolerances of every other kernel."""
import dataclasses

import numpy as np
import pytest

from paper_2307_03404_amd import synth
from tests._parity import TAU_FWD, TAU_GRAD, assert_pose, assert_r28, reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _workload(n, lit, deg):
    wl = synth.subset_rays(synth.config3(), n, seed=n)
    rng = np.random.default_rng(8)
    data = wl.grid.data.copy()
    m = data.shape[0]
    if lit == "fog":                    # every sample
        data[:, 0] = rng.uniform(0.01, 0.2, size=m)
    elif lit == "half":                 # a fog in one half of the lattice, nothing in the other
        x = np.arange(m) // (32 * 32)
        data[:, 0] = np.where(x < 16, rng.uniform(0.01, 0.2, size=m), 0.0)
    else:                               # lit and dark vertices in turn, negative densities among them
        data[:, 0] = np.where(rng.random(m) < 0.5, rng.uniform(0.05, 0.4, size=m), rng.uniform(-0.3, 0.0, size=m))
    return wl.replace(grid=synth.with_sh_degree(dataclasses.replace(wl.grid, data=data), deg))


@pytest.mark.parametrize("lit", ["fog", "half", "mixed"])
@pytest.mark.parametrize("n,deg", [(64, 2), (5000, 2), (5000, 0), (60000, 1), (230000, 2), (230000, 0)])
def test_partly_lit(n, lit, deg):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    wl, ref = reference(_workload(n, lit, deg))
    print(f"[gpu] {lit} map, degree {deg}, {n} rays", flush=True)
    g, r = pxm.grid_to_device(wl.grid), pxm.rays_to_device(wl.rays)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()           # noqa: E731
    host = lambda t: t.cpu().numpy()                                                       # noqa: E731
    tgt = [dev(x) for x in (wl.targets.rgb, wl.targets.depth, wl.targets.frame_weight)]
    rgb, depth, ns = pxm.render_forward(g, r, wl.opts)
    assert_r28(host(rgb), ref["rgb"], TAU_FWD, "rgb")
    assert_r28(host(depth), ref["depth"], TAU_FWD, "depth")
    assert np.mean(host(ns) != ref["nsamp"]) <= 1e-3
    for variant in (0, 1) if n == 60000 else (0,):
        old = pxm.get_tuning()
        pxm.set_tuning(256, variant)
        try:
            for want in (pxm.WANT_POSE, pxm.WANT_GRID | pxm.WANT_POSE):
                grad, pose = torch.zeros_like(g.data), torch.zeros(wl.rays.n_frames, 6, dtype=torch.float64, device="cuda")
                pxm.render_fused(g, r, wl.opts, *tgt, want, grad_data=grad, grad_pose=pose)
                assert_pose(host(pose), ref["grad_pose"], TAU_GRAD, f"want {want} variant {variant} pose")
                if want & pxm.WANT_GRID:
                    assert_r28(host(grad), ref["grad_data"], TAU_GRAD, f"variant {variant} grad_data")
        finally:
            pxm.set_tuning(*old)
    up = dev(ref["g_rgb"]), dev(ref["g_depth"])
    assert_r28(host(pxm.render_backward_grid(g, r, wl.opts, rgb, depth, ns, *up)), ref["grad_data"], TAU_GRAD, "backward grid")
    assert_pose(host(pxm.render_backward_pose(g, r, wl.opts, rgb, depth, ns, *up)), ref["grad_pose"], TAU_GRAD, "backward pose")
