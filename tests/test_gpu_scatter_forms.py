"""GPU parity of the grid gradient where the rays of a wave lie apart, so that
its lanes work at sample indices of their own, and where the gradient array is
larger than 32-bit byte offsets reach.  Against the FP64 oracle, with the
tolerances of every other kernel."""
import dataclasses

import numpy as np
import pytest

from paper_2307_03404_amd import synth
from tests._parity import TAU_FWD, TAU_GRAD, assert_pose, assert_r28, reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _scattered(n, seed, mixed):
    """n rays of config3's frames in random order within each frame; mixed:
    only every other run of 64 rays is, so both kinds of wave occur."""
    wl = synth.subset_rays(synth.config3(), n, seed=seed)
    off = wl.rays.frame_offsets
    rng = np.random.default_rng(seed)
    order = np.arange(n)
    for lo, hi in zip(off[:-1], off[1:]):
        p = lo + rng.permutation(hi - lo)
        keep = (np.arange(lo, hi) // 64) % 2 == 0 if mixed else np.zeros(hi - lo, bool)
        order[lo:hi] = np.where(keep, np.arange(lo, hi), 0)
        rest = p[~np.isin(p, order[lo:hi][keep])]
        order[lo:hi][~keep] = rest
    assert np.array_equal(np.sort(order), np.arange(n))
    rays = dataclasses.replace(wl.rays, pix=np.ascontiguousarray(wl.rays.pix[order]))
    tgt = dataclasses.replace(wl.targets, rgb=np.ascontiguousarray(wl.targets.rgb[order]),
                              depth=np.ascontiguousarray(wl.targets.depth[order]))
    return wl.replace(rays=rays, targets=tgt)


def _check(wl, shift=0, variants=(0, 1, 2)):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    wl, ref = reference(wl)
    print(f"[gpu] scatter: {wl.name}, {wl.rays.n_rays} rays, record shift {shift}", flush=True)
    g, r = pxm.grid_to_device(wl.grid), pxm.rays_to_device(wl.rays)
    n0 = g.data.shape[0]
    if shift:                                   # the same grid, its records behind `shift` unused ones
        g.link[g.link >= 0] += shift
        g.data = torch.cat([torch.zeros(shift, g.data.shape[1], device="cuda"), g.data])
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda", torch.float32)   # noqa: E731
    host = lambda t: t.detach().cpu().numpy()                                              # noqa: E731
    tgt = [dev(x) for x in (wl.targets.rgb, wl.targets.depth, wl.targets.frame_weight)]
    rgb, depth, ns = pxm.render_forward(g, r, wl.opts)
    assert_r28(host(rgb), ref["rgb"], TAU_FWD, "rgb")
    grad = torch.zeros_like(g.data)

    def matches(what):
        assert_r28(host(grad[shift:]), ref["grad_data"], TAU_GRAD, what)
        assert shift == 0 or not bool(grad[:shift].any()), what
        grad.zero_()

    try:
        for v in variants:
            pxm.set_tuning(256, v)
            pose = torch.zeros(wl.rays.n_frames, 6, dtype=torch.float64, device="cuda")
            pxm.render_fused(g, r, wl.opts, *tgt, pxm.WANT_GRID | pxm.WANT_POSE, grad_data=grad, grad_pose=pose)
            matches(f"variant {v} grad_data")
            assert_pose(host(pose), ref["grad_pose"], TAU_GRAD, f"variant {v} grad_pose")
    finally:
        pxm.set_tuning(256, 0)
    pxm.render_backward_grid(g, r, wl.opts, rgb, depth, ns, dev(ref["g_rgb"]), dev(ref["g_depth"]), grad_data=grad)
    matches("backward grad_data")
    assert n0 + shift == grad.shape[0]


# variants 1 and 2 keep a wave to one ray per lane at every size
@pytest.mark.parametrize("n", [63, 64, 1000, 20000])
@pytest.mark.parametrize("mixed", [False, True])
def test_rays_apart(n, mixed):
    _check(_scattered(n, n, mixed))


# one ray per lane in the backward alone as well
def test_many_rays_apart():
    _check(_scattered(180000, 3, True), variants=(0,))


# 112-byte records: 2^32 bytes end within record 38,347,922
def test_gradient_beyond_32_bit_offsets():
    _check(_scattered(3000, 7, True), shift=38_400_000)
