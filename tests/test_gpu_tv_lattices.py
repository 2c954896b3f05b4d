"""The TV gradient on lattices whose blocks do not fill cubes (one block on an axis),
and on one with more blocks than a single launch holds, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2307_03404_amd import synth
from tests._parity import TAU_GRAD, assert_r28

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pxm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    return pxm


def _grid(R, rng, mask=None):
    mask = rng.random(int(np.prod(R))) < 0.4 if mask is None else mask
    return synth.grid_from_mask(R, (0.0, 0.0, 0.0), 0.1, mask, rng.normal(size=int(mask.sum())).astype(np.float32), rng)


@pytest.mark.parametrize("R", [(40, 9, 3), (3, 70, 5), (130, 4, 7), (17, 33, 2), (2, 2, 300), (9, 2, 2), (26, 140, 8)])
@pytest.mark.parametrize("occupancy", [True, False])
def test_flat_lattices(R, occupancy):
    pxm = _pxm()
    grid = _grid(R, np.random.default_rng(11))
    g = pxm.grid_to_device(grid, occupancy=occupancy)
    ref = oracle.tv(grid, 0.3, 0.2, 1e-9)[1]
    print(f"[gpu] tv {R}", flush=True)
    assert_r28(pxm.tv_grad_set(g, 0.3, 0.2, 1e-9).cpu().numpy(), ref, TAU_GRAD, "tv set")
    assert_r28(pxm.tv_grad(g, 0.3, 0.2, 1e-9).cpu().numpy(), ref, TAU_GRAD, "tv add")


def test_more_blocks_than_a_launch_holds():
    # 2 x 2 x 70 million vertices: 8.75 million blocks.  Allocated only in the
    # first 64 layers and the last, each also a small map of its own whose
    # layer towards the gap is empty.
    pxm = _pxm()
    Z, n = 70_000_000, 64
    rng = np.random.default_rng(12)
    lo = rng.random((2, 2, n + 1)) < 0.7
    lo[:, :, n] = False
    hi = rng.random((2, 2, n + 1)) < 0.7
    hi[:, :, 0] = False
    a, b = _grid((2, 2, n + 1), rng, lo.ravel()), _grid((2, 2, n + 1), rng, hi.ravel())
    link = torch.full((2, 2, Z), -1, dtype=torch.int32, device="cuda")
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()                        # noqa: E731
    la, lb = dev(a.link).reshape(2, 2, n + 1), dev(b.link).reshape(2, 2, n + 1)
    link[:, :, :n + 1] = la
    link[:, :, Z - n - 1:] = torch.where(lb >= 0, lb + a.n_alloc, -1)
    g = pxm.DeviceGrid((2, 2, Z), a.aabb_min, a.voxel_size, link.reshape(-1), torch.cat([dev(a.data), dev(b.data)]))
    ref = np.concatenate([oracle.tv(x, 0.3, 0.2, 1e-9)[1] for x in (a, b)])
    print(f"[gpu] tv on {4 * Z} vertices", flush=True)
    assert_r28(pxm.tv_grad_set(g, 0.3, 0.2, 1e-9).cpu().numpy(), ref, TAU_GRAD, "tv set")
