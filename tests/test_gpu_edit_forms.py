"""Grid growth and the occupancy bitfield at the edges of their waves' work (runs of
60 cells, segments of 64 and steps of 256 and 512 vertices along z, odd
lattices), bit for bit against the oracle; and growth of a map whose records
span 4 GiB against the same map in a small array."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2307_03404_amd import synth
from tests.test_gpu_parity import _occupancy_numpy

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pxm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    return pxm


def _grid(R, share, seed, signed=True):
    rng = np.random.default_rng(seed)
    mask = rng.random(int(np.prod(R))) < share
    mask[[0, -1]] = True                                       # both ends of the lattice
    sig = rng.normal(size=int(mask.sum())) if signed else rng.uniform(0.1, 2.0, int(mask.sum()))
    return synth.grid_from_mask(R, (0.0, 0.0, 0.0), 0.1, mask, sig.astype(np.float32), rng)


@pytest.mark.parametrize("R", [(2, 2, 2), (3, 2, 61), (2, 5, 62), (6, 3, 64), (3, 6, 65), (5, 2, 122), (2, 3, 129),
                               (3, 2, 257), (2, 2, 513)])
@pytest.mark.parametrize("share", [0.02, 0.5])
def test_lattices_at_the_edges(R, share):
    pxm = _pxm()
    grid = _grid(R, share, 7)
    grid.data[::3, 1] = -0.0                                   # signed zeros, as an empty corner beside them reads +0
    print(f"[gpu] edit {R} share {share}: {grid.n_alloc} records", flush=True)
    g = pxm.grid_to_device(grid)
    np.testing.assert_array_equal(g.occ.cpu().numpy().view(np.uint32), _occupancy_numpy(grid))
    want = oracle.grid_upsample(grid)
    got = pxm.grid_upsample(g)
    np.testing.assert_array_equal(got.link.cpu().numpy(), want.link)
    np.testing.assert_array_equal(got.data.cpu().numpy(), want.data)


def test_growth_of_records_beyond_4_gib():
    pxm = _pxm()
    small = pxm.grid_to_device(_grid((20, 17, 70), 0.3, 9))
    n = small.n_alloc
    total = (1 << 32) // (4 * 28) + 1000
    print(f"[gpu] growth from {total} records", flush=True)
    data = torch.zeros(total, 28, device="cuda")
    data[total - n:] = small.data
    big = dataclasses.replace(small, link=torch.where(small.link >= 0, small.link + (total - n), -1).to(torch.int32),
                              data=data)
    a, b = pxm.grid_upsample(small), pxm.grid_upsample(big)
    assert torch.equal(a.link, b.link) and torch.equal(a.data, b.data) and torch.equal(a.occ, b.occ)
