"""Grid growth and the occupancy bitfield on lattices with short rows along z, whose
rows share a wave (2 to 64 vertices, and the lengths on either side of each number
of lanes a row gets), bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2307_03404_amd import synth
from tests.test_gpu_parity import _occupancy_numpy

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [(19, 7, 2), (9, 11, 3), (13, 6, 4), (21, 13, 5), (7, 21, 8), (33, 3, 9), (5, 13, 16), (6, 9, 17),
                               (7, 5, 32), (4, 6, 33), (3, 7, 64), (65, 66, 2), (2, 70, 12)])
@pytest.mark.parametrize("share", [0.03, 0.6])
def test_short_rows(R, share):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    rng = np.random.default_rng(sum(R))
    mask = rng.random(int(np.prod(R))) < share
    mask[[0, -1]] = True
    grid = synth.grid_from_mask(R, (0.0, 0.0, 0.0), 0.1, mask, rng.normal(size=int(mask.sum())).astype(np.float32), rng)
    print(f"[gpu] edit {R} share {share}: {grid.n_alloc} records", flush=True)
    g = pxm.grid_to_device(grid)
    np.testing.assert_array_equal(g.occ.cpu().numpy().view(np.uint32), _occupancy_numpy(grid))
    want = oracle.grid_upsample(grid)
    got = pxm.grid_upsample(g)
    np.testing.assert_array_equal(got.link.cpu().numpy(), want.link)
    np.testing.assert_array_equal(got.data.cpu().numpy(), want.data)
