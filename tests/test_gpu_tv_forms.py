"""The two choices of the TV gradient's launch: scaled square roots for an eps
below the normal numbers, and 64-bit record offsets for maps of 4 GiB and more
(against the same map in a small array, bit for bit)."""
import dataclasses

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


@pytest.mark.parametrize("deg", [0, 1, 2])
@pytest.mark.parametrize("eps", [1e-39, 1.1754944e-38, 1e-9])
def test_eps_below_and_at_the_smallest_normal_number(deg, eps):
    # 17 x 9 x 12 vertices: blocks and cubes of blocks with remainders on every
    # axis; every neighbour difference is far from zero, so the sums stay normal
    # in both precisions and eps decides nothing but the form
    pxm = _pxm()
    rng = np.random.default_rng(3)
    R = (17, 9, 12)
    mask = rng.random(np.prod(R)) < 0.6
    grid = synth.grid_from_mask(R, (0.0, 0.0, 0.0), 0.1, mask, rng.uniform(0.5, 3.0, int(mask.sum())), rng)
    grid = synth.with_sh_degree(grid, deg)
    ref = oracle.tv(grid, 0.3, 0.2, float(np.float32(eps)))[1]
    g = pxm.grid_to_device(grid)
    print(f"[gpu] tv degree {deg} eps {eps}", flush=True)
    out = pxm.tv_grad_set(g, 0.3, 0.2, eps).cpu().numpy()
    assert_r28(out, ref, TAU_GRAD, "tv set")
    out = pxm.tv_grad(g, 0.3, 0.2, eps, torch.ones_like(g.data)).cpu().numpy()
    used = oracle.used_fields(deg)
    assert_r28(out[:, :used], ref[:, :used] + 1.0, TAU_GRAD, "tv add")
    assert np.all(out[:, used:] == 1.0)


def test_records_beyond_4_gib():
    pxm = _pxm()
    small = pxm.grid_to_device(synth.sphere_grid(1, 32)[0])
    n = small.n_alloc
    total = (1 << 32) // (4 * 28) + 1000                       # the last thousand records lie beyond 4 GiB
    print(f"[gpu] tv on {total} records", flush=True)
    data = torch.zeros(total, 28, device="cuda")
    data[total - n:] = small.data
    big = dataclasses.replace(small, link=torch.where(small.link >= 0, small.link + (total - n), -1).to(torch.int32),
                              data=data)
    ref = pxm.tv_grad_set(small, 0.3, 0.2, 1e-9)
    out = pxm.tv_grad_set(big, 0.3, 0.2, 1e-9)
    assert torch.equal(out[total - n:], ref)
    assert not bool(out[:total - n].any())
