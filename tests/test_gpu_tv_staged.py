"""The TV gradient's two forms (records read straight from memory, and staged in LDS
for large maps of SH degree 2 that allocate most of their lattice) on either side of the rule
between them, against plain FP64 torch on the GPU."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LAM = (0.3, 0.2, 1e-6)


def _reference(link, data, R, used):
    """dTV/d record in FP64 by autograd, a few fields at a time."""
    lam_d, lam_sh, eps = LAM
    link = link.reshape(R).long()
    has, out = link >= 0, torch.zeros_like(data)
    for m in range(used):
        v = data[:, m].double().requires_grad_(True)
        f = torch.where(has, v[link.clamp(min=0)], torch.zeros((), dtype=torch.float64, device="cuda"))
        c = f[:-1, :-1, :-1]
        d = (f[1:, :-1, :-1] - c) ** 2 + (f[:-1, 1:, :-1] - c) ** 2 + (f[:-1, :-1, 1:] - c) ** 2 + eps
        t = torch.where(has[:-1, :-1, :-1], d.sqrt(), torch.zeros_like(d)).sum()
        out[:, m] = ((lam_d if m == 0 else lam_sh) * torch.autograd.grad(t, v)[0]).float()
    return out


# records on either side of 192 MiB (1,797,558 of SH degree 2) and of half of the
# lattice, ragged lattices, and the lower degrees, which have one form
@pytest.mark.parametrize("deg,R,share", [
    (2, (121, 122, 121), 1.0), (2, (122, 122, 123), 1.0), (2, (150, 151, 155), 0.55), (2, (150, 151, 166), 0.49),
    (1, (147, 148, 147), 1.0), (0, (234, 233, 234), 1.0), (2, (5, 700, 531), 0.98)])
def test_both_forms(deg, R, share):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_03404_amd import pxm
    gen = torch.Generator(device="cuda").manual_seed(3)
    n = R[0] * R[1] * R[2]
    mask = torch.rand(n, device="cuda", generator=gen) < share
    link = torch.where(mask, torch.cumsum(mask, 0, dtype=torch.int32) - 1, -1).to(torch.int32)
    k, S, used = int(mask.sum()), pxm.record_floats(deg), {0: 4, 1: 13, 2: 28}[deg]
    data = torch.randn(k, S, device="cuda", generator=gen)
    g = pxm.DeviceGrid(R, (0.0, 0.0, 0.0), 0.1, link, data, sh_degree=deg).build_occupancy()
    print(f"[gpu] tv degree {deg} {R}: {4 * S * k / 2 ** 20:.1f} MiB of records", flush=True)
    ref = _reference(link, data, R, used)
    put = pxm.tv_grad_set(g, *LAM, torch.full_like(data, 0.25))
    add = pxm.tv_grad(g, *LAM, torch.full_like(data, 0.25))
    assert bool((put[:, used:] == 0.25).all()) and bool((add[:, used:] == 0.25).all())
    rms = ref[:, :used].double().pow(2).mean().sqrt()
    tol = 1e-4 * torch.maximum(ref[:, :used].abs().double(), rms)
    assert bool(((put[:, :used].double() - ref[:, :used].double()).abs() <= tol).all())
    assert bool(((add[:, :used].double() - 0.25 - ref[:, :used].double()).abs() <= tol).all())
