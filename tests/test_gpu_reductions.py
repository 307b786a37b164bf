"""The on-device reductions at the edges of their workgroups: one launch for
every member of a batch against each member's own call (bitwise), and the
sums against the same sums of the fields read back."""
import numpy as np
import pytest

from paper_2312_10318_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_10318_amd import lattice
    return lattice


# nodes: 1, one workgroup less one / exactly / plus one, several, the most
# workgroups (512 x 256 nodes) exactly and more than once round
SIZES = [(1, 1), (51, 5), (64, 4), (257, 1), (130, 70), (512, 256), (515, 301)]


def _lattice(L, nx, ny, storage, walls=False):
    mask = None
    if walls and ny > 4:
        mask = np.zeros((ny, nx), np.uint8)
        mask[0] = 1
        mask[2, : nx // 2] = 1
    lat = L.Lattice(nx, ny, 0.7, 1.1, g=(1e-6, 0.0) if walls else (0.0, 0.0), mask=mask,
                    storage=storage)
    rng = np.random.default_rng(nx * 1000 + ny)
    lat.set_populations(inputs.random_populations(rng, (ny, nx)))
    return lat


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("steps", [0, 1, 5, 6])
def test_batch_diagnostics_are_each_members_own(L, storage, steps):
    # members of both classes (several steps per launch, and one), which flip
    # their lattices at different rates
    lats = [_lattice(L, nx, ny, storage, walls=k % 2 == 1) for k, (nx, ny) in enumerate(SIZES)]
    lats[2].step(3)  # members that start at different times
    b = L.Batch(lats)
    b.step(steps)
    got = b.diagnostics()
    want = np.array([[lat.diagnostics()[k] for k in L.DIAG_NAMES] for lat in lats])
    b.close()
    assert np.array_equal(got, want)
    assert got[2, 7] == 3 + steps and got[0, 7] == steps
    assert np.array_equal(got[:, 5], [int(lat.ny * lat.nx if lat.mask is None else
                                          (lat.mask == 0).sum()) for lat in lats])


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("storage", ["f64", "f16"])
def test_sums_match_the_fields(L, size, storage):
    import torch
    nx, ny = size
    lat = _lattice(L, nx, ny, storage)
    lat.step(2)
    rho, ux, uy = (t.cpu().numpy() for t in lat.macros())
    d = lat.diagnostics()
    # a sum of n positive terms in FP64 is within n ulp of its terms' sum
    n = nx * ny
    tol = n * 2.0 ** -52
    assert abs(d["mass"] - rho.sum()) <= tol * rho.sum()
    assert abs(d["mom_x"] - (rho * ux).sum()) <= tol * np.abs(rho * ux).sum()
    assert abs(d["mom_y"] - (rho * uy).sum()) <= tol * np.abs(rho * uy).sum()
    assert d["max_speed"] == pytest.approx(np.hypot(ux, uy).max(), rel=1e-14)
    assert d["min_rho"] == rho.min() and d["n_fluid"] == n
    prev = tuple(torch.full((ny, nx), v, dtype=torch.float64, device=lat.device)
                 for v in (0.25, -0.125))
    mx, s2, n2, p2 = lat.velocity_change(prev)
    dx, dy = ux - 0.25, uy + 0.125
    assert mx == max(np.abs(dx).max(), np.abs(dy).max())
    assert abs(s2 - (dx * dx + dy * dy).sum()) <= 2 * tol * s2
    assert abs(n2 - (ux * ux + uy * uy).sum()) <= 2 * tol * n2
    assert p2 == n * (0.25 ** 2 + 0.125 ** 2)
    assert np.array_equal(prev[0].cpu().numpy(), ux) and np.array_equal(prev[1].cpu().numpy(), uy)
    lat.close()
