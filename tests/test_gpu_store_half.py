"""Populations enter an FP16 lattice rounded once, to nearest even, from FP64:
against numpy's conversion, bit for bit, at ties and beside them, in halves'
subnormal range and at random."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_10318_amd import lattice
    return lattice


W = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)


def _values(kind, n, rng):
    h = rng.integers(0, 0x3400, n).astype(np.uint16).view(np.float16).astype(np.float64)
    up = np.nextafter(h.astype(np.float16), np.float16(1)).astype(np.float64)
    sign = rng.choice([-1.0, 1.0], n)
    if kind == "tie":
        return sign * (h + up) / 2
    if kind == "beside":
        mid = (h + up) / 2
        return sign * (mid + rng.choice([-1.0, 1.0], n) * 2.0 ** -50)
    if kind == "tiny":
        return sign * rng.random(n) * 2.0 ** rng.integers(-40, -12, n)
    return sign * rng.random(n) * 0.1


@pytest.mark.parametrize("kind", ["tie", "beside", "tiny", "any"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 5), (64, 1), (70, 33)])
def test_populations_round_once(L, nx, ny, kind):
    rng = np.random.default_rng(nx * 100 + ny)
    lat = L.Lattice(nx, ny, 0.6, 0.7, storage="f16")
    w = W[:, None, None]
    f = w + _values(kind, 9 * nx * ny, rng).reshape(9, ny, nx)
    lat.set_populations(f)
    want = (f - w).astype(np.float16).astype(np.float64) + w
    assert np.array_equal(lat.get_populations().cpu().numpy(), want)
