"""The launch shape a lattice reports, set again, keeps the passes it came from
and the bits; one field off asks for the passes that the fields describe."""
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


# resident, one row per block, several, odd, one of 1 mod 128, fewer than 16 rows
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("nx,ny", [(30, 34), (64, 40), (257, 130), (700, 301), (200, 12)])
def test_reported_shape_keeps_its_pass(L, nx, ny, walls, storage):
    mask = None
    if walls:
        mask = np.zeros((ny, nx), np.uint8)
        mask[ny // 2, : nx // 2] = 1
    f = inputs.random_populations(np.random.default_rng(nx + ny), (ny, nx))
    got = []
    for again in (False, True):
        lat = L.Lattice(nx, ny, 0.7, 1.1, mask=mask, storage=storage)
        auto = lat.tuning()
        if again:
            lat.set_tuning(*auto)
            assert lat.tuning() == auto
        lat.set_populations(f)
        lat.step(7)
        got.append(lat.get_populations().cpu().numpy())
    assert np.array_equal(got[0], got[1])
    if storage == "f64" and auto[5] > 1:
        off = list(auto)
        off[0] += 1
        lat.set_tuning(*off)
        assert lat.tuning()[5] == 1
