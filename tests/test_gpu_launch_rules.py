"""Either side of the rules that choose steps and rows per launch: the bits of
one step per launch, and the steps the rules are meant to give."""
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


def _lattice(L, nx, ny, storage, walls, seed=0):
    mask = None
    if walls:
        mask = np.zeros((ny, nx), np.uint8)
        mask[ny // 3: ny // 3 + 9, nx // 4: nx // 4 + 7] = 1
    lat = L.Lattice(nx, ny, 0.7, 1.1, mask=mask, storage=storage)
    lat.set_populations(inputs.random_populations(np.random.default_rng(nx + ny + seed), (ny, nx)))
    return lat


@pytest.mark.parametrize("nx,ny,storage,walls,steps", [
    (256, 256, "f32", False, 2), (257, 256, "f32", False, 3),   # 65536 nodes and more
    (1024, 512, "f32", True, 2), (1024, 513, "f32", True, 3),   # 524288 with a mask
    (57, 1025, "f32", True, 2), (116, 1025, "f32", True, 2),    # one row per block, two
    (58, 2048, "f16", True, 2), (59, 2049, "f16", True, 2),
    (700, 700, "f16", False, 2), (900, 901, "f64", False, 3),   # rows by rounds
    (900, 901, "f64", True, 3), (1300, 2017, "f64", False, 3),  # 2621440 nodes
    (1301, 2017, "f64", False, 3),
])
def test_steps_per_launch_keep_the_bits(L, nx, ny, storage, walls, steps):
    import torch
    a = _lattice(L, nx, ny, storage, walls)
    assert a.tuning()[5] == steps
    b = _lattice(L, nx, ny, storage, walls)
    b.set_tuning(steps_per_sweep=1)
    for lat in (a, b):
        lat.step(7)
    assert torch.equal(a.get_populations(), b.get_populations())


# FP32 batches of fewer and of more than 4096 windows, of members that 64-column
# windows cover with a twentieth fewer lanes, and FP16 ones
@pytest.mark.parametrize("storage,side,count", [
    ("f32", 400, 20), ("f32", 400, 21), ("f32", 160, 110), ("f32", 410, 45), ("f16", 400, 21)])
def test_batch_members_keep_their_bits(L, storage, side, count):
    import torch
    lats = [_lattice(L, side, side + k % 3, storage, False, seed=k % 4) for k in range(count)]
    batch = L.Batch(lats)
    batch.step(7)
    for k in (0, 1, count - 1):
        alone = _lattice(L, side, side + k % 3, storage, False, seed=k % 4)
        alone.set_tuning(steps_per_sweep=1)
        alone.step(7)
        assert torch.equal(lats[k].get_populations(), alone.get_populations())
    batch.close()
