"""Lattices of at most 1024 nodes, whose steps of a call take one launch:
every population of one step per launch, bit for bit, alone and in a batch."""
import numpy as np
import pytest

from gpu_util import say
from paper_2312_10318_amd import inputs
from test_gpu_narrow import _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_10318_amd import lattice
    return lattice


# nodes at the edges of the workgroup sizes (128, 256, 512, 1024 threads) and
# just past the largest; one column, odd widths
SIZES = [(1, 16), (4, 34), (8, 16), (16, 16), (3, 43), (16, 17), (31, 16), (32, 16), (27, 19),
         (32, 32), (51, 20), (60, 17), (41, 25)]


def _lattice(L, kind, nx, ny, storage):
    mask, g, inflow = _problem(kind, nx, ny)
    lat = L.Lattice(nx, ny, 0.8, 1.2, g=g, mask=mask, storage=storage, inflow=inflow)
    lat.set_populations(inputs.random_populations(np.random.default_rng(nx + ny), (ny, nx)))
    return lat


@pytest.mark.parametrize("kind", ["open", "walls", "obstacle", "random", "cylinder"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_equals_one_step_per_launch(L, kind, storage):
    for nx, ny in SIZES:
        if nx < 2 and kind == "cylinder":
            continue
        out = []
        for sps in (1, 0):
            lat = _lattice(L, kind, nx, ny, storage)
            if sps:
                lat.set_tuning(steps_per_sweep=sps)
            # a shape set on the way changes the pass, not the state
            for n in (1, 4, 7):
                lat.prepare(n)
                lat.step(n)
            if not sps:
                lat.set_tuning(steps_per_sweep=1)
            lat.step(3)
            lat.set_tuning(steps_per_sweep=sps)
            lat.step(6)
            force = lat.wall_force() if lat.mask is not None else 0
            out.append((lat.get_populations().cpu().numpy(), lat.state()[1], force,
                        lat.diagnostics()))
            lat.close()
        differ = int(np.sum(out[0][0] != out[1][0]))
        say("case: %s %s %dx%d: differs at %d entries" % (kind, storage, nx, ny, differ))
        assert out[0][1:] == out[1][1:] and out[0][1] == 21 and differ == 0


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("others", [[], [("open", 70, 40), ("cylinder", 66, 30)]])
def test_batches_equal_one_step_batches(L, storage, others):
    """Resident members alone, and among members that are not."""
    specs = [("walls", 4, 34), ("open", 32, 32), ("cylinder", 40, 20), ("obstacle", 17, 50)] + others
    runs = []
    for sps in (1, 0):
        lats = [_lattice(L, k, nx, ny, storage) for k, nx, ny in specs]
        b = L.Batch(lats)
        b.set_tuning(steps_per_sweep=sps)
        diags = []
        for n in (1, 6, 2, 9):
            b.step(n)
            diags.append(b.diagnostics())
        b.update(lats[::-1])
        b.step(5)
        diags.append(b.diagnostics())
        b.close()
        runs.append(([(m.get_populations().cpu().numpy(), m.state()[1]) for m in lats], diags))
        for m in lats:
            m.close()
    for (a, ta), (c, tc) in zip(*(r[0] for r in runs)):
        assert ta == tc == 23 and np.array_equal(a, c)
    assert all(np.array_equal(a, c) for a, c in zip(*(r[1] for r in runs)))


def test_a_call_longer_than_one_launch(L):
    """8192 steps go in one launch; a longer call is cut."""
    out = []
    for splits in ((8192 + 100,), (8192 - 8, 108)):
        lat = _lattice(L, "walls", 4, 20, "f32")
        for n in splits:
            lat.step(n)
        assert lat.state()[1] == 8292
        out.append(lat.get_populations())
        lat.close()
    assert bool((out[0] == out[1]).all())
