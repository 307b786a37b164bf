"""Several time steps per launch with one column per lane (the default for
FP64 lattices, lattices with obstacles or open x boundaries, and FP32 and
FP16 lattices too small to fill the machine with 128-column windows): every
population of one step per launch, bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import rel_errors, say
from paper_2312_10318_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_10318_amd import lattice
    return lattice


def _problem(kind, nx, ny):
    """(mask, g, inflow) of a problem."""
    mask, g, inflow = None, (0.0, 0.0), None
    if kind == "walls":
        mask, g = inputs.channel_mask(nx, ny - 2), (1e-6, 2e-7)
    elif kind == "obstacle":
        mask, g = inputs.square_obstacle_mask(nx, ny, max(2, min(nx, ny) // 5)), (1e-6, 0.0)
    elif kind == "random":
        mask = (np.random.default_rng(5).random((ny, nx)) < 0.2).astype(np.uint8)
        g = (1e-6, -1e-6)
    elif kind in ("inflow", "cylinder"):
        inflow = (0.01, 1.0, 1.01)
        if kind == "cylinder":
            mask = inputs.square_obstacle_mask(nx, ny, max(2, min(nx, ny) // 10))
    return mask, g, inflow


# widths: narrower than a window, one and two windows of 58 or 54 columns
# and one column either side, the link summary's 64-column edges, odd ones;
# heights: the fewest rows, blocks with a remainder
SIZES = [(3, 350), (54, 19), (58, 18), (64, 40), (65, 33), (116, 70), (117, 16), (130, 64),
         (257, 51), (301, 90)]


@pytest.mark.parametrize("kind", ["open", "walls", "obstacle", "random", "inflow", "cylinder"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_equals_one_step_per_launch(L, kind, storage):
    for nx, ny in SIZES:
        mask, g, inflow = _problem(kind, nx, ny)
        out = []
        for sps in (1, 0):
            lat = L.Lattice(nx, ny, 0.8, 1.2, g=g, mask=mask, storage=storage, inflow=inflow)
            if sps:
                lat.set_tuning(steps_per_sweep=sps)
            assert lat.tuning()[5] == (sps or 2)
            lat.set_populations(inputs.random_populations(np.random.default_rng(nx), (ny, nx)))
            for n in (5, 4, 7):
                lat.step(n)
            out.append((lat.get_populations().cpu().numpy(), lat.state()[1]))
            lat.close()
        differ = int(np.sum(out[0][0] != out[1][0]))
        say("case: %s %s %dx%d: differs at %d entries" % (kind, storage, nx, ny, differ))
        assert out[0][1] == out[1][1] == 16 and differ == 0


@pytest.mark.parametrize("kind,storage,nx,ny,k", [
    ("open", "f32", 1300, 901, 3), ("obstacle", "f32", 1100, 600, 3), ("walls", "f32", 1300, 901, 3),
    ("cylinder", "f32", 1050, 700, 3), ("open", "f64", 700, 530, 2), ("cylinder", "f64", 900, 640, 3),
    ("walls", "f64", 1301, 901, 3), ("open", "f64", 2101, 1501, 3),
    ("obstacle", "f16", 1500, 1100, 2), ("open", "f16", 900, 800, 2), ("open", "f16", 1411, 1001, 2)])
def test_larger_lattices_equal_one_step_per_launch(L, kind, storage, nx, ny, k):
    """The sizes from which the rule takes more steps, longer blocks and
    wider workgroups; steps that are not a multiple of the launch's."""
    mask, g, inflow = _problem(kind, nx, ny)
    out = []
    for sps in (1, 0):
        lat = L.Lattice(nx, ny, 0.8, 1.2, g=g, mask=mask, storage=storage, inflow=inflow)
        if sps:
            lat.set_tuning(steps_per_sweep=sps)
        assert lat.tuning()[5] == (sps or k)
        lat.set_populations(inputs.random_populations(np.random.default_rng(nx), (ny, nx)))
        for n in (2, 3, 14):
            lat.step(n)
        out.append(lat.get_populations())
        lat.close()
    assert bool((out[0] == out[1]).all())


@pytest.mark.parametrize("storage,tol", [("f64", 1e-12), ("f32", 1e-5)])
def test_cylinder_against_the_oracle(L, storage, tol):
    """The oracle's run of the open cylinder, at each storage's tolerance."""
    nx, ny, steps, u = 150, 96, 60, 0.02
    mask = inputs.square_obstacle_mask(nx, ny, 12)
    rho, ux, uy = np.ones((ny, nx)), np.where(mask, 0.0, u), np.zeros((ny, nx))
    lat = L.Lattice(nx, ny, 0.8, 1.3, mask=mask, storage=storage, inflow=(u, 1.0, 1.0))
    assert lat.tuning()[5] == 2
    lat.init_equilibrium(rho, ux, uy).step(steps)
    _, gu, gv = (t.cpu().numpy() for t in lat.macros())
    lat.close()
    f = oracle.run_open(oracle.init_equilibrium(rho, ux, uy, mask), steps, 0.8, 1.3, u, 1.0, 1.0,
                        mask=mask)
    _, ou, ov = oracle.macros(f, mask=mask)
    emax, el2 = rel_errors(gu, gv, ou, ov)
    say("case: cylinder %s: rel max %.3e L2 %.3e" % (storage, emax, el2))
    assert emax <= tol and el2 <= tol


def test_a_set_shape_keeps_the_passes_it_describes(L):
    """Any launch-shape field that is set asks for the passes those fields
    describe; graph length alone does not."""
    for kw in (dict(rows_per_wave=8), dict(waves_per_block=2), dict(cols_per_lane=1),
               dict(steps_per_sweep=2), dict(steps_per_sweep=1), dict(prefetch_rows=1)):
        lat = L.Lattice(256, 64, 0.7, 1.0, storage="f64")
        assert lat.tuning()[5] == 2
        lat.set_tuning(**kw)
        assert lat.tuning()[5] == 1, kw
        lat.set_tuning(graph_steps=8)
        assert lat.tuning()[5] == 2 and lat.tuning()[4] == 8
        lat.close()
    # fewer rows than a block's fill
    lat = L.Lattice(256, 15, 0.7, 1.0, storage="f64")
    assert lat.tuning()[5] == 1
    lat.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("large", [False, True])
def test_batches_equal_one_step_batches(L, storage, large):
    """Members of every kind in one batch (with `large`, one big enough that
    the open FP32 and FP16 members keep the 128-column windows), over splits
    that leave single steps and pairs, with diagnostics in between and a
    membership change."""
    specs = [("open", 130, 64), ("cylinder", 117, 60), ("walls", 65, 33), ("obstacle", 140, 41),
             ("open", 257, 51), ("random", 61, 17), ("open", 200, 9)]
    if large:
        specs.append(("open", 1400, 1500))
    runs = []
    for sps in (1, 0):
        lats = []
        for kind, nx, ny in specs:
            mask, g, inflow = _problem(kind, nx, ny)
            lat = L.Lattice(nx, ny, 0.8, 1.2, g=g, mask=mask, storage=storage, inflow=inflow)
            lat.set_populations(inputs.random_populations(np.random.default_rng(nx), (ny, nx)))
            lats.append(lat)
        b = L.Batch(lats)
        b.set_tuning(steps_per_sweep=sps, graph_steps=4)
        k = 3 if storage == "f32" or (storage == "f64" and large) else 2
        assert b.tuning()[7] == (1 if sps else k)
        diags = []
        for n in (1, 2, 5, 6, 13):
            b.step(n)
            diags.append(b.diagnostics())
        b.update(lats[1:])
        b.step(4)
        diags.append(b.diagnostics())
        b.close()
        runs.append(([(m.get_populations().cpu().numpy(), m.state()[1]) for m in lats], diags))
        for m in lats:
            m.close()
    for k, ((a, ta), (c, tc)) in enumerate(zip(*(r[0] for r in runs))):
        say("case: member %d %s: time %d/%d, differs at %d" % (k, storage, ta, tc, int((a != c).sum())))
        assert ta == tc == (31 if k else 27) and np.array_equal(a, c)
    assert all(np.array_equal(a, c) for a, c in zip(*(r[1] for r in runs)))
