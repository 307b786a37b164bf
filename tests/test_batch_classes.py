"""One batch that holds members of every way to advance at once: 128-column windows
(FP32, FP16; in FP64 64-column windows without a link map), 64-column windows with
one, one workgroup a member, and one step per launch.  Its work list and descriptor
table hold them one after the other; the CPU test names the launches that a step
makes, the GPU test compares every population and every diagnostic with one step per
launch."""
import numpy as np
import pytest

import host_hip

STORAGES = ("f64", "f32", "f16")
LARGE = [("open", 2000, 2200), ("open", 1400, 1500), ("open", 2000, 1600)]
GENERAL = [("cylinder", 300, 200), ("obstacle", 257, 130), ("random", 140, 90)]
ONE_STEP = [("inflow", 200, 9), ("inflow", 65, 12)]
TINY = [("open", 20, 20), ("cylinder", 30, 18), ("inflow", 17, 40)]
TINY_COPIES = 11   # 33 of at most 1024 nodes: too many to ride in the others' launches


def _specs(storage):
    large = [("open", 700, 500), ("open", 301, 400)] if storage == "f64" else LARGE
    out = []   # interleaved, so that no class is a run of members
    for k in range(TINY_COPIES):
        out += TINY
        out += [spec for group in (large, GENERAL, ONE_STEP) for spec in group[k:k + 1]]
    return out


def launches():
    capi = host_hip.capi
    first = {"f64": "narrow_batch", "f32": "sweep_tb3_batch", "f16": "sweep_tb2_batch"}
    for storage in STORAGES:
        if storage != "f64":   # more 128-column windows than the 64-column rule takes
            assert sum(-(-nx // 120) * -(-ny // 8) for _, nx, ny in LARGE) >= 8192
        b = capi.trt_batch_create([host_hip.sim(nx, ny, storage, inflow=kind != "open")[0]
                                   for kind, nx, ny in _specs(storage)])
        k = 2 if storage == "f16" else 3
        host_hip.clear()
        capi.trt_batch_step(b, k)
        got = [name for name, _, _ in host_hip.launches()]
        want = ["resident_batch", first[storage], "narrow_batch"] + ["sweep_batch"] * k
        assert len(got) == len(want) and all(w in g for w, g in zip(want, got)), (storage, got)
        capi.trt_batch_destroy(b)


def test_a_step_makes_every_kind_of_launch(tmp_path):
    host_hip.in_process("test_batch_classes", "launches", str(tmp_path))


@pytest.mark.gpu
@pytest.mark.parametrize("storage", STORAGES)
def test_every_class_keeps_its_bits(storage):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_util import say
    from paper_2312_10318_amd.lattice import Batch, Lattice
    from test_gpu_narrow import _problem
    specs = _specs(storage)
    runs = []
    for steps_per_sweep in (1, 0):
        lats = []
        for j, (kind, nx, ny) in enumerate(specs):
            mask, g, inflow = _problem(kind, nx, ny)
            gen = torch.Generator(device="cuda").manual_seed(j)
            lat = Lattice(nx, ny, 0.8, 1.2, g=g, mask=mask, storage=storage, inflow=inflow)
            u = 0.01 * torch.randn((3, ny, nx), generator=gen, device="cuda", dtype=torch.float64)
            lats.append(lat.init_equilibrium(1.0 + u[0], u[1], u[2]))
        b = Batch(lats)
        b.set_tuning(steps_per_sweep=steps_per_sweep, graph_steps=4)
        diags = []
        for n in (1, 2, 5, 13):
            b.step(n)
            diags.append(b.diagnostics())
        b.update(lats[::-1])
        b.step(4)
        diags.append(b.diagnostics())
        b.close()
        runs.append(([m.get_populations() for m in lats], [m.state()[1] for m in lats], diags))
        for m in lats:
            m.close()
    for j, (a, c) in enumerate(zip(runs[0][0], runs[1][0])):
        say("case: member %d %s %s: differs at %d" % (j, specs[j], storage, int((a != c).sum())))
        assert torch.equal(a, c)
    assert runs[0][1] == runs[1][1] == [25] * len(specs)
    assert all(np.array_equal(a, c) for a, c in zip(runs[0][2], runs[1][2]))


@pytest.mark.gpu
@pytest.mark.parametrize("storage", STORAGES)
def test_members_that_ride_keep_their_bits(storage):
    """A few members of at most 1024 nodes beside larger ones, in 64-column and (FP16,
    FP32) 128-column launches."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_10318_amd import inputs
    from paper_2312_10318_amd.lattice import Batch, Lattice
    from test_gpu_narrow import _problem
    for large in ([("open", 150, 128)], [("open", 2000, 2200), ("open", 2001, 2000)]):
        out = []
        for steps_per_sweep in (1, 0):
            lats = []
            for kind, nx, ny in TINY[:1] + large + TINY[1:]:
                mask, g, inflow = _problem(kind, nx, ny)
                lat = Lattice(nx, ny, 0.8, 1.2, g=g, mask=mask, storage=storage, inflow=inflow)
                f = inputs.random_populations(np.random.default_rng(nx), (64, 64))
                f = np.tile(f, (1, -(-ny // 64), -(-nx // 64)))[:, :ny, :nx]
                lats.append(lat.set_populations(f))
            b = Batch(lats)
            b.set_tuning(steps_per_sweep=steps_per_sweep)
            for n in (3, 1, 8):
                b.step(n)
            out.append([m.get_populations() for m in lats])
            b.close()
            for m in lats:
                m.close()
        assert all(torch.equal(a, c) for a, c in zip(*out))
