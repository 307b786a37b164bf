"""FP16 lattices and batches that both kinds of windows can take, at sizes where
the 128-column launches fill their rounds of wavefronts and where they do not: the
kernel that the rule launches (host logic alone), and on the GPU the bits of one
step per launch on either side."""
import numpy as np
import pytest

import host_hip

WIDE = [(1300, 1300), (1600, 1600), (1052, 1750), (2738, 942), (1601, 1601), (1107, 2359)]
NARROW = [(1250, 1250), (1450, 1450), (1014, 1378), (1561, 1561), (1299, 1300), (300, 300)]
WIDE_BATCH = [(9, 500, 500), (5, 700, 700), (24, 300, 300), (13, 500, 500)]
NARROW_BATCH = [(7, 500, 500), (10, 500, 500), (9, 501, 500), (4, 700, 700), (28, 300, 300)]


def _names(step):
    host_hip.clear()
    step()
    return [k for k, _, _ in host_hip.launches()]


def routes():
    capi = host_hip.capi
    for kernel, sizes in (("sweep_tb2_kernel", WIDE), ("narrow_kernel", NARROW)):
        for nx, ny in sizes:
            h, _ = host_hip.sim(nx, ny, "f16")
            got = _names(lambda: capi.trt_step(h, 2))
            assert len(got) == 1 and kernel in got[0], (nx, ny, got)
    for kernel, batches in (("sweep_tb2_batch_kernel", WIDE_BATCH),
                            ("narrow_batch_kernel", NARROW_BATCH)):
        for n, nx, ny in batches:
            b = capi.trt_batch_create([host_hip.sim(nx, ny, "f16")[0] for _ in range(n)])
            got = _names(lambda: capi.trt_batch_step(b, 2))
            assert len(got) == 1 and kernel in got[0], (n, nx, ny, got)
            capi.trt_batch_destroy(b)


def test_the_launch_that_fills_its_rounds(tmp_path):
    host_hip.in_process("test_f16_rounds", "routes", str(tmp_path))


@pytest.mark.gpu
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("nx,ny", [(1300, 1300), (1600, 1600), (1250, 1250), (1601, 1600), (1561, 1561)])
def test_either_side_keeps_the_bits(nx, ny, walls):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_10318_amd import inputs
    from paper_2312_10318_amd.lattice import Lattice
    mask = inputs.channel_mask(nx, ny - 2) if walls else None
    f = inputs.random_populations(np.random.default_rng(nx + ny), (ny, nx))
    out = []
    for steps_per_sweep in (1, 0):
        lat = Lattice(nx, ny, 0.8, 1.2, mask=mask, storage="f16")
        if steps_per_sweep:
            lat.set_tuning(steps_per_sweep=1)
        lat.set_populations(f)
        lat.step(7)
        out.append(lat.get_populations())
        lat.close()
    assert torch.equal(*out)
