"""A batch's diagnostics recorded into a graph and replayed after the batch was
rebuilt and after it was closed: every replay is the members' own diagnostics of
the lattices that were current at the recording."""
import numpy as np
import pytest

from paper_2312_10318_amd import inputs

pytestmark = pytest.mark.gpu


def test_recorded_batch_diagnostics_outlive_the_tables():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_10318_amd import capi
    from paper_2312_10318_amd.lattice import Batch, Lattice
    s = torch.cuda.Stream()
    lats = []
    for k, (nx, ny) in enumerate([(130, 64), (65, 33), (40, 20), (257, 51)]):
        f = inputs.random_populations(np.random.default_rng(k), (ny, nx))
        lats.append(Lattice(nx, ny, 0.8, 1.2, storage="f32", stream=s).set_populations(f))
    b = Batch(lats)
    b.step(1)
    want = np.array([list(m.diagnostics().values()) for m in lats])
    out = torch.zeros((4, capi.TRT_NDIAG), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        capi.trt_batch_diagnostics(b.handle, out.data_ptr())
    for then in (lambda: None, lambda: b.update(lats[::-1]), lambda: b.update(lats[:2]), b.close):
        then()
        with torch.cuda.stream(s):
            out.zero_()
            g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want)
