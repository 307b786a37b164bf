"""Diagnostics of a batch recorded into a caller's graph: a replay may come after
a membership change or after the batch is gone, so the recorded launches name no
table of the batch, only each member's own descriptor and lattice."""
import host_hip


def recorded():
    capi, hip = host_hip.capi, host_hip.hip
    sims = [host_hip.sim(200, 100, s) for s in ("f64",) * 3]
    b = capi.trt_batch_create([h for h, _ in sims])
    capi.trt_batch_step(b, 1)
    hip.host_capturing(1)
    host_hip.clear()
    capi.trt_batch_diagnostics(b, 4096)
    hip.host_capturing(0)
    got = [(w, s) for k, w, s in host_hip.launches() if "final" not in k]
    assert got == [(a, 1) for _, a in sims]   # after one step: lattice 1
    host_hip.clear()
    capi.trt_batch_diagnostics(b, 4096)       # not recorded: two launches for all
    assert host_hip.hip.host_launches() == 2
    capi.trt_batch_destroy(b)


def test_recorded_diagnostics_hold_their_own_descriptors(tmp_path):
    host_hip.in_process("test_batch_capture_cpu", "recorded", str(tmp_path))
