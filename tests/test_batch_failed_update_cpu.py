"""A membership change that fails for want of memory (for the device tables or for
their staging): the batch keeps its members, whose diagnostics are still their own
and as many as its caller has room for; it refuses to step until a rebuild succeeds,
no launch names a table that is missing or holds other members, and the simulations
that did not join are free."""
import pytest

import host_hip


def _check(fail):
    capi, hip = host_hip.capi, host_hip.hip
    small = [host_hip.sim(200, 100) for _ in range(2)]
    large = [host_hip.sim(1024, 1024) for _ in range(60)]   # outgrow the first tables
    b = capi.trt_batch_create([h for h, _ in small])
    capi.trt_batch_step(b, 1)
    hip.host_fail(*fail)
    assert host_hip.status(lambda: capi.trt_batch_update(b, [h for h, _ in large])) == \
        capi.TRT_EDEVICE
    hip.host_fail(0, 0)
    host_hip.clear()
    capi.trt_batch_diagnostics(b, 4096)
    got = [(w, s) for k, w, s in host_hip.launches() if "final" not in k]
    assert got == [(a, 1) for _, a in small]   # each from its own descriptor and lattice
    host_hip.clear()
    assert host_hip.status(lambda: capi.trt_batch_step(b, 3)) == capi.TRT_ESTATE
    assert host_hip.launches() == []
    assert host_hip.status(lambda: capi.trt_step(small[0][0], 1)) == capi.TRT_ESTATE
    capi.trt_step(large[0][0], 1)
    capi.trt_batch_update(b, [h for h, _ in large])
    capi.trt_batch_diagnostics(b, 4096)
    capi.trt_batch_step(b, 3)
    assert host_hip.launches() and all(w != 0 for _, w, _ in host_hip.launches())
    capi.trt_batch_destroy(b)


def device_tables(): _check((1, 0))


def staging(): _check((0, 1))


@pytest.mark.parametrize("case", ["device_tables", "staging"])
def test_failed_rebuild(case, tmp_path):
    host_hip.in_process("test_batch_failed_update_cpu", case, str(tmp_path))
