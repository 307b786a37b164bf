"""A membership change sends the batch's tables to the device in one copy, whatever
passes its members take and whether or not the tables grow."""
import host_hip


def changes():
    capi, hip = host_hip.capi, host_hip.hip
    tiny = [host_hip.sim(8, 34, "f32")[0] for _ in range(3)]
    small = [host_hip.sim(200, 100, "f32")[0] for _ in range(5)]
    opened = [host_hip.sim(150, 120, "f32", inflow=True)[0] for _ in range(2)]
    large = [host_hip.sim(1500, 1200, "f32")[0] for _ in range(8)]
    b = capi.trt_batch_create(tiny)
    for members in (tiny[:1], small, tiny + small + opened, large + tiny, large + opened, small):
        host_hip.clear()
        capi.trt_batch_update(b, members)
        assert hip.host_copies() == 1
    capi.trt_batch_destroy(b)


def test_one_copy_per_change(tmp_path):
    host_hip.in_process("test_batch_update_cpu", "changes", str(tmp_path))
