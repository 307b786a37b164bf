"""Which launches a batch makes for members of at most 1024 nodes: their own where
they are alone or many, those of the other members where they are few."""
import host_hip

RESIDENT, NARROW, WIDE, ONE = ("resident_batch_kernel", "narrow_batch_kernel",
                               "sweep_tb2_batch_kernel", "sweep_batch_kernel")
TINY = [(32, 32)]


def routes():
    capi = host_hip.capi
    for storage, sizes, want in [
            ("f64", TINY * 3, [RESIDENT]),
            ("f64", TINY * 1 + [(128, 128)] * 4, [NARROW]),
            ("f64", TINY * 16 + [(128, 128)] * 4, [NARROW]),
            ("f64", TINY * 17 + [(128, 128)] * 4, [RESIDENT, NARROW]),
            ("f64", TINY * 2 + [(200, 9)], [RESIDENT, ONE, ONE]),   # others: one step a launch
            ("f16", TINY * 1 + [(1024, 1024)] * 4, [WIDE]),
            ("f16", TINY * 32 + [(1024, 1024)] * 4, [WIDE]),
            ("f16", TINY * 33 + [(1024, 1024)] * 4, [RESIDENT, WIDE]),
            ("f16", TINY * 1 + [(512, 512)] * 16, [RESIDENT, WIDE])]:  # five full rounds
        b = capi.trt_batch_create([host_hip.sim(nx, ny, storage)[0] for nx, ny in sizes])
        host_hip.clear()
        capi.trt_batch_step(b, 2)
        got = [k for k, _, _ in host_hip.launches()]
        assert len(got) == len(want) and all(w in g for w, g in zip(want, got)), (sizes, got)
        capi.trt_batch_destroy(b)


def test_small_members_ride_where_they_are_few(tmp_path):
    host_hip.in_process("test_batch_small_members_cpu", "routes", str(tmp_path))
