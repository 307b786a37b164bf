"""The launch shape that a batch reports, and the launches that a set one asks for."""
import host_hip

BATCHES = {
    "f64 two steps": ("f64", [(130, 100), (64, 33)], 0),
    "f64 three steps": ("f64", [(700, 800)], 0),
    "f64 open boundaries": ("f64", [(130, 100), (90, 70)], 2),
    "f64 one step": ("f64", [(130, 12)], 0),
    "f32 64 columns": ("f32", [(200, 100)] * 3, 1),
    "f32 64 columns, many": ("f32", [(500, 400)] * 9, 0),
    "f32 128 columns": ("f32", [(1500, 1500)] * 4, 0),
    "f16 64 columns": ("f16", [(130, 100)] * 4, 1),
    "f16 128 columns": ("f16", [(1500, 1500)] * 4, 0),
    "f16 both": ("f16", [(130, 100)] + [(1500, 1500)] * 4, 1),
    "resident": ("f64", [(32, 32), (4, 34)], 0),
    "resident and others": ("f32", [(32, 32)] * 40 + [(300, 300)], 0),
}
# rows ahead that its launches of several steps load
PREFETCH = {
    "f64 two steps": 2, "f64 three steps": 1, "f64 open boundaries": 2, "f64 one step": 0,
    "f32 64 columns": 2, "f32 64 columns, many": 1, "f32 128 columns": 1, "f16 64 columns": 2,
    "f16 128 columns": 1, "f16 both": 2, "resident": 0, "resident and others": 2,
}


def _batch(name):
    """The batch; its first `inflows` members have open boundaries."""
    storage, sizes, inflows = BATCHES[name]
    return host_hip.capi.trt_batch_create([host_hip.sim(nx, ny, storage, inflow=k < inflows)[0]
                                           for k, (nx, ny) in enumerate(sizes)])


def prefetch():
    for name, want in PREFETCH.items():
        assert host_hip.capi.trt_batch_get_tuning(_batch(name))[8] == want, name


def test_prefetch_of_every_kind_of_launch(tmp_path):
    host_hip.in_process("test_batch_tuning_cpu", "prefetch", str(tmp_path))


def _step(b, n=6):
    """The launches of n steps in one call, from its first lattices: kernels, grids."""
    host_hip.clear()
    host_hip.capi.trt_batch_step(b, n)
    return [(k, host_hip.hip.host_grid(i, 0)) for i, (k, _, _) in enumerate(host_hip.launches())]


def _new_passes(b):
    return any("narrow" in k or "resident" in k for k, _ in _step(b))


def requests():
    capi = host_hip.capi
    fields = (dict(rows_per_wave=8), dict(waves_per_block=2), dict(cols_per_lane=1),
              dict(steps_per_sweep=2), dict(steps_per_sweep=1), dict(prefetch_rows=1),
              dict(batch_items=16384))
    others = (dict(xcd_remap=1), dict(batch_order=2), dict(graph_steps=8), dict(batch_items=-1))
    for name in ("f64 two steps", "f64 three steps", "f64 open boundaries", "f32 64 columns",
                 "f16 64 columns", "resident", "resident and others"):
        assert _new_passes(_batch(name)), name
        for kw in fields + others:
            b = _batch(name)
            capi.trt_batch_set_tuning(b, **kw)
            assert _new_passes(b) == (kw in others), (name, kw)
            capi.trt_batch_set_tuning(b)
            assert _new_passes(b), (name, kw)


def test_a_set_field_asks_for_the_passes_it_describes(tmp_path):
    host_hip.in_process("test_batch_tuning_cpu", "requests", str(tmp_path))


def round_trip():
    capi = host_hip.capi
    for name in BATCHES:
        for kw in (dict(), dict(graph_steps=8), dict(batch_order=2), dict(xcd_remap=1)):
            a, b = _batch(name), _batch(name)
            capi.trt_batch_set_tuning(a, **kw)
            capi.trt_batch_set_tuning(b, **kw)
            shape = capi.trt_batch_get_tuning(b)
            capi.trt_batch_set_tuning(b, *shape)
            assert capi.trt_batch_get_tuning(b) == shape, (name, kw)
            assert _step(b, 7) == _step(a, 7), (name, kw)
            fresh = _batch(name)          # read from one batch, set on another
            capi.trt_batch_set_tuning(fresh, *shape)
            assert capi.trt_batch_get_tuning(fresh) == shape
        # the default's six leading fields, as the tuner names it
        b = _batch(name)
        capi.trt_batch_set_tuning(b, 0, 4, 0, 0, -1, 1)
        assert _step(b) == _step(_batch(name)), name
    # one field off: the passes that the fields describe
    b = _batch("f64 two steps")
    shape = list(capi.trt_batch_get_tuning(b))
    for field, value in ((1, 2), (7, 1), (8, 1)):
        off = list(shape)
        off[field] = value
        capi.trt_batch_set_tuning(b, *off)
        assert not _new_passes(b), (field, value)


def test_a_reported_shape_set_again_keeps_the_passes(tmp_path):
    host_hip.in_process("test_batch_tuning_cpu", "round_trip", str(tmp_path))
