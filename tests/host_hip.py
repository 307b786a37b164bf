"""The library over the stand-in HIP runtime of host_hip.c, in a process of its
own (`in_process`): simulations, batches and the launches they would make."""
import ctypes
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
STORAGE = {"f64": 0, "f32": 1, "f16": 2}


def in_process(module: str, case: str, tmp: str) -> None:
    """Run `module.case()` in a new process with the stand-in built in `tmp`."""
    so = os.path.join(tmp, "libhost_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7",
                    os.path.join(HERE, "host_hip.c"), "-o", so], check=True)
    code = "import sys; sys.path[:0] = [%r, %r]; import host_hip; host_hip.start(%r); " \
           "import %s as m; m.%s()" % (HERE, ROOT, so, module, case)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def start(so: str) -> None:
    """Load the stand-in, then the library on it (without PyTorch, which would
    bring its own runtime)."""
    global hip, capi
    sys.modules["torch"] = None
    hip = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
    hip.host_kernel.restype = ctypes.c_char_p
    hip.host_word.restype = ctypes.c_uint64
    from paper_2312_10318_amd import capi as c
    capi = c
    assert capi.load() is not None


_next = 1 << 40


def sim(nx, ny, storage="f32", inflow=False):
    """A simulation whose lattices are addresses that nothing reads; returns
    (handle, address of its first lattice)."""
    global _next
    p = capi._prob(nx, ny, 0.7, 1.0, 0.0, 0.0, None, STORAGE[storage],
                   *((capi.TRT_X_INFLOW_OUTFLOW, 0.01, 1.0, 1.0) if inflow else ()))
    size = (capi.trt_lattice_bytes(p) + 255) // 256 * 256
    a, _next = _next, _next + 2 * size
    return capi.trt_create(p, a, a + size, 0), a


def launches():
    """[(kernel, first 8 bytes of its first argument, its second argument), ...]
    since `clear`."""
    return [(hip.host_kernel(i).decode(), hip.host_word(i), hip.host_second(i))
            for i in range(hip.host_launches())]


def clear():
    hip.host_clear()


def status(call):
    """The status that a failing call raises."""
    try:
        call()
    except capi.TrtError as e:
        return e.status
    return 0
