"""The resident kernels are under the same guards as the other kernels of the step
path: a build that spills fails, a profile finds them, its source hash covers them."""
import os

from paper_2312_10318_amd import build, profiling
from test_profiling_cpu import _fake_run

KERNEL = "void trt::(anonymous namespace)::resident_kernel<0, 1024>(trt::InstDesc, int, long)"


def test_a_spill_fails_the_build():
    text = "\n".join("a.hip:1:1: remark: " + t for t in (
        "Function Name: _ZN3trt12_GLOBAL__N_115resident_kernelILi0ELi1024EEEvNS_8InstDescEil",
        "    VGPRs Spill: 3", "Function Name: _ZN3trt12_GLOBAL__N_111macros_kernelILi0EEEv",
        "    VGPRs Spill: 2"))
    assert list(build.spilled_sweeps(text).values()) == [3]


def test_the_source_hash_covers_every_step_kernel():
    listed = {os.path.basename(p) for p in profiling.SWEEP_SOURCES}
    assert listed >= {s for s in build.SOURCES if s not in ("api.hip", "fields.hip")}


def test_a_profile_of_a_resident_run(tmp_path):
    """One dispatch takes all 100 steps of the run, warm-up and all."""
    alg = 144 * 32 * 32 * 100
    (t, f, w), log = _fake_run(str(tmp_path), [120000], [2000] * 3, [16.0], [32.0],
                               [(1 << 30) / 1024.0] * 3, [(1 << 30) / 1024.0] * 3, sweep=KERNEL)
    rec = profiling.summarize(t, f, w, "f64", 32, 90, 10, os.path.join(str(tmp_path), "s"),
                              run_log=log)
    assert rec["kernel"] == "resident_kernel<0, 1024>" and rec["dispatches"] == 1
    assert rec["updates_per_launch"] == 100 and rec["avg_duration_us"] == 120.0
    assert rec["algorithmic_bytes_per_launch"] == alg
    assert rec["hbm_bytes_per_launch"] == 48 * 1024
