"""Boundary checks that need no GPU: the library loads, exports every symbol the
header declares, sizes its workspace, and rejects bad arguments before any launch."""
import ctypes as C
import os
import re

import pytest

import paper_2505_05086_amd as asi
from paper_2505_05086_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = C.c_void_p(0x1000)          # non-null, 256-aligned, never dereferenced by validation


def _declared():
    names = set()
    for fn in os.listdir(os.path.join(ROOT, "include")):
        if fn.endswith(".h"):
            src = open(os.path.join(ROOT, "include", fn)).read()
            src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
            names |= set(re.findall(r"\b(asi_[a-z0-9_]+)\s*\(", src))
    return names


def test_library_exports_every_declared_symbol():
    L = asi.lib()
    declared = _declared()
    assert {"asi_compress", "asi_core_project", "asi_weight_grad_conv2d", "asi_weight_grad_linear",
            "asi_workspace_bytes", "asi_status_string", "asi_version"} <= declared
    for name in declared:
        assert hasattr(L, name), name
    assert set(B.EXPORTS) == declared
    assert asi.asi_version() >= 1000
    assert asi.asi_status_string(0) == "ASI_OK" and asi.asi_status_string(3) == "ASI_ERR_WORKSPACE"


def test_workspace_query():
    d = asi.make_desc((64, 512, 7, 7), (16, 48, 5, 5))
    base = asi.asi_workspace_bytes(d)
    assert base > 0 and base % 256 == 0
    assert asi.asi_workspace_bytes(d, asi.make_conv(512, 3, 3, pad=(1, 1))) >= base
    assert asi.asi_workspace_bytes(asi.make_desc((64, 512, 7, 7), (16, 48, 5, 8))) == 0      # rank > dim
    assert asi.asi_workspace_bytes(asi.make_desc((64, 512), (16, 48))) == 0                  # ndim
    assert asi.asi_workspace_bytes(d, asi.make_conv(512, 3, 3, groups=3)) == 0               # groups
    assert asi.asi_workspace_bytes(d, None, 100) == 0                                        # linear needs 3 modes
    d3 = asi.make_desc((4, 5, 6), (2, 3, 4), "bf16")
    assert asi.asi_workspace_bytes(d3, None, 7) > 0
    # a wide mode (rank above 64) with many Gram slices: the plan includes the tree level's buffer
    wide = asi.asi_workspace_bytes(asi.make_desc((64, 197, 3072), (32, 64, 192), "bf16"), None, 768)
    assert wide > 0 and wide % 256 == 0
    # a rank above the number of columns of its unfolding (90 > 4 * 20) cannot be reached
    assert asi.asi_workspace_bytes(asi.make_desc((4, 20, 2100), (3, 8, 90)), None, 12) == 0


def test_planning_a_very_long_mode_takes_no_time():
    """The plan of a call is made anew on every call: its host time must not grow with a mode's length."""
    import time
    best = {}
    for n in (1 << 12, 1 << 30):
        d = asi.make_desc((4, 4, n), (2, 2, 8))
        times = []
        for _ in range(5):
            t = time.perf_counter()
            assert asi.asi_workspace_bytes(d) > 0
            times.append(time.perf_counter() - t)
        best[n] = min(times)
    assert best[1 << 30] <= 10 * best[1 << 12] + 1e-4, best


def test_layers_that_just_fit_the_static_scratch():
    # long modes of rank 64 in few columns: what grows with the 16-row Gram slices must not push them over the limit
    for dims, ranks in (((3, 214, 3423), (1, 64, 64)), ((3, 299, 2618), (2, 64, 64)), ((6, 94, 3614), (1, 58, 64))):
        assert 0 < asi.asi_workspace_bytes(asi.make_desc(dims, ranks)) <= B.STATIC_SCRATCH_BYTES, dims


def _arr(n=4):
    a = (C.c_void_p * 4)()
    for i in range(n):
        a[i] = 0x1000
    return a


def test_compress_rejects_bad_arguments_without_launching():
    L = asi.lib()
    good = asi.make_desc((8, 6, 5, 4), (2, 3, 2, 2))
    need = asi.asi_workspace_bytes(good)
    call = lambda d, A, up, uo, ws, n: L.asi_compress(C.byref(d), A, up, uo, ws, n, None, None)
    assert call(asi.make_desc((8, 6, 5, 4), (2, 3, 2, 5)), FAKE, _arr(), _arr(), FAKE, need) == 1
    assert call(asi.make_desc((8, 6, 5, 4), (0, 3, 2, 2)), FAKE, _arr(), _arr(), FAKE, need) == 1
    assert call(asi.make_desc((8, 0, 5, 4), (2, 3, 2, 2)), FAKE, _arr(), _arr(), FAKE, need) == 1
    assert call(asi.make_desc((8, 6, 5, 4), (2, 3, 2, 2), 7), FAKE, _arr(), _arr(), FAKE, need) == 2
    assert call(good, None, _arr(), _arr(), FAKE, need) == 1
    assert call(good, FAKE, _arr(3), _arr(), FAKE, need) == 1
    assert call(good, FAKE, _arr(), _arr(), FAKE, need - 1) == 3
    assert call(good, FAKE, _arr(), _arr(), None, need) == 3
    assert call(good, FAKE, _arr(), _arr(), C.c_void_p(0x1010), need) == 3               # misaligned
    # rank may not exceed the other side of the unfolding either (Alg. 1's range)
    assert call(asi.make_desc((8, 1, 1, 1), (2, 1, 1, 1)), FAKE, _arr(), _arr(), FAKE, 1 << 20) == 1


def test_cold_start_rejects_bad_arguments_without_launching():
    L = asi.lib()
    good = asi.make_desc((8, 6, 5, 4), (2, 3, 2, 2))
    need = asi.asi_workspace_bytes(good)
    call = lambda d, A, uo, ws, n: L.asi_compress_cold(C.byref(d), A, C.c_uint64(7), uo, ws, n, None, None)
    assert call(asi.make_desc((8, 6, 5, 4), (2, 3, 2, 5)), FAKE, _arr(), FAKE, need) == 1
    assert call(asi.make_desc((8, 6, 5, 4), (2, 3, 2, 2), 7), FAKE, _arr(), FAKE, need) == 2
    assert call(good, None, _arr(), FAKE, need) == 1
    assert call(good, FAKE, _arr(3), FAKE, need) == 1
    assert call(good, FAKE, None, FAKE, need) == 1
    assert call(good, FAKE, _arr(), FAKE, 255) == 3
    assert call(good, FAKE, _arr(), None, need) == 3
    assert L.asi_cold_start_matrix(C.byref(good), 4, C.c_uint64(7), FAKE, None) == 1
    assert L.asi_cold_start_matrix(C.byref(good), -1, C.c_uint64(7), FAKE, None) == 1
    assert L.asi_cold_start_matrix(C.byref(good), 0, C.c_uint64(7), None, None) == 1


def test_compress_static_rejects_before_touching_the_device():
    """The entry point that allocates nothing checks descriptor and size limit on the host first."""
    L = asi.lib()
    call = lambda d: L.asi_compress_static(C.byref(d), FAKE, _arr(), _arr(), None, None)
    assert call(asi.make_desc((8, 6, 5, 4), (2, 3, 2, 5))) == 1                      # rank > dim
    assert call(asi.make_desc((8, 6, 5, 4), (2, 3, 2, 2), 7)) == 2                   # dtype
    big = asi.make_desc((64, 197, 3072), (32, 64, 192), "bf16")
    assert asi.asi_workspace_bytes(big) > B.STATIC_SCRATCH_BYTES
    assert call(big) == 3                                                            # beyond the static array
    src = open(os.path.join(ROOT, "include", "asi.h")).read()
    assert re.search(r"#define\s+ASI_STATIC_SCRATCH_BYTES\s+\(16u\s*<<\s*20\)", src)
    assert B.STATIC_SCRATCH_BYTES == 16 << 20


def test_other_entry_points_reject_bad_arguments():
    L = asi.lib()
    d4 = asi.make_desc((8, 6, 5, 4), (2, 3, 2, 2))
    d3 = asi.make_desc((8, 6, 5), (2, 3, 2))
    big = 1 << 24
    assert L.asi_core_project(C.byref(d4), FAKE, _arr(), None, FAKE, big, None) == 1
    assert L.asi_core_project(C.byref(d4), FAKE, _arr(), FAKE, FAKE, 0, None) == 3
    cv = asi.make_conv(6, 3, 3, pad=(1, 1))
    assert L.asi_weight_grad_conv2d(C.byref(d3), FAKE, _arr(), FAKE, C.byref(cv), FAKE, 0, FAKE, big, None) == 1
    assert L.asi_weight_grad_conv2d(C.byref(d4), FAKE, _arr(), FAKE, None, FAKE, 0, FAKE, big, None) == 1
    bad = asi.make_conv(6, 9, 9)            # kernel larger than the padded map
    assert L.asi_weight_grad_conv2d(C.byref(d4), FAKE, _arr(), FAKE, C.byref(bad), FAKE, 0, FAKE, big, None) == 1
    bad = asi.make_conv(6, 3, 3, stride=(0, 1))
    assert L.asi_weight_grad_conv2d(C.byref(d4), FAKE, _arr(), FAKE, C.byref(bad), FAKE, 0, FAKE, big, None) == 1
    assert L.asi_weight_grad_conv2d(C.byref(d4), FAKE, _arr(), FAKE, C.byref(cv), FAKE, 0, FAKE, 16, None) == 3
    assert L.asi_weight_grad_linear(C.byref(d4), FAKE, _arr(), FAKE, 7, FAKE, 0, FAKE, big, None) == 1
    assert L.asi_weight_grad_linear(C.byref(d3), FAKE, _arr(), FAKE, 0, FAKE, 0, FAKE, big, None) == 1
    assert L.asi_weight_grad_linear(C.byref(d3), FAKE, _arr(), FAKE, 7, FAKE, 0, FAKE, 16, None) == 3


def test_binding_refuses_host_tensors():
    import torch
    d = asi.make_desc((8, 6, 5, 4), (2, 3, 2, 2))
    x = torch.zeros(8, 6, 5, 4)
    with pytest.raises(ValueError):
        asi.asi_core_project(d, x, [x] * 4, x, x)


def test_batched_entry_points_reject_bad_arguments():
    L = asi.lib()
    good = asi.make_desc((8, 6, 5, 4), (2, 3, 2, 2))
    bad = asi.make_desc((8, 6, 5, 4), (2, 3, 2, 5))
    need = asi.asi_workspace_bytes(good)

    def descs(*ds):
        arr = (B.TensorDesc * len(ds))()
        for i, d in enumerate(ds):
            arr[i] = d
        return arr

    def ptrs(n, v=0x1000):
        arr = (C.c_void_p * n)()
        for i in range(n):
            arr[i] = v
        return arr

    def modes(n):
        inner = [_arr() for _ in range(n)]
        outer = (C.c_void_p * n)()
        for i, a in enumerate(inner):
            outer[i] = C.addressof(a)
        return outer, inner

    def sizes(*vals):
        arr = (C.c_size_t * len(vals))()
        for i, v in enumerate(vals):
            arr[i] = v
        return arr

    up, k1 = modes(2)
    uo, k2 = modes(2)
    call = lambda n, ds, sz: L.asi_compress_batch(n, ds, ptrs(2), up, uo, ptrs(2), sz, None, None)
    assert call(0, descs(good, good), sizes(need, need)) == 2                 # count out of range
    assert call(9, descs(good, good), sizes(need, need)) == 2
    assert call(2, descs(good, bad), sizes(need, need)) == 1                  # second layer rejected: nothing runs
    assert call(2, descs(good, good), sizes(need, need - 1)) == 3
    assert L.asi_compress_batch(2, None, ptrs(2), up, uo, ptrs(2), sizes(need, need), None, None) == 1
    assert L.asi_core_project_batch(2, descs(good, good), ptrs(2), up, ptrs(2, 0), ptrs(2), sizes(need, need), None) == 1
    cv = (B.Conv2dDesc * 2)()
    cv[0] = asi.make_conv(6, 3, 3, pad=(1, 1))
    cv[1] = asi.make_conv(6, 9, 9)
    big = 1 << 24
    assert L.asi_weight_grad_conv2d_batch(2, descs(good, good), ptrs(2), up, ptrs(2), cv, ptrs(2), None, ptrs(2),
                                          sizes(big, big), None) == 1
    d3 = asi.make_desc((8, 6, 5), (2, 3, 2))
    dout = (C.c_int64 * 2)(7, 0)
    assert L.asi_weight_grad_linear_batch(2, descs(d3, d3), ptrs(2), up, ptrs(2), dout, ptrs(2), None, ptrs(2),
                                          sizes(big, big), None) == 1


def test_autograd_layers_refuse_to_run_without_the_gpu_path():
    """The training-loop wrappers have no CPU fallback: a CPU activation in training mode is an error."""
    import torch
    from paper_2505_05086_amd.autograd import AsiConv2d, AsiLinear
    conv = AsiConv2d(3, 4, 3, padding=1, ranks=(2, 2, 2, 2)).train()
    with pytest.raises(RuntimeError):
        conv(torch.zeros(2, 3, 5, 5))
    lin = AsiLinear(6, 4, ranks=(2, 2, 2)).train()
    with pytest.raises(RuntimeError):
        lin(torch.zeros(2, 3, 6))
    with pytest.raises(ValueError):
        lin(torch.zeros(3, 6))
    assert conv.eval()(torch.zeros(2, 3, 5, 5)).shape == (2, 4, 5, 5)      # inference is the plain operator


def test_bench_refuses_more_than_one_gpu():
    """This build runs on exactly one GPU: bench.py says so and exits before it touches a device."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert res.returncode == 2
    assert "one GPU" in res.stderr and res.stdout.strip() == ""


def test_bench_line_is_short_enough_to_be_kept_whole():
    """The line leaves out the figures of single launches (60 KB of them came to nothing where a log keeps the last 8000 characters)."""
    import importlib.util
    import json
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    spec = importlib.util.spec_from_file_location("bench", os.path.join(root, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    x = 1234.56789012345
    whole = {k: x for k in ("algorithmic_bytes_per_step", "hbm_us_at_peak", "hbm_frac", "flop_frac", "counter_traffic_over_algorithmic", "other")}
    roof = dict({k: x for k in ("achieved", "peak", "frac", "avg_launch_us", "launches_per_step", "kernel_time_share", "traffic", "more")},
                kernel="k_subspace_planes<float, 4, true>", bound="mfma", unit="TFLOP/s", whole_step=whole)
    passes = {f"compress|k_some_kernel<{i}, true>:P": {str(j): x for j in range(11)} for i in range(40)}
    phases = {p: {"us_per_step": x, "launches_per_step": x} for p in ("compress", "core", "weight_grad")}
    cpu = {"seconds_per_step": x, "variants": {f"variant {i}": {str(j): x for j in range(6)} for i in range(3)}}
    config = {"workload": "a workload of two layers " * 6, **{f"key {i}": x for i in range(9)}, "queue_probe": {str(i): x for i in range(12)}}
    one = dict(value=x, ms_per_step=x, host_enqueue_ms_per_step=x, dtype="bf16", roofline=roof, phases_eager_single_stream=phases)
    out = dict({k: "some text" for k in ("metric", "unit", "scaling", "data")}, **one, n_gpus=1, steps=20, warmup=5, higher_is_better=True,
               vs_baseline=None, config=config, cpu_baseline=cpu, kernel_breakdown=passes, gpu_ms_per_step_events=x,
               per_config=[dict(one, config=i, workload="w" * 150, passes=passes, cpu_baseline=cpu) for i in range(1, 7)])
    assert len(json.dumps(out)) > 60000
    line = bench.headline(out)
    text = json.dumps(line, separators=(",", ":"))
    assert len(text) <= bench.LINE_MAX < 8000 and "\n" not in text
    assert line["value"] == 1234.6 and len(line["per_config"]) == 6 and line["cpu_baseline"] and "kernel_breakdown" not in line
    out["per_config"] *= 8                               # a longer list goes rather than the line
    assert len(json.dumps(bench.headline(out), separators=(",", ":"))) <= bench.LINE_MAX


LDS_PROBE = r"""
#include "asi_lds.h"
#include <cstdio>
static int dev = 0, calls = 0, fail = 0;
extern "C" hipError_t hipGetDevice(int* d) { *d = dev; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int bytes) {
    ++calls;
    return fail || bytes != 90000 ? hipErrorInvalidValue : hipSuccess;
}
int main() {
    static asi::LdsAllowed allowed, other;
    auto at = [&](int d, asi::LdsAllowed& a) { dev = d; calls = 0; const hipError_t e = asi::allow_lds(nullptr, 90000, a); std::printf("%d%c ", calls, e == hipSuccess ? '+' : '-'); };
    at(0, allowed); at(0, allowed); at(1, allowed); at(0, allowed); at(1, allowed); at(63, allowed); at(63, allowed); at(64, allowed); at(64, allowed);
    at(0, other);
    fail = 1; at(5, allowed); fail = 0; at(5, allowed); at(5, allowed);
    return 0;
}
"""


def test_lds_allowance_is_asked_for_on_every_gpu(tmp_path):
    """A kernel's allowance of more than 64 KB of LDS belongs to one GPU: the second that the process launches on has to ask for it
    too (the runtime is a stand-in here), and a failure is not remembered as success."""
    import shutil
    import subprocess
    csrc = os.path.join(ROOT, "paper_2505_05086_amd", "csrc")
    users = [f for f in os.listdir(csrc) if "hipFuncSetAttribute" in open(os.path.join(csrc, f)).read()]
    assert users == ["asi_lds.h"]
    src, exe = tmp_path / "probe.cpp", tmp_path / "probe"
    src.write_text(LDS_PROBE)
    subprocess.run([shutil.which("g++") or "g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + csrc, str(src),
                    "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()
    assert out == ["1+", "0+", "1+", "0+", "0+", "1+", "0+", "1+", "1+", "1+", "1-", "1+", "0+"]
