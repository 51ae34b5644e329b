"""Which way a plan blob goes to the device, on the host alone: the runtime's answers about the two buffers are given by a stand-in for its
functions, which records the launch or the copy that apt_plan_upload issues."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# answers from the environment: allocation around each buffer (its bytes before and from it on), kind of memory, devices, capture
RUNTIME = r"""
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
static long value(const char* name) { const char* v = getenv(name); return v ? strtol(v, 0, 0) : 0; }
static char* host() { return (char*)value("HOST"); }
static char* device() { return (char*)value("DEVICE"); }
extern "C" {
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    memset(a, 0, sizeof *a);
    const bool h = p == host();
    if (value(h ? "HOST_UNKNOWN" : "DEVICE_UNKNOWN")) return hipErrorInvalidValue;
    a->type = (hipMemoryType)value(h ? "HOST_TYPE" : "DEVICE_TYPE");
    a->device = (int)value("POINTER_DEVICE");
    a->devicePointer = (char*)p + (h ? value("MAPPED_AT") : 0);
    return hipSuccess;
}
hipError_t hipPointerGetAttribute(void* out, hipPointer_attribute what, hipDeviceptr_t p) {
    const bool h = p == host();
    if (what == HIP_POINTER_ATTRIBUTE_RANGE_START_ADDR) *(char**)out = (char*)p - value(h ? "HOST_BEFORE" : "DEVICE_BEFORE");
    else if (what == HIP_POINTER_ATTRIBUTE_RANGE_SIZE)
        *(size_t*)out = value(h ? "HOST_BEFORE" : "DEVICE_BEFORE") + value(h ? "HOST_BYTES" : "DEVICE_BYTES");
    else return hipErrorInvalidValue;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = (int)value("CURRENT_DEVICE"); return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = (int)value("STREAM_DEVICE"); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = (hipStreamCaptureStatus)value("CAPTURING"); return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    printf("copy %d %zu\n", d == device() && s == host(), n);
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t) {
    printf("launch %d\n", *(void**)args[0] == device());
    return hipSuccess;
}
}
"""

SCRIPT = """
import ctypes as C, os, sys
C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)                  # before the library, whose calls it then answers
import numpy as np
from paper_2504_07494_amd import binding as ab
shape = ab.make_shape(128, 1, 128, 16, "f16", 32, 1.0)
for n in (20, 200, 1000):
    lens, kinds = np.full(n, 17, dtype=np.int32), np.zeros(n, dtype=np.uint8)
    words = np.zeros(ab.apt_plan_max_bytes(shape, n, 512) // 4 + 64, dtype=np.int32)
    words = words[-words.ctypes.data // 4 % 4:]          # to 16 bytes
    blob = words[int(sys.argv[2]):]
    info = ab.apt_plan(shape, lens, kinds, blob)
    # setenv of the C library, which the stand-in reads
    settings = dict(HOST=blob.ctypes.data, DEVICE=0x7000000000 + int(sys.argv[3]), HOST_TYPE=1, DEVICE_TYPE=2, HOST_BYTES=info.plan_bytes,
                    DEVICE_BYTES=info.plan_bytes)
    settings.update((k, eval(v, {"n": int(info.plan_bytes)})) for k, v in (s.split("=") for s in sys.argv[4:]))
    for k, v in settings.items():
        C.CDLL(None).setenv(k.encode(), str(v).encode(), 1)
    print(n, info.plan_bytes, end=" ", flush=True)
    ab.apt_plan_upload(blob, settings["DEVICE"], 0)
    C.CDLL(None).fflush(None)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    where = tmp_path_factory.mktemp("runtime")
    (where / "runtime.cpp").write_text(RUNTIME)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", os.path.join(rocm, "include"), str(where / "runtime.cpp"), "-o",
                    str(where / "runtime.so")], check=True)
    return str(where / "runtime.so")


@pytest.mark.parametrize("host_at,device_at,settings,by_kernel", [
    (0, 0, [], True),
    (0, 0, ["HOST_BEFORE=4096", "HOST_BYTES=n+64", "DEVICE_BEFORE=512", "DEVICE_BYTES=n+1"], True),     # inside larger allocations
    (0, 0, ["HOST_BYTES=n-1"], False), (0, 0, ["HOST_BEFORE=4096", "HOST_BYTES=n-4"], False),           # reads past the source
    (0, 0, ["DEVICE_BYTES=n-1"], False), (0, 0, ["DEVICE_BEFORE=1<<20", "DEVICE_BYTES=n-4"], False),    # writes past the destination
    (0, 0, ["DEVICE_BYTES=8"], False),
    (0, 0, ["HOST_TYPE=0"], False), (0, 0, ["HOST_TYPE=3"], False), (0, 0, ["MAPPED_AT=4096"], False), (0, 0, ["HOST_UNKNOWN=1"], False),
    (0, 0, ["DEVICE_TYPE=1"], False), (0, 0, ["DEVICE_TYPE=3"], False), (0, 0, ["DEVICE_UNKNOWN=1"], False),
    (0, 0, ["CURRENT_DEVICE=1"], False), (0, 0, ["STREAM_DEVICE=1"], False), (0, 0, ["POINTER_DEVICE=1"], False),
    (0, 0, ["POINTER_DEVICE=1", "CURRENT_DEVICE=1", "STREAM_DEVICE=1"], True),
    (0, 0, ["CAPTURING=1"], False), (2, 0, [], True), (1, 0, [], False), (0, 4, [], False), (0, 8, [], True)])
def test_route(runtime, host_at, device_at, settings, by_kernel):
    env = dict(os.environ, PYTHONPATH=ROOT)
    out = subprocess.run([sys.executable, "-c", SCRIPT, runtime, str(host_at), str(device_at), *settings], env=env, text=True,
                         capture_output=True, check=True).stdout
    rows = [line.split() for line in out.splitlines()]
    assert [int(r[0]) for r in rows] == [20, 200, 1000]
    small, middle, large = rows
    assert int(small[1]) <= 3840 < int(middle[1]) <= 16384 < int(large[1])
    # a small blob rides in a launch (not under capture); a middle one is the runtime's, as is every one the kernel may not read or write
    assert small[2:] == (["copy", "1", small[1]] if "CAPTURING=1" in settings else ["launch", "1"])
    assert middle[2:] == ["copy", "1", middle[1]]
    assert large[2:] == (["launch", "1"] if by_kernel else ["copy", "1", large[1]])
