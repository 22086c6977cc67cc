"""CPU: the limit of a kernel's dynamic LDS (csrc/lds_grant.h) against a runtime of a few lines that keeps it per device, as HIP does."""
import ctypes as C
import subprocess
import threading

import pytest

from paper_2603_07169_amd import build as lib_build

RUNTIME = r"""
#include "lds_grant.h"
static thread_local int current = 0;
static int limits[4] = {65536, 65536, 65536, 65536}, calls = 0, failing = 0;
extern "C" {
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) { a->sharedSizeBytes = 2112; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int v) {
    ++calls;
    if (failing || v > 163840 - 2112) return hipErrorInvalidValue;
    limits[current] = v;
    return hipSuccess;
}
int ask(int device, size_t lds) {  // a launch: 0 when it is let through and the runtime's limit holds it
    static spmv::LdsGrant grant;
    current = device;
    if (grant(nullptr, lds) != hipSuccess) return 1;
    return lds + 2112 <= 65536 || lds <= static_cast<size_t>(limits[device]) ? 0 : 2;
}
void fail(int on) { failing = on; }
int asked() { return calls; }
}
"""


@pytest.fixture
def runtime(tmp_path):
    (tmp_path / "runtime.cpp").write_text(RUNTIME)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{lib_build.CSRC}", str(tmp_path / "runtime.cpp"), "-o", str(tmp_path / "runtime.so")], check=True)
    lib = C.CDLL(str(tmp_path / "runtime.so"))
    lib.ask.argtypes = [C.c_int, C.c_size_t]
    return lib


def on_a_thread(call):
    out = []
    t = threading.Thread(target=lambda: out.append(call()))
    t.start()
    t.join()
    return out[0]


def test_one_thread_takes_nothing_from_another(runtime):
    assert runtime.ask(0, 150000) == 0
    assert on_a_thread(lambda: runtime.ask(0, 70000)) == 0
    assert runtime.ask(0, 150000) == 0
    assert runtime.asked() == 1


def test_every_device_is_told(runtime):
    assert [runtime.ask(d, 150000) for d in (0, 1, 3, 1, 0)] == [0] * 5
    assert runtime.asked() == 3


def test_edges(runtime):
    assert [runtime.ask(0, lds) for lds in (0, 60 * 1024)] == [0, 0] and runtime.asked() == 0  # the default limit holds them
    assert [runtime.ask(0, lds) for lds in (60 * 1024 + 1, 64 * 1024, 64 * 1024 + 1)] == [0, 0, 0]
    assert runtime.ask(0, 160 * 1024 - 2112) == 0 and runtime.ask(0, 160 * 1024 - 2111) == 1   # all there is, and more


def test_a_refusal_is_handed_on_and_not_kept(runtime):
    runtime.fail(1)
    assert runtime.ask(0, 70000) == 1
    runtime.fail(0)
    assert runtime.ask(0, 70000) == 0 and runtime.asked() == 2
