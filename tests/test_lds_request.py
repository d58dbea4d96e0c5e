"""Requests for LDS beyond 64 KiB: once per kernel and device, and again after
one that failed.  The rule is compiled from the library's header against
stand-ins for the two runtime calls."""
import os
import subprocess

from conftest import ROOT

SOURCE = r"""
#include "tg_internal.hpp"
#include <cassert>
#include <cstdio>
#include <set>
#include <utility>

static int device, calls, fail;
static std::set<std::pair<int, const void *>> have;
extern "C" hipError_t hipGetDevice(int *d) {
    *d = device;
    return hipSuccess;
}
extern "C" hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute,
                                          int) {
    ++calls;
    if (fail) return hipErrorOutOfMemory;
    have.insert({device, f});
    return hipSuccess;
}

int main() {
    int a, b;
    tg::LdsRequest r;
    fail = 1;
    assert(r({&a, nullptr, &b}, 1) == hipErrorOutOfMemory && calls == 1);
    fail = 0;
    assert(r({&a, nullptr, &b}, 1) == hipSuccess && calls == 3);
    assert(r({&a, nullptr, &b}, 1) == hipSuccess && calls == 3);
    for (device = 1; device < 70; ++device) {
        assert(r({&a, &b}, 1) == hipSuccess);
        assert(have.count({device, &a}) && have.count({device, &b}));
    }
    device = 0;
    const int before = calls;
    assert(r({&a, &b}, 1) == hipSuccess && calls == before);
    puts("ok");
}
"""


def test_once_per_kernel_and_device(tmp_path):
    src, exe = tmp_path / "r.cpp", tmp_path / "r"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2606_15991_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.stdout.strip() == "ok", r.stderr


def test_every_request_goes_through_it():
    """No launch keeps the answer of its first request for all devices."""
    csrc = os.path.join(ROOT, "paper_2606_15991_amd", "csrc")
    for f in os.listdir(csrc):
        for line in open(os.path.join(csrc, f)):
            assert not ("static" in line and "hipFuncSetAttribute" in line), f
