"""The block deposit's bin counts (csrc/pm.hip) are zero whenever a launch
that adds to them runs, also where an allocation or a launch failed or a call
was captured in between: the host code of pm.hip against a stand-in of the HIP
runtime that keeps track of which count buffers hold zeros.  Counts left over
would send the sort's writes out of range, so this runs on the CPU alone."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_14008_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

STAND_IN = r"""
#include "pm.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

static std::map<const void*, std::string> names;   // host stub -> kernel
static std::set<const void*> zeroed;               // count buffers that hold zeros
static std::vector<std::function<void()>> graph;   // launches of the captured call
static bool capturing = false;
static int fail_malloc = 0;                        // the n-th allocation from here fails
static const char* fail_launch = "";               // the next launch of this kernel fails
static int error = 0, bad = 0, counted = 0;
static dim3 cfg_g, cfg_b;
static size_t cfg_m;
static hipStream_t cfg_s;

static void execute(const std::string& k, const void* p) {
    if (k.find("pm_zero") != std::string::npos) zeroed.insert(p);
    if (k.find("pm_bin_count") != std::string::npos) {
        ++counted;
        if (!zeroed.count(p)) ++bad;
        zeroed.erase(p);
    }
    if (k.find("pm_bin_scan") != std::string::npos) zeroed.insert(p);
}

extern "C" {
char FATBIN[64];
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*,
                           void*, int*) { names[f] = name; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
    cfg_g = g; cfg_b = b; cfg_m = m; cfg_s = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
    *g = cfg_g; *b = cfg_b; *m = cfg_m; *s = cfg_s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
    const std::string k = names[f];
    if (*fail_launch && k.find(fail_launch) != std::string::npos) {
        fail_launch = "";
        error = 1;
        return hipErrorUnknown;
    }
    // the count buffer's place among the arguments
    const int at = k.find("pm_bin_count") != std::string::npos ? 4 : k.find("pm_bin_scan") != std::string::npos ? 1 : 0;
    const void* p = *(const void* const*)args[at];
    if (capturing) graph.push_back([=] { execute(k, p); });
    else execute(k, p);
    return hipSuccess;
}
hipError_t hipGetLastError() { const int e = error; error = 0; return e ? hipErrorUnknown : hipSuccess; }
hipError_t hipMalloc(void** p, size_t) {
    if (capturing || (fail_malloc > 0 && --fail_malloc == 0)) { error = 1; return hipErrorOutOfMemory; }
    *p = std::malloc(16);
    return hipSuccess;
}
hipError_t hipFree(void* p) { zeroed.erase(p); return hipSuccess; }   // addresses are not used again
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
    *c = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipfftResult hipfftDestroy(hipfftHandle) { return HIPFFT_SUCCESS; }
hipfftResult hipfftExecD2Z(hipfftHandle, hipfftDoubleReal*, hipfftDoubleComplex*) { return HIPFFT_SUCCESS; }
hipfftResult hipfftExecZ2D(hipfftHandle, hipfftDoubleComplex*, hipfftDoubleReal*) { return HIPFFT_SUCCESS; }
hipfftResult hipfftPlan3d(hipfftHandle* h, int, int, int, hipfftType) { *h = (hipfftHandle)1; return HIPFFT_SUCCESS; }
hipfftResult hipfftPlanMany(hipfftHandle* h, int, int*, int*, int, int, int*, int, int, hipfftType, int) {
    *h = (hipfftHandle)2;
    return HIPFFT_SUCCESS;
}
hipfftResult hipfftSetStream(hipfftHandle, hipStream_t) { return HIPFFT_SUCCESS; }
}

static double x[1];
static pmfmm::PMPlan plan;
static hipError_t force(int64_t np, int n = 32) {
    hipError_t e = pmfmm::pm_plan(plan, n, nullptr);
    return e != hipSuccess ? e : pmfmm::pm_long_range(plan, x, x, np, 100.0, 3.0, 1.0, x, nullptr);
}

int main(int, char** argv) {
    const std::string what = argv[1];
    if (what == "grow" || what == "first") {
        // the bin buffer grows, the tiles behind it do not fit; the next call
        // that fits is captured, and one runs before the graph does
        if (what == "grow") force(20000);
        else pmfmm::pm_plan(plan, 32, nullptr);
        fail_malloc = 4;
        force(100000);
        capturing = true;
        force(20000);
        capturing = false;
        force(20000);
        for (auto& l : graph) l();
        force(20000);
        for (auto& l : graph) l();
    } else if (what == "launch") {
        force(20000);
        fail_launch = "pm_bin_scan";
        if (force(20000) == hipSuccess) return 2;
        force(20000);
        force(20000);
    } else if (what == "mesh") {
        for (int n : {32, 34, 32, 64}) { force(70000, n); force(150000, n); force(70000, n); }
    }
    std::printf("%d counts, %d on a buffer that held no zeros\n", counted, bad);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(HIPCC) or shutil.which("nm") is None:
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("pm")
    (d / "stand_in.cpp").write_text(STAND_IN)
    inc = [f"-I{ROOT}/include", f"-I{CSRC}", "-std=c++17", "-O1", "-fPIC", "-w"]
    subprocess.run([HIPCC, *inc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-c",
                    os.path.join(CSRC, "pm.hip"), "-o", str(d / "pm.o")], check=True)
    sym = subprocess.run(["nm", str(d / "pm.o")], capture_output=True, text=True, check=True).stdout
    fat = re.search(r"U (__hip_fatbin\w*)", sym).group(1)
    subprocess.run(["g++", *inc, "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include", f"-DFATBIN={fat}",
                    str(d / "stand_in.cpp"), str(d / "pm.o"), "-o", str(d / "run")], check=True)
    return str(d / "run")


@pytest.mark.parametrize("what,counts", [("grow", 5), ("first", 2), ("launch", 4), ("mesh", 12)])
def test_bin_counts_are_zero_when_they_are_added_to(program, what, counts):
    out = subprocess.run([program, what], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr
    assert out.stdout == f"{counts} counts, 0 on a buffer that held no zeros\n", out.stdout
