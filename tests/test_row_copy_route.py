"""Which way populations are copied when devices differ, on the CPU: the library runs
against a stand-in runtime (the test program's own hip* functions take the place of the
HIP library's) that records kernel launches and copies and says on which device a
pointer lies.  The row kernel is for memory of the current device on both sides."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..")
ROCM = "/opt/rocm"

PROGRAM = r"""
#include <dlfcn.h>
#include <stdio.h>
#include <hip/hip_runtime_api.h>
#include "lbm.h"

static int current, launches, copies;
// addresses of this test: device * 2^40 + offset
static char *at(int device, size_t offset) { return (char *)(((size_t)device + 1) << 40) + offset; }

extern "C" {
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    *a = hipPointerAttribute_t{};
    a->type = hipMemoryTypeDevice;
    a->device = int((size_t)p >> 40) - 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = current; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t)
{
    ++launches;
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, hipMemcpyKind,
                            hipStream_t)
{
    ++copies;
    return hipSuccess;
}
}

int main(int argc, char **argv)
{
    void *lib = dlopen(argv[1], RTLD_NOW | RTLD_GLOBAL);
    if (!lib) return printf("%s\n", dlerror()), 2;
    auto create = (decltype(&lbm_create))dlsym(lib, "lbm_create");
    auto need = (decltype(&lbm_workspace_bytes))dlsym(lib, "lbm_workspace_bytes");
    auto get = (decltype(&lbm_get_populations))dlsym(lib, "lbm_get_populations");
    auto set = (decltype(&lbm_set_populations))dlsym(lib, "lbm_set_populations");
    lbm_params p{};
    p.struct_size = sizeof p;
    p.lattice = LBM_D2Q37;
    p.storage = LBM_F32;
    p.force_order = LBM_FORCE_N2;
    p.nx = p.ny = 501;  // 37 MB in rows of 2004 bytes: the row kernel's
    p.nz = 1;
    p.tau_hat = 0.8;
    p.rho0 = 1.0;
    int bad = 0;
    for (int home = 0; home < 2; ++home)
        for (int caller = 0; caller < 2; ++caller)
            for (current = 0; current < 2; ++current) {
                lbm_sim *s = nullptr;
                const double *f = (const double *)at(home, (size_t)1 << 39);
                if (create(&p, at(home, 0), need(&p), nullptr, f, f, f, &s) != LBM_OK) return 3;
                launches = copies = 0;
                void *dense = at(caller, (size_t)1 << 38);
                if (get(s, dense) != LBM_OK || set(s, dense) != LBM_OK) return 4;
                const int kernels = home == caller && home == current ? 2 : 0;
                if (launches != kernels || copies != 2 - kernels) {
                    printf("handle on %d, caller's memory on %d, current device %d: "
                           "%d kernels, %d copies\n", home, caller, current, launches, copies);
                    bad = 1;
                }
            }
    return bad;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_row_kernel_only_where_both_sides_are_on_the_current_device(tmp_path):
    from paper_2302_04741_amd import _lib

    _lib.load()
    src, exe = tmp_path / "route.cpp", tmp_path / "route"
    src.write_text(PROGRAM)
    cmd = ["g++", "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__=1",
           "-I" + os.path.join(ROCM, "include"), "-I" + os.path.join(ROOT, "include"), str(src),
           "-o", str(exe), "-ldl"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe), _lib.LIB_PATH], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
