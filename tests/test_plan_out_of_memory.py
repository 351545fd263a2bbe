"""Host memory that runs out while a plan is uploaded: sht_plan_ex and
sht_plan_load return NULL with SHT_ENOMEM and hold no device memory; no C++
exception leaves the C entry.

A small program links the library and takes the place of the device runtime's
memory calls (plain host memory, launches that do nothing) and of operator
new, which it lets fail at the k-th allocation after the upload began, for
every k.  No GPU needed.
"""
import os
import subprocess

import pytest

from paper_1110_4874_amd import build

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

#include "sht.h"

static long live = 0, count = -1, fail_at = -1;  // count: allocations since the upload began

extern "C" {
int hipGetDevice(int *d) { return *d = 0; }
int hipSetDevice(int) { return 0; }
int hipMalloc(void **p, size_t n) {
    if (count < 0) count = 0;
    *p = calloc(1, n ? n : 1);
    live += *p != nullptr;
    return *p ? 0 : 2;
}
int hipFree(void *p) {
    live -= p != nullptr;
    free(p);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) {
    memcpy(d, s, n);
    return 0;
}
int hipLaunchKernel(...) { return 0; }
int hipGetLastError() { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetSymbolAddress(void **p, const void *) {
    static char scratch;
    *p = &scratch;
    return 0;
}
}

void *operator new(size_t n) {
    if (count >= 0 && fail_at >= 0 && count++ == fail_at) throw std::bad_alloc();
    if (void *p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

// argv: plan file ("" = build the plan), L, nside, eps
int main(int, char **argv) {
    for (fail_at = 0;; fail_at++) {
        count = -1;
        sht_plan_opts o;
        sht_plan_opts_default(&o);
        o.nthreads = 1;
        o.store_fp32 = 1;
        o.max_levels = 1;
        sht_plan_t *p = argv[1][0] ? sht_plan_load_ex(argv[1], &o) : sht_plan_ex(atoi(argv[2]), atoi(argv[3]), atof(argv[4]), &o);
        const long seen = count;
        count = -1;
        if (p) {
            sht_plan_free(p);
            if (seen > fail_at && !live) continue;  // an allocation the library can do without
            printf("%ld allocations, %ld device blocks left\n", fail_at, live);
            return live ? 1 : 0;
        }
        if (sht_last_status() != SHT_ENOMEM || live) {
            printf("allocation %ld: status %d, %ld device blocks left\n", fail_at, sht_last_status(), live);
            return 1;
        }
    }
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_1110_4874_amd import sht
    sht.load()
    d = tmp_path_factory.mktemp("oom")
    src, exe = str(d / "driver.cpp"), str(d / "driver")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(build.ROOT, "include"), src, "-o",
                           exe, build.LIB, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + os.path.dirname(build.LIB)])
    return exe


@pytest.mark.parametrize("L,N,eps", [(40, 12, 0.0), (47, 12, 1e-6)])
@pytest.mark.parametrize("loaded", [False, True])
def test_upload_reports_lack_of_memory(driver, tmp_path, L, N, eps, loaded):
    from paper_1110_4874_amd import sht
    path = ""
    if loaded:
        path = str(tmp_path / "p.plan")
        sht.Plan(L, N, eps, max_levels=1, host_only=True).save(path)
    r = subprocess.run([driver, path, str(L), str(N), str(eps)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    assert int(r.stdout.split()[0]) > 0
