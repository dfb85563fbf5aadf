"""Memory that a context keeps of a destroyed operator: csrc/context.cpp built
for the host over a device of 1000 bytes.  Kept blocks serve requests of a
similar size, make room when an allocation fails, are replaced by the next
operator's, and are all given back, whichever of context and operator goes
first.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1404_0812_amd", "csrc")
ROCM = "/opt/rocm/include"

SOURCE = r"""
#include "common.h"
#include <cstdlib>
#include <map>
static std::map<void*, size_t> held;
static size_t capacity = 1000, used = 0;
static int waits = 0;
static hipError_t last = hipSuccess;
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if (used + n > capacity) return last = hipErrorOutOfMemory;
    *p = std::malloc(1);
    held[*p] = n;
    used += n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!held.count(p)) std::abort();
    used -= held[p];
    held.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++waits; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "?"; }
}
int noalloc_scratch_setup(rbffd_ctx, int) { return RBFFD_OK; }
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
typedef SpareMemory::Block Block;
int main() {
    rbffd_ctx ctx = nullptr;
    CHECK(rbffd_create(&ctx, nullptr) == RBFFD_OK);
    SpareMemory* sp = ctx->spare;
    ++sp->owners;  // an operator
    Block a, w;
    CHECK(spare_take(sp, 400, a) && a.bytes == 400 && used == 400);
    CHECK(spare_take(sp, 100, w) && used == 500);
    spare_give(sp, {a, w}, true);
    CHECK(used == 500);
    Block b;
    CHECK(spare_take(sp, 90, b) && b.p == w.p && b.bytes == 100 && used == 500);  // the smaller that fits
    Block c;
    CHECK(spare_take(sp, 99, c) && c.bytes == 99 && used == 599);  // 400 is more than four times that
    CHECK(spare_take(sp, 200, w) && w.p == a.p && w.bytes == 400 && used == 599);
    spare_give(sp, {w, b}, true);
    CHECK(used == 599);
    // an allocation that fails with the spare held succeeds without it
    void* big = nullptr;
    CHECK(device_alloc(sp, &big, 800) == hipSuccess && used == 899);
    CHECK(hipFree(big) == hipSuccess);
    void* much = &ctx;
    CHECK(device_alloc(sp, &much, 1001) != hipSuccess && much == nullptr);
    CHECK(last == hipSuccess);  // a failure that was reported is not left for the next call
    // scratch: 4/3 of a megabyte at least
    capacity = (size_t)3 << 20;
    Block d;
    CHECK(spare_take(sp, (size_t)2 << 20, d));
    spare_give(sp, {d, c}, true);
    CHECK(ensure_scratch(ctx, (size_t)1 << 20) == RBFFD_OK);
    CHECK(ensure_scratch(ctx, (size_t)1 << 20) == RBFFD_OK);
    CHECK(ensure_scratch(ctx, (size_t)3 << 20) == RBFFD_E_NOMEM && last == hipSuccess);
    CHECK(used == 0 && ensure_scratch(ctx, 1) == RBFFD_OK);
    // the next operator's blocks replace the kept ones; none at all replace nothing
    capacity = (size_t)8 << 30;
    const size_t scratch = used;
    Block e, f;
    CHECK(spare_take(sp, 1000, e) && spare_take(sp, 1000, f));
    spare_give(sp, {e, Block{}}, true);
    spare_give(sp, {f, Block{}}, true);
    spare_give(sp, {Block{}, Block{}}, true);
    CHECK(used == scratch + 1000);
    // too much to keep, or not idle: freed
    CHECK(spare_take(sp, SPARE_MAX, e) && spare_take(sp, 5000, f));
    spare_give(sp, {e, f}, true);
    CHECK(spare_take(sp, 5000, f));
    spare_give(sp, {f, Block{}}, false);
    CHECK(used == scratch + 1000);
    // an operator that outlives its context
    CHECK(spare_take(sp, 800, e) && e.bytes == 1000);
    CHECK(rbffd_destroy(ctx) == RBFFD_OK);
    CHECK(used == 1000 && !sp->open);
    spare_give(sp, {e, Block{}}, true);
    CHECK(used == 0);
    spare_leave(sp, false);
    // and the usual order
    CHECK(rbffd_create(&ctx, nullptr) == RBFFD_OK);
    ++ctx->spare->owners;
    CHECK(spare_take(ctx->spare, 700, a));
    spare_give(ctx->spare, {a, Block{}}, true);
    spare_leave(ctx->spare, false);
    CHECK(rbffd_destroy(ctx) == RBFFD_OK && used == 0);
    std::printf("ok\n");
    return 0;
}
"""


def test_kept_blocks(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.isdir(os.path.join(ROCM, "hip")):
        pytest.skip("no host compiler or HIP headers")
    (tmp_path / "t.cpp").write_text(SOURCE)
    subprocess.run([cxx, "-std=c++17", "-g", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__", "-w", "-I", ROCM,
                    "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(tmp_path / "t.cpp"),
                    os.path.join(CSRC, "context.cpp"), "-o", str(tmp_path / "t"), "-pthread"], check=True)
    r = subprocess.run([str(tmp_path / "t")], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
