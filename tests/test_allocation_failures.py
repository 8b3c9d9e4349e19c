"""Host memory that runs out at any point of an entry point's work comes back as PATDNN_ENOMEM, never as an
exception through the C interface, leaves the handle usable and leaks no device memory.  The program defines
the HIP calls itself (device memory is host memory, kernels do not run) and an operator new whose n-th call
fails; it repeats every entry point with n = 1, 2, ... until the call gets through."""

import os
import subprocess

from conftest import ROOT
from paper_2001_00138_amd import binding as B

SOURCE = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <new>
#include <vector>
#include "patdnn.h"
static long fail_at = 0, calls = 0, device_blocks = 0;       // fail_at 0: never
void* operator new(size_t n)
{
    if (fail_at && ++calls == fail_at) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
extern "C" {
struct dim { uint32_t x, y, z; };
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipMalloc(void** p, size_t n) { ++device_blocks; *p = std::malloc(n); return *p ? 0 : 2; }
int hipFree(void* p) { device_blocks -= p != nullptr; std::free(p); return 0; }
int hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void*) { std::memset(p, v, n); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int kind)
{
    std::memcpy(d, s, n);
    const uint32_t passed[5] = {0x1006, 0x1006, 0x1007, 0x100b, 10};     // the self-test's kernel, which does not run
    if (kind == 2 && n == sizeof(passed) && !static_cast<const uint32_t*>(s)[0]) std::memcpy(d, passed, n);
    return 0;
}
int hipStreamSynchronize(void*) { return 0; }
int hipLaunchKernel(const void*, dim, dim, void**, size_t, void*) { return 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipEventCreate(void** e) { ++device_blocks; *e = std::malloc(1); return 0; }
int hipEventDestroy(void* e) { --device_blocks; std::free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
}

// `call` with the first, second, ... allocation failing, until none does
static bool all(const char* what, const std::function<patdnn_status_t()>& call, long stride = 1)
{
    for (long n = 1;; n += stride) {
        calls = 0;
        fail_at = n;
        const patdnn_status_t st = call();
        const bool failed = calls >= fail_at;
        fail_at = 0;
        if (st != PATDNN_OK && st != PATDNN_ENOMEM) { std::printf("%s, allocation %ld: %s\n", what, n, patdnn_last_error()); return false; }
        if (!failed) { std::printf("%s: %ld allocations\n", what, calls); return st == PATDNN_OK; }
    }
}
int main()
{
    for (int k = 0; k < 3; ++k) {                       // pruned, dense, depthwise
        const int c = 20, per = k == 2 ? 1 : c;
        std::vector<float> w((size_t)c * per * 9, 0.5f), x((size_t)c * 64), y(x.size());
        std::vector<uint8_t> ids((size_t)c * per), mask(ids.size(), 1);
        const uint16_t masks[2] = {27, 30};
        for (size_t i = 0; i < ids.size(); ++i) ids[i] = i % 2;
        patdnn_layer_desc_t d{};
        d.c_out = d.c_in = c;
        d.groups = k == 2 ? c : 1;
        d.stride = d.pad = 1;
        d.num_patterns = 2;
        d.pattern_masks = masks;
        d.flags = k == 1 ? PATDNN_DENSE : 0;
        if (patdnn_selftest() != PATDNN_OK) return 1;
        patdnn_handle_t h = nullptr;
        if (!all("encode", [&] {
                if (h) patdnn_destroy(h);
                return patdnn_encode(&d, w.data(), ids.data(), mask.data(), &h);
            })) return 2;
        patdnn_stats_t stats;
        if (!all("layout_stats", [&] { return patdnn_layout_stats(h, &stats); })) return 3;
        for (int v = 0; v < patdnn_num_variants(); ++v) {
            const patdnn_config_t cfg{v, 5, 0, 1};
            if (patdnn_set_config(h, &cfg) != PATDNN_OK) continue;
            // a fresh handle: the layout is built again
            if (!all(patdnn_variant_name(v), [&] {
                    patdnn_handle_t g = nullptr;
                    const long at = fail_at;
                    fail_at = 0;
                    if (patdnn_encode(&d, w.data(), ids.data(), mask.data(), &g) != PATDNN_OK) return PATDNN_EINVAL;
                    fail_at = at;
                    patdnn_status_t st = patdnn_set_config(g, &cfg);
                    if (st == PATDNN_OK) st = patdnn_conv2d(g, x.data(), 1, 8, 8, nullptr, y.data(), 1, nullptr);
                    const long now = fail_at;
                    fail_at = 0;
                    const bool usable = patdnn_set_config(g, &cfg) == PATDNN_OK;
                    patdnn_destroy(g);
                    fail_at = now;
                    return usable ? st : PATDNN_EINVAL;
                })) return 4;
        }
        if (!all("tune", [&] { return patdnn_tune(h, x.data(), 1, 8, 8, nullptr, y.data(), nullptr, nullptr); }, 7)) return 5;
        const patdnn_config_t choose{-1, 0, 0, 1};
        if (!all("conv2d", [&] {
                patdnn_status_t st = patdnn_set_config(h, &choose);
                return st != PATDNN_OK ? st : patdnn_conv2d(h, x.data(), 1, 8, 8, nullptr, y.data(), 1, nullptr);
            })) return 6;
        patdnn_stack_t stack = nullptr;
        const patdnn_stack_layer_t layers[2] = {{h, nullptr, 1, 0}, {h, nullptr, 1, k != 2}};
        if (!all("stack", [&] {
                if (stack) patdnn_stack_destroy(stack);
                patdnn_status_t st = patdnn_stack_create(layers, 2, 1, 8, 8, &stack);
                return st != PATDNN_OK ? st : patdnn_stack_run(stack, x.data(), y.data(), 0, nullptr);
            })) return 7;
        patdnn_stack_destroy(stack);
        patdnn_destroy(h);
        if (device_blocks) { std::printf("%ld device blocks left\n", device_blocks); return 8; }
    }
    return 0;
}
"""


def test_every_failing_allocation_is_reported(tmp_path):
    if not os.path.exists(B.LIB_PATH):
        from paper_2001_00138_amd import buildlib
        buildlib.build()
    (tmp_path / "t.cpp").write_text(SOURCE)
    exe = str(tmp_path / "t")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"), str(tmp_path / "t.cpp"), B.LIB_PATH,
                        "-Wl,-rpath," + os.path.dirname(B.LIB_PATH), "-Wl,--allow-shlib-undefined", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, LD_LIBRARY_PATH="/opt/rocm/lib:" + os.environ.get("LD_LIBRARY_PATH", "")))
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
