"""What encoding a layer for a device asks of the HIP runtime: a few allocations and copies, since each
costs some ten microseconds and a small layer's call about as much.  The program defines the runtime's
calls itself (device memory is host memory), so this runs without a GPU; it also checks that what was
uploaded is what patdnn_decode finds."""

import os
import subprocess

from conftest import ROOT
from paper_2001_00138_amd import binding as B

SOURCE = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "patdnn.h"
static int mallocs = 0, copies = 0;
extern "C" {
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipMalloc(void** p, size_t n) { ++mallocs; *p = std::malloc(n); return *p ? 0 : 2; }
int hipFree(void* p) { std::free(p); return 0; }
int hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void*) { std::memset(p, v, n); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int kind)
{
    ++copies;
    std::memcpy(d, s, n);
    const uint32_t passed[5] = {0x1006, 0x1006, 0x1007, 0x100b, 10};     // the self-test's kernel, which does not run
    if (kind == 2 && n == sizeof(passed) && !static_cast<const uint32_t*>(s)[0]) std::memcpy(d, passed, n);
    return 0;
}
int hipStreamSynchronize(void*) { return 0; }
struct dim { uint32_t x, y, z; };
int hipLaunchKernel(const void*, dim, dim, void**, size_t, void*) { return 0; }
int hipGetLastError() { return 0; }
}
int main()
{
    // channels, stride, dense, depthwise, most allocations, most copies
    const int cases[][6] = {{16, 1, 0, 0, 6, 6}, {64, 1, 0, 0, 6, 6}, {64, 2, 0, 0, 3, 3}, {20, 1, 1, 0, 3, 3}, {40, 1, 0, 1, 2, 2},
                            {300, 1, 0, 0, 6, 30}};
    const uint16_t masks[2] = {27, 30};
    for (auto& t : cases) {
        const int c = t[0], per = t[3] ? 1 : c;
        std::vector<float> w((size_t)c * per * 9), back(w.size());
        std::vector<uint8_t> ids((size_t)c * per), mask(ids.size(), 1), ids_back(ids.size()), mask_back(ids.size());
        for (size_t k = 0; k < ids.size(); ++k) {
            ids[k] = k * 7 % 3 % 2;
            for (int q = 0; q < 9; ++q)
                if (t[2] || (masks[ids[k]] >> q & 1)) w[k * 9 + q] = (float)(k * 9 + q);
        }
        patdnn_layer_desc_t d{};
        d.c_out = d.c_in = c;
        d.groups = t[3] ? c : 1;
        d.stride = t[1];
        d.pad = 1;
        d.num_patterns = 2;
        d.pattern_masks = masks;
        d.flags = t[2] ? PATDNN_DENSE : 0;
        patdnn_handle_t h = nullptr;
        if (patdnn_selftest() != PATDNN_OK) return 5;  // its own allocation, once per process
        mallocs = copies = 0;
        if (patdnn_encode(&d, w.data(), ids.data(), mask.data(), &h) != PATDNN_OK) { std::printf("%s\n", patdnn_last_error()); return 1; }
        std::printf("%d channels: %d allocations, %d copies\n", c, mallocs, copies);
        if (mallocs > t[4] || copies > t[5]) return 2;
        if (patdnn_decode(h, back.data(), ids_back.data(), mask_back.data()) != PATDNN_OK) return 3;
        if (back != w || mask_back != mask || (!t[2] && ids_back != ids)) return 4;
        patdnn_destroy(h);
    }
    return 0;
}
"""


def test_a_layer_is_uploaded_in_few_pieces(tmp_path):
    if not os.path.exists(B.LIB_PATH):
        from paper_2001_00138_amd import buildlib
        buildlib.build()
    (tmp_path / "t.cpp").write_text(SOURCE)
    exe = str(tmp_path / "t")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"), str(tmp_path / "t.cpp"), B.LIB_PATH,
                        "-Wl,-rpath," + os.path.dirname(B.LIB_PATH), "-Wl,--allow-shlib-undefined", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, env=dict(os.environ, LD_LIBRARY_PATH="/opt/rocm/lib:" + os.environ.get("LD_LIBRARY_PATH", "")))
    assert r.returncode == 0, r.stdout + r.stderr
