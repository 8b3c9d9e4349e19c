// Device-side views of an encoded layer and the launchers of each kernel family.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <string>

#include "layout.hpp"

namespace patdnn {

struct ConvShape {
    int32_t n, c_in, c_out, h, w, ho, wo, stride, pad, relu;
    // pool != 0: ReLU, then 2x2 max pooling with stride 2 (floor), fused into the epilogue.
    // The output tensor is [n][c_out][ho/2][wo/2] and, for all kernels but the tap-product, the split and the
    // dense one (whole windows in registers), must hold zeros when the kernel starts: every lane folds its values in
    // with an unsigned integer atomic max on the float bits, which orders non-negative floats like the
    // floats themselves.
    int32_t pool = 0;
    // Zero-fill hand-off between consecutive launches of a stack (all optional).  The launches
    // that add into their target with atomics (split, pooled) need it zeroed beforehand, which
    // costs a kernel launch of its own; a launch that ends with a finishing kernel can clear
    // the next launch's target in that same kernel instead.
    //   pre_zeroed / pre_zeroed_count: a region that already holds zeros on entry; a zero fill of
    //     exactly that region (same start, no more floats) is skipped.
    //   zero_next / zero_next_count: a region to clear in this launch's finishing kernel, if it
    //     has one and the region is not one the kernel still reads; *zero_next_done is set when
    //     it was cleared (left alone otherwise).
    const float* pre_zeroed = nullptr;
    size_t pre_zeroed_count = 0;
    float* zero_next = nullptr;
    size_t zero_next_count = 0;
    bool* zero_next_done = nullptr;
};

// Fills `count` floats with zero (a kernel, so that it can be captured into a HIP graph).
hipError_t launch_fill_zero(float* p, size_t count, hipStream_t stream);

// Floats between the partial-sum buffers of a split launch whose output has `total` floats (a
// launch with `ksplit` slices stores to buffers if its scratch holds ksplit of them).
size_t split_slice_stride(size_t total);

// Division of a value below 2^31 by a launch-time constant d >= 1 without the divider loop:
// with l = ceil(log2 d) and m = ceil(2^(31+l) / d) (which fits 32 bits), floor(n / d) =
// (n * m) >> (31 + l) exactly for every n < 2^31 (the error term n * (m*d - 2^(31+l)) /
// (d * 2^(31+l)) stays below 2^-l <= 1/d).  The tiled kernel divides band numbers by the bands per
// image row and column seven times per thread before it can start; the depthwise kernel, which
// has a dozen FMAs per thread, spends most of its instructions on turning a thread number into
// (image, channel, row, column).
struct FastDiv {
    uint32_t m, shift;
};
inline FastDiv make_fast_div(uint32_t d)
{
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;
    const uint64_t p = 1ull << (31 + l);
    return FastDiv{(uint32_t)((p + d - 1) / d), 31 + l};
}
__host__ __device__ __forceinline__ uint32_t fast_div(uint32_t n, FastDiv f)
{
    return (uint32_t)(((uint64_t)n * f.m) >> f.shift);
}


// FKW arrays on the device (paper section 5.3).
struct DevFkw {
    const int32_t* offset = nullptr;
    const int32_t* reorder = nullptr;
    const int32_t* index = nullptr;
    const int32_t* stride = nullptr;
    const float* weight = nullptr;
    const uint16_t* masks = nullptr;
    int32_t num_patterns = 0;
    int32_t taps = 4;
    // depthwise layers: per stored filter, the pattern mask of its one kernel (0 if the
    // kernel was removed) and its four weights
    const int32_t* dw_mask = nullptr;
    const float* dw_weight = nullptr;
    bool dw_finite = false;          // all of those weights are finite
    // the same by channel, four tap positions in nibbles (-1: removed); NULL where a weight is
    // not finite in binary16 (zero padding must not meet it)
    const int32_t* dw_taps = nullptr;
    const float* dw_tap_weight = nullptr;
    // the weights once more as IEEE binary16 (round to nearest even), for the
    // half-precision-storage entry point: `weight` and `dw_weight` element for element
    const void* weight_f16 = nullptr;
    const void* dw_weight_f16 = nullptr;
    // all nine taps of every kernel in binary16, zeros where pruning removed a weight, in the
    // matrix instructions' order (kernel_f16.hip); NULL: depthwise layers, very large ones and
    // those with a weight that is not finite in binary16
    const void* expanded_f16 = nullptr;
    // likewise as pairs of binary16 numbers (kernel_split.hip), and per stored filter, to whole blocks of 64,
    // its channel (-1: none) and the power of two that its weights were multiplied with (kSplitEmpty: it has none)
    const void* split_f16 = nullptr;
    const int32_t* split_filters = nullptr;
    // so small a sum, in the scales of weights and inputs, may be off by 2^-24 of itself for inputs below the scale
    float split_seen = 0.0f;
};

// Filter-group layout on the device: record streams (sparse) or 9-tap weights (dense).
struct DevTiled {
    int32_t G = 0;
    int32_t num_groups = 0;
    int32_t ck = 0;            // input channels staged per LDS pass (fixes the chunking of the streams)
    int32_t num_chunks = 0;
    const int32_t* slot_channel = nullptr;
    const uint32_t* chunk_ptr = nullptr;   // [num_groups][num_chunks] first step of a chunk | entry block << 28
    const uint32_t* steps = nullptr;       // [steps][kStepDwords]
    const float* w9 = nullptr;
};

// Filter-major walk of the FKW arrays, one lane per output pixel.
hipError_t launch_fkw(const DevFkw& f, const ConvShape& s, const float* in, const float* bias,
                      float* out, hipStream_t stream);

// The comparison kernels' views of a layer (kernel_compare.hip): the layer before
// filter-kernel reorder, and as a CSR matrix.
struct DevCompare {
    const int32_t* row_ptr = nullptr;
    const int32_t* col = nullptr;
    const int32_t* kmask = nullptr;
    const float* val = nullptr;
};
hipError_t launch_compare(bool csr, const DevCompare& d, const ConvShape& s, const float* in, const float* bias,
                          float* out, hipStream_t stream);

// Depthwise layers: one pass over input and output, vector accesses, two rows of four or eight outputs per lane.
hipError_t launch_dw(const DevFkw& f, const ConvShape& s, const float* in, const float* bias,
                     float* out, hipStream_t stream);
// The same two kernels on binary16 tensors and weights (fp32 arithmetic, fp32 bias); the walk where
// launch_f16 does not reach.
hipError_t launch_dw_f16(const DevFkw& f, const ConvShape& s, const void* in, const float* bias,
                         void* out, hipStream_t stream);
hipError_t launch_fkw_f16(const DevFkw& f, const ConvShape& s, const void* in, const float* bias,
                          void* out, hipStream_t stream);
// What a depthwise call launches: 0 element by element, 1 planes through LDS, else rows: 2, one more where they are whole vectors, two
// more for eight outputs a lane, four more for stores past the L2s.
int dw_choice(const DevFkw& f, const ConvShape& s, const void* in, const void* out, bool half);
// Pruned and dense layers on the matrix cores (needs DevFkw::expanded_f16).
hipError_t launch_f16(const DevFkw& f, const ConvShape& s, const void* in, const float* bias,
                      void* out, hipStream_t stream);
// What it launches: twice the index of the launch shape, plus one where rows are staged in pairs of
// pixels; -1: the walk.
int f16_choice(const ConvShape& s, const void* in);
size_t f16_expanded_halves(int32_t c_in, int32_t c_out);
// Fills `out` (f16_expanded_halves, zeroed) from the FKW arrays.
hipError_t launch_f16_expand(const DevFkw& f, int32_t c_in, int32_t c_out, void* out, hipStream_t stream);

// fp32 on the binary16 matrix cores (needs DevFkw::split_f16).
// False where its numbers do not reach; else the units of work that the busiest workgroup has, the channel steps of
// each and the pixels of a wavefront.
bool split_cost(const ConvShape& s, int& rounds, int& steps, int& pixels);
// What launch_split launches for a tensor at `in`: twice the number of the shape, plus one for loads of pixel pairs
// (-1: nothing fits), and the units of work.
int split_choice(const ConvShape& s, const void* in, int& units);
hipError_t launch_split(const DevFkw& f, const ConvShape& s, const float* in, const float* bias, float* out, hipStream_t stream);
constexpr int kSplitEmpty = 1 << 20;
size_t split_expanded_halves(int32_t c_in, int32_t c_out);
// Fills `out` (split_expanded_halves, zeroed) from the FKW arrays and split_filters.
hipError_t launch_split_expand(const DevFkw& f, int32_t c_in, int32_t c_out, void* out, hipStream_t stream);

// Dense layers of up to so many input channels on the fp32 matrix cores (kernel_dense.hip); weights finite.
constexpr int kDenseChannels = 4;
bool dense_fits(const ConvShape& s);
hipError_t launch_dense(const DevFkw& f, const ConvShape& s, const float* in, const float* bias, float* out, hipStream_t stream);

// ---------------------------------------------------------------------------
// Tiled kernels: compile-time geometry per variant, run-time launch parameters.
// ---------------------------------------------------------------------------
struct TiledVariant {
    const char* name;
    int32_t G;        // filters per group (one group per wavefront)
    int32_t PR, PC;   // output patch per lane (rows x columns)
    int32_t S;        // stride
    int32_t TGX;      // lanes across a band; a wavefront covers 64/TGX bands
    bool dense;       // nine taps, every kernel present
    bool double_window;   // two sets of window registers: the next channel's window loads early
    bool threaded;        // every code block jumps straight to the next kernel's block
    bool experimental;    // not yet measured on hardware: never chosen by default or by the tuner
    int32_t mode;         // MODE bits: 0-3 the interpreter's (gen_dispatch.py), 4 one staging buffer
    int32_t lds_buffers;  // staging buffers of `ck` channels each (1 or 2)
    int32_t lds_floats_per_channel;   // LDS floats one staged channel takes
    int32_t stage_elems;              // elements staged per channel (without bank padding)
    int32_t max_slots;                // staging elements per thread the kernel can hold
    // code-table geometry of the step interpreter (sparse variants)
    uint32_t block_bytes;             // size of one (set, slot, pattern) block
    uint32_t table_off;               // offset of block 0 from the code base
    uint32_t ctrl_bytes;              // control block k sits at k*ctrl_bytes
    uint32_t records;                 // kernels per step
    // ksplit > 1 (sparse variants): slices of the input channels on gridDim.y.  `scratch` (DEVICE,
    // 16-byte aligned, `scratch_floats` floats, may be NULL): with room for ksplit buffers of
    // split_slice_stride([n][c_out][ho][wo]) floats every slice stores its partial sums to its
    // own buffer and a finishing kernel adds them up; otherwise the slices are summed with
    // atomics, in the output or - with fused pooling, which then needs [n][c_out][ho][wo]
    // floats of scratch - in `scratch`, and a finishing kernel writes the pooled output.
    hipError_t (*launch)(const DevTiled&, const ConvShape&, const float*, const float*, float*,
                         int32_t waves, int32_t ksplit, float* scratch, size_t scratch_floats, hipStream_t);
};

// Tap-product layout on the device (layout.hpp, Taps).
struct DevTaps {
    int32_t num_groups = 0, ck = 0, num_chunks = 0;
    const int32_t* slot_channel = nullptr;
    const uint32_t* chunk_ptr = nullptr;
    const uint32_t* records = nullptr;
    const float* weights = nullptr;
};
// How an input is cut into tiles of 16 x 16 input pixels (14 x 14 outputs inside an image).
constexpr int kTile = 16, kTileOut = 14;
struct TapTiles {
    int32_t sx = 1, sy = 1, px = 0, py = 0;      // images side by side in a tile, and their pitch
    int32_t bx = 1, by = 1;                      // tiles per image (1 where sx, sy exceed 1)
};
inline TapTiles tap_tiles(const ConvShape& s)
{
    TapTiles t;
    auto side = [&](int size, int32_t& tiles, int32_t& images, int32_t& pitch) {
        const int used = size + s.pad;                // an image and the padding before it (the next one's is behind it)
        tiles = used <= kTile ? 1 : 1 + (used - kTile + kTileOut - 1) / kTileOut;
        pitch = used + (s.pool ? used & 1 : 0);       // pooling windows start at even rows and columns
        images = tiles == 1 ? std::max(1, (kTile + pitch - used) / pitch) : 1;
        if (images == 1) pitch = 2 * kTile;           // one image: never a second one
    };
    side(s.w, t.bx, t.sx, t.px);
    side(s.h, t.by, t.sy, t.py);
    return t;
}
inline long long tap_tile_count(const ConvShape& s)
{
    const TapTiles t = tap_tiles(s);
    return (long long)((s.n + t.sx * t.sy - 1) / (t.sx * t.sy)) * t.bx * t.by;
}
// Staging offsets are 32-bit byte offsets from the first image of a tile.
inline bool taps_fit_input(const ConvShape& s)
{
    const TapTiles t = tap_tiles(s);
    return (long long)t.sx * t.sy * s.c_in * s.h * s.w < (1ll << 30) && tap_tile_count(s) * ((s.c_out + 7) / 8) <= INT32_MAX;
}
// Stride 1 only; `filters` per wavefront is 2, 4, 8 or 16, the rest as TiledVariant::launch.
hipError_t launch_taps(int filters, const DevTaps& t, const ConvShape& s, const float* in, const float* bias, float* out,
                       int32_t waves, int32_t ksplit, float* scratch, size_t scratch_floats, hipStream_t stream);

// ---------------------------------------------------------------------------
// Launches that split the input channels: where the slices' partial sums go (before the slices
// run), and the kernel that makes the output of them (after).
// ---------------------------------------------------------------------------
struct SplitTarget {
    float* sums = nullptr;           // first buffer
    int slices = 1;                  // buffers, one per slice; 1 = the slices are added up in `sums` with atomics
    size_t slice_stride = 0;         // floats between the buffers
};
// With room for one buffer per slice the slices store their sums; otherwise they add into the
// output (pooled layers: into the scratch, which must hold one un-pooled output), cleared here.
hipError_t begin_split(const ConvShape& s, float* out, int32_t ksplit, float* scratch, size_t scratch_floats,
                       hipStream_t stream, SplitTarget& t);
// sum + bias + activation (+ pooling), and the zero fill handed over by s.zero_next
hipError_t finish_split(const ConvShape& s, const SplitTarget& t, const float* bias, float* out, hipStream_t stream);
// More than 64 KB of dynamic LDS: the function attribute, once per device.
hipError_t allow_big_lds(const void* fn, std::atomic<uint64_t>& done);

// Device check that s_movrels_b32 / _b64 behave as the threaded interpreter assumes.
bool movrel_selftest(std::string& err);

int num_tiled_variants();
const TiledVariant& tiled_variant(int i);

}  // namespace patdnn
