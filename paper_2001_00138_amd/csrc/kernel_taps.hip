// Tap-product kernel: pattern-sparse 3x3 convolution, stride 1, on the matrix cores in fp32.
//
// A kept kernel is four weights that all multiply the same input channel.  Seen from the input
// it is an outer product - four weights times the pixels - and v_mfma_f32_4x4x1_16b_f32 is
// exactly that for 64 pixels: one instruction does the 256 multiply-adds of a kernel on 64 pixels in
// 8 cycles, where v_fmac_f32 needs four instructions and 16 cycles.  No weight is stored for,
// or multiplied with, a position that pruning removed.  gen_taps.py has the inner loop and what
// becomes of the four tap sums.
//
// Work decomposition
//   * A tile is 16 x 16 input pixels of one image (a halo of one pixel on each side of 14 x 14
//     outputs; where the image ends inside the tile its zero padding lies there too, so images up
//     to 15 x 15 are one tile, and small images share a tile, separated by their padding).
//   * A wavefront computes one or two filter groups of eight filters, or a half or a quarter of one, on all 256
//     pixels: lane (q, column) owns rows 4q .. 4q+3.  A workgroup is up to 16 wavefronts that share the
//     tile and take consecutive groups.
//   * The tile's input channels are staged `ck` at a time in LDS, a channel as 64 x 16 bytes: the
//     lane's four rows side by side, one ds_read_b128 per kernel and lane.
//   * Output sums stay in registers over the chunks; each lane writes its own four rows.
//
// What bounds it (256 -> 256 at 56 x 56, 64 images, 550 us): the matrix cores are busy 46 % of the SIMDs'
// cycles, four instructions of 8 cycles for a kernel on 256 pixels (42 clocks with four wavefronts per
// SIMD); the adds of a flush (16, about 48 clocks with its jump, after every 4.4 kernels at 128 channels a
// chunk and a keep ratio of 1/3.6) and of the filters' ends take 18 to 36 %; a third of a wavefront's
// life is waiting.  15 of every 64 input pixels of an inner tile are halo (14 x 14 of 16 x 16).  A
// workgroup's own reads and writes are hidden only by another workgroup on its CU, so layers of few
// channels and large planes (64 -> 64 at 224 x 224: 0.80 ms for 64 images) are left to the tiled kernel
// (0.60).  Measured, the tiled kernel's best configuration -> this one: 512 -> 512 at 28 x 28, 64 images
// 0.67 -> 0.54 ms (54 TFLOP/s of kept weights), at 14 x 14 0.19 -> 0.15, at 7 x 7 0.098 -> 0.053; one
// image of 64 -> 64 at 224 x 224 35 -> 24 us, of 512 -> 512 at 14 x 14 28 -> 21 us (split).
//
// A small launch waits: a wavefront that has its SIMD to itself takes some 230 cycles a kernel, for pixels that are three
// kernels on their way and flushes with their jumps, one image of 512 -> 512 at 14 x 14 in 1024 wavefronts 7.8 of its 14
// us for 71 kernels each.  There the filters of a group go to two or four wavefronts, which have their pixels six kernels
// ahead (taps_parts in patdnn_api.hip): 20.5 -> 14.0 us with its finishing kernel, of 256 -> 256 at 56 x 56 31.6 -> 23.5, of 64 ->
// 64 at 224 x 224 23.2 -> 18.7.
#include <algorithm>
#include <atomic>

#include "kernels.hpp"
#include "layout.hpp"

namespace patdnn {

template <int F>
struct TapLoop;

#include "gen/taps_all.inc"

struct TapArgs {
    const float* in;
    const float* bias;
    float* out;
    const int32_t* slot_channel;
    const uint32_t* chunk_ptr;
    const uint32_t* records;
    const float* weights;
    int32_t n, c_in, c_out, h, w, ho, wo, pad, relu, pool;
    int32_t num_groups, ck, num_chunks, waves, fgsets;       // (waves of a workgroup)
    int32_t sx, sy, px, py;          // images side by side in a tile, and their pitch
    int32_t bx, by;                  // tiles per image (1 where sx, sy exceed 1)
    FastDiv div_fgsets, div_bx, div_by, div_px, div_py;
    size_t slice_stride;             // split launches: 0 = atomic adds into out, else slice y's own buffer
};

typedef __attribute__((address_space(3))) float lds_f32;

template <int F, bool SPLITK>
__global__ __launch_bounds__(1024) void tap_conv_kernel(TapArgs a)
{
    extern __shared__ float lds[];
    constexpr int NG = F > kTapGroup ? F / kTapGroup : 1;     // groups of a wavefront, or
    constexpr int PARTS = F < kTapGroup ? kTapGroup / F : 1;  // wavefronts of a group
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroups go to the 8 XCDs round-robin; give each XCD a contiguous range, so that the
    // workgroups that stage the same tile share an L2
    const int per_xcd = gridDim.x >> 3, rank = blockIdx.x >> 3;
    const int bid = rank < per_xcd ? (blockIdx.x & 7) * per_xcd + rank : blockIdx.x;
    const int tile = (int)fast_div((uint32_t)bid, a.div_fgsets);
    const int unit = (bid - tile * a.fgsets) * a.waves + wave;
    const int group0 = unit / PARTS * NG, part = unit % PARTS;
    const int t1 = (int)fast_div((uint32_t)tile, a.div_bx), tx = tile - t1 * a.bx;
    const int ig = (int)fast_div((uint32_t)t1, a.div_by), ty = t1 - ig * a.by;
    const int img0 = ig * a.sx * a.sy;
    const int plane = a.h * a.w;

    // ---- staging: lane (column, row of four) of load q fetches tile row 4q + lane % 4, column
    // lane / 4; byte offset from the tile's first image, ~0u (reads as zero) outside an image
    unsigned voff[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = 4 * q + (lane & 3), j = lane >> 2;
        const int si = (int)fast_div((uint32_t)i, a.div_py), sj = (int)fast_div((uint32_t)j, a.div_px);
        const int y = ty * kTileOut + i - si * a.py - a.pad, x = tx * kTileOut + j - sj * a.px - a.pad;
        const int img = si * a.sx + sj;
        const bool ok = si < a.sy && sj < a.sx && img0 + img < a.n && y >= 0 && y < a.h && x >= 0 && x < a.w;
        voff[q] = ok ? 4u * (unsigned)(img * a.c_in * plane + y * a.w + x) : ~0u;
    }
    const float* in_blk = a.in + (size_t)img0 * a.c_in * plane;
    const size_t blk_bytes = (size_t)(a.n - img0) * a.c_in * plane * 4;

    float o[F][4];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[f][r] = 0.0f;

    int chunk = 0, chunk_last = a.num_chunks;
    if constexpr (SPLITK) {
        const int k = (int)gridDim.y, y = (int)blockIdx.y;
        chunk = (int)((long long)a.num_chunks * y / k);
        chunk_last = (int)((long long)a.num_chunks * (y + 1) / k);
    }
    const unsigned lane_lds = 16u * lane;              // no static LDS: the chunk starts at LDS address 0
    for (; chunk < chunk_last; ++chunk) {
        const int c0 = chunk * a.ck, cn = min(a.ck, a.c_in - c0);
        __syncthreads();                              // everyone has left the previous chunk
        for (int c = wave; c < cn; c += a.waves) {
            const size_t skip = (size_t)(c0 + c) * plane * 4;
            const size_t left = blk_bytes - skip;
            const unsigned nrec = left > 0xFFFFFFFFull ? 0xFFFFFFFFu : (unsigned)left;
            __amdgpu_buffer_rsrc_t rsrc =
                __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)in_blk + skip), 0, (int)nrec, 0x00020000);
            lds_f32* dst = (lds_f32*)lds + c * (kTile * kTile);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst + 64 * q, 4, (int)voff[q], 0, 0, 0);
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);           // vmcnt(0)
        __syncthreads();
#pragma unroll 1
        for (int g = 0; g < NG; ++g) {
            if (group0 + g >= a.num_groups) break;
            typedef const uint32_t __attribute__((address_space(4))) * cptr;
            const size_t start = ((cptr)(uintptr_t)a.chunk_ptr)[((size_t)(group0 + g) * a.num_chunks + chunk) * kTapStarts + part * (kTapStarts / PARTS)];
            TapLoop<F>::run(o, lane_lds, a.records + start, a.weights + 4 * start, g * kTapGroup);
        }
    }

    // ---- epilogue: output row 4q + r, column `col` of the tile
    const int q = lane >> 4, col = lane & 15;
    const int sj = (int)fast_div((uint32_t)col, a.div_px);
    const int ox = tx * kTileOut + col - sj * a.px;
    // columns 14 and 15 of a tile are whole only where the image (and its padding) ends in it
    const bool col_ok = sj < a.sx && ox < a.wo && (col < kTileOut || tx == a.bx - 1);
    const size_t oplane = (size_t)a.ho * a.wo;
    int img[4], oy[4];
    bool ok[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 4 * q + r;
        const int si = (int)fast_div((uint32_t)i, a.div_py);
        oy[r] = ty * kTileOut + i - si * a.py;
        img[r] = img0 + si * a.sx + sj;
        ok[r] = col_ok && si < a.sy && img[r] < a.n && oy[r] < a.ho && (i < kTileOut || ty == a.by - 1);
    }
    float* const out = SPLITK ? a.out + (size_t)blockIdx.y * a.slice_stride : a.out;
    typedef const int32_t __attribute__((address_space(4))) * iptr;
    typedef const float __attribute__((address_space(4))) * fptr;
    if (!SPLITK && a.pool) {
        // the two rows of a pooling window are registers of one lane, its two columns neighbours
        const int pho = a.ho >> 1, pwo = a.wo >> 1;
        const size_t pplane = (size_t)pho * pwo;
#pragma unroll
        for (int f = 0; f < F; ++f) {
            if (group0 + f / kTapGroup >= a.num_groups) break;
            const int co = ((iptr)(uintptr_t)a.slot_channel)[(size_t)group0 * kTapGroup + part * F + f];
            if (co < 0) continue;
            const float b = a.bias ? ((fptr)(uintptr_t)a.bias)[co] : 0.0f;
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
                float m = fmaxf(o[f][r], o[f][r + 1]);
                m = fmaxf(m, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(m), 0xB1, 0xf, 0xf, true)));   // quad_perm [1,0,3,2]
                if (ok[r] && !(col & 1) && (oy[r] >> 1) < pho && (ox >> 1) < pwo)
                    out[((size_t)img[r] * a.c_out + co) * pplane + (size_t)(oy[r] >> 1) * pwo + (ox >> 1)] = fmaxf(m + b, 0.0f);
            }
        }
        return;
    }
    size_t off[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) off[r] = (size_t)img[r] * a.c_out * oplane + (size_t)oy[r] * a.wo + ox;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        if (group0 + f / kTapGroup >= a.num_groups) break;
        const int co = ((iptr)(uintptr_t)a.slot_channel)[(size_t)group0 * kTapGroup + part * F + f];
        if (co < 0) continue;
        float* dst = out + (size_t)co * oplane;
        const float b = !SPLITK && a.bias ? ((fptr)(uintptr_t)a.bias)[co] : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (!ok[r]) continue;
            if constexpr (SPLITK) {
                if (a.slice_stride) dst[off[r]] = o[f][r];
                else unsafeAtomicAdd(&dst[off[r]], o[f][r]);
            } else {
                const float v = o[f][r] + b;
                dst[off[r]] = a.relu ? fmaxf(v, 0.0f) : v;
            }
        }
    }
}

template <int F>
static hipError_t launch_taps_f(const DevTaps& t, const ConvShape& s, const float* in, const float* bias, float* out,
                                int32_t waves, int32_t ksplit, float* scratch, size_t scratch_floats, hipStream_t stream)
{
    TapArgs a{};
    a.in = in; a.bias = bias; a.out = out;
    a.slot_channel = t.slot_channel; a.chunk_ptr = t.chunk_ptr; a.records = t.records; a.weights = t.weights;
    a.n = s.n; a.c_in = s.c_in; a.c_out = s.c_out; a.h = s.h; a.w = s.w; a.ho = s.ho; a.wo = s.wo;
    a.pad = s.pad; a.relu = s.relu; a.pool = s.pool;
    a.num_groups = t.num_groups; a.ck = t.ck; a.num_chunks = t.num_chunks; a.waves = waves;
    a.fgsets = (t.num_groups * kTapGroup + waves * F - 1) / (waves * F);
    const TapTiles tiles = tap_tiles(s);
    a.sx = tiles.sx; a.sy = tiles.sy; a.px = tiles.px; a.py = tiles.py; a.bx = tiles.bx; a.by = tiles.by;
    a.div_fgsets = make_fast_div((uint32_t)a.fgsets);
    a.div_bx = make_fast_div((uint32_t)a.bx);
    a.div_by = make_fast_div((uint32_t)a.by);
    a.div_px = make_fast_div((uint32_t)a.px);
    a.div_py = make_fast_div((uint32_t)a.py);
    const long long blocks = tap_tile_count(s) * a.fgsets;
    if (blocks > INT32_MAX || waves < 1 || waves > 16 || t.ck < 1 || t.ck > kTapMaxChunk) return hipErrorInvalidValue;
    const size_t lds_bytes = (size_t)t.ck * kTile * kTile * sizeof(float);
    const bool split = ksplit > 1;
    if (lds_bytes > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0}, allowed_k{0};
        hipError_t e = split ? allow_big_lds(reinterpret_cast<const void*>(&tap_conv_kernel<F, true>), allowed_k)
                             : allow_big_lds(reinterpret_cast<const void*>(&tap_conv_kernel<F, false>), allowed);
        if (e != hipSuccess) return e;
    }
    if (!split) {
        hipLaunchKernelGGL((tap_conv_kernel<F, false>), dim3((unsigned)blocks), dim3(64 * waves), lds_bytes, stream, a);
        return hipGetLastError();
    }
    if (ksplit > t.num_chunks || ksplit > 65535) return hipErrorInvalidValue;
    SplitTarget target;
    hipError_t e = begin_split(s, out, ksplit, scratch, scratch_floats, stream, target);
    if (e != hipSuccess) return e;
    a.out = target.sums;
    a.slice_stride = target.slices > 1 ? target.slice_stride : 0;
    hipLaunchKernelGGL((tap_conv_kernel<F, true>), dim3((unsigned)blocks, (unsigned)ksplit), dim3(64 * waves), lds_bytes,
                       stream, a);
    return finish_split(s, target, bias, out, stream);
}

hipError_t launch_taps(int filters, const DevTaps& t, const ConvShape& s, const float* in, const float* bias, float* out,
                       int32_t waves, int32_t ksplit, float* scratch, size_t scratch_floats, hipStream_t stream)
{
    const auto launch = filters == 16 ? &launch_taps_f<16> : filters == 8 ? &launch_taps_f<8> : filters == 4 ? &launch_taps_f<4> : &launch_taps_f<2>;
    return launch(t, s, in, bias, out, waves, ksplit, scratch, scratch_floats, stream);
}

}  // namespace patdnn
