// 3x3 convolution on binary16 storage, on the matrix cores: the half-precision storage of the
// paper's GPU runs (section 6.1) for pruned and dense layers, stride 1 or 2.
//
// v_mfma_f32_32x32x16_f16 multiplies 32 filters x 16 input channels with 16 channels x 32
// pixels in 32 cycles: sixteen times the rate of the vector ALU.  That is more than the factor
// 8.1 of multiply-adds which connectivity and pattern pruning leave out (at a keep ratio of 1/3.6
// and four of nine taps), and a kept kernel by itself fills no matrix instruction.  The layer is
// therefore expanded once, at encode time, to all nine taps with zeros where pruning removed a
// weight, and runs as an implicit GEMM: products of binary16 values are exact, sums are fp32 as
// before, and a zero adds nothing.
//
// The one case where a zero weight is not nothing is an input that is infinite or NaN (0 * inf).
// Every output such an input reaches through any of the nine taps then has a sum that is not
// finite, so the wavefront looks at its sums once, at the end, and computes the blocks of pixels
// concerned again, from the tensor itself: in two accumulators whether an infinity or a NaN met a kept
// weight, and with which sign, and then the sum over the finite inputs (kept weights that
// are zero are stored as -0, so that they can be told from the removed ones).  Layers with a weight
// that is not finite in binary16 run the walk over the kept weights instead.
// 128 -> 128 at 56 x 56, 64 images: 76 us with finite inputs, 1060 with one infinity in ten thousand
// inputs, 1700 with nothing but NaN; one lane after the other walking the FKW arrays for its own
// pixels took 19400 and 23800, the walk over the whole layer takes 2000.
//
// Work decomposition
//   * Output columns are cut into strips of at most 32; the pixels of a strip are numbered
//     row after row through all images, and a tile is PIX consecutive ones: no tile is padded
//     out to an image's edge (the rows of all images, each with its zero padding, are
//     thought of as one tall image of vh rows each).  The strips of the same rows follow each other, so
//     that the cache lines at their common edges are fetched once: 64 -> 64 at 224x224, 64 images, seven
//     strips 613 -> 514 us, 128 -> 128 at 112x112 336 -> 305, at 56x56 102 -> 94 (before the loads were in flight
//     as they are now).
//   * A wavefront owns FM x PN blocks of 32 filters x 32 pixels; a workgroup WF x WP of
//     them, and WK wavefronts share a block and take 16 input channels each of a chunk of 16 * WK
//     (their sums meet in LDS): layers with few tiles.
//   * A chunk of the tile's input rows is staged in LDS as [8 channels][row][column] of
//     16 bytes, which is the order in which a lane wants its eight channels of a pixel; a
//     wavefront gathers 64 units x 8 channels at a time, zero where the image ends: a unit is a pair
//     of pixels (4-byte loads) where rows have an even length and start on whole pairs, else one pixel
//     (2-byte loads).  Two buffers, the next chunk's loads in flight while this one is computed; one
//     buffer where wavefronts split the channels, whose chunks are larger.
//     The loads are left as they come until they are put into LDS: packing them where they are issued waited for
//     memory once per unit (128 -> 128 at 56 x 56, 64 images 94 -> 81 us).
//   * Weights are read from L2 in fragment order, 16 bytes per lane, some taps ahead.  (Eight wavefronts on 128 filters x
//     512 pixels with each fragment brought into LDS once were even at 385 to 512 workgroups on resident tensors, 4 % ahead
//     on changing ones and for 512 channels, and 10 to 20 % slower at other numbers: 128 -> 128 at 56 x 56, 42 images 74 us
//     and 62, 84 images 110 and 92, 120 images 122 and 110.)
//   * Channel and bias of the filters wait in LDS for the epilogue, which waited for each in turn; its stores are 32-bit
//     offsets into a buffer that ends where the tensor does.
//
// What bounds it: 128 -> 128 at 56 x 56, 64 images (59 GFLOP with the zeros, 51 MB in and out) takes
// 72 us on changing tensors, 0.8 PFLOP/s, where the walk over the kept weights took 1990; one image of 256 -> 256
// at 28 x 28 7 us (57).  784 workgroups, two on a CU, are one and a half rounds, the matrix cores are busy 48 % of the SIMDs'
// cycles, LDS 28 % of the CUs', and a tile's first loads are hidden by nothing.  (Inputs two
// chunks ahead: 84 us; what is in flight is enough.)
#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>

#include "kernels.hpp"

namespace patdnn {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned short ushort8 __attribute__((ext_vector_type(8)));

struct F16Args {
    const __half* in;
    const float* bias;
    __half* out;
    const uint4* weights;            // fragments [filter block][channel step][tap][lane]
    const int32_t* reorder;          // stored filter -> channel
    int32_t n, c_in, c_out, h, w, ho, wo, conv_stride, pad, relu;
    int32_t vh, sw, strips, pitch, npp;      // rows per image, strip width, strips, staged columns, staged pixels / 64 * 64
    int32_t lead, pair_out;                  // columns staged before output column 0; output rows of aligned pairs
    int32_t steps, fblocks, fsets, tiles;    // channel steps of 16, filter blocks, filter sets, tiles of a strip
    int32_t pixels;                          // of a strip: n * ho * sw
    FastDiv div_fsets, div_strips, div_sw, div_ho, div_vh, div_pitch;
};

typedef const F16Args __attribute__((address_space(4))) * F16ArgsPtr;      // the kernel's own arguments

// Staging buffers: wavefronts that share a block stage so many channels that a second buffer would
// cost more workgroups per CU than it hides.
constexpr int f16_buffers(int wk) { return wk > 1 ? 1 : 2; }

// What a block of 32 filters x 32 pixels needs of eight inputs or weights (binary16 bits) where
// inputs are not finite.
struct NonFinite {
    half8 finite, any, sign;         // the values, 0 where not finite; 1 where not; +-1 for an infinity
};
static __device__ __forceinline__ NonFinite split_inputs(ushort8 x)
{
    ushort8 f, a, s;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const unsigned short b = x[j], e = b & 0x7FFF;
        f[j] = e >= 0x7C00 ? 0 : b;
        a[j] = e >= 0x7C00 ? 0x3C00 : 0;
        s[j] = e == 0x7C00 ? (b & 0x8000) | 0x3C00 : 0;
    }
    return {__builtin_bit_cast(half8, f), __builtin_bit_cast(half8, a), __builtin_bit_cast(half8, s)};
}
// 1 where a weight is kept; its sign, 0 for a kept zero (-0)
static __device__ __forceinline__ void split_weights(ushort8 w, half8& kept, half8& sign)
{
    ushort8 k, s;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const unsigned short b = w[j];
        k[j] = b ? 0x3C00 : 0;
        s[j] = b & 0x7FFF ? (b & 0x8000) | 0x3C00 : 0;
    }
    kept = __builtin_bit_cast(half8, k);
    sign = __builtin_bit_cast(half8, s);
}

// Products of eight channels and one tap at a time, over all channels: of the finite inputs (plain), or of
// what tells where inputs are not (up, down; see f16_again).
template <bool PLAIN>
static __device__ __forceinline__ void f16_walk(F16ArgsPtr a, __amdgpu_buffer_rsrc_t rsrc, unsigned image, const uint4* wt, int y, int x,
                                                float16v& up, float16v& down)
{
    const int plane = a->h * a->w;
#pragma unroll 1
    for (int step = 0; step < a->steps; ++step)
#pragma unroll 1
        for (int pos = 0; pos < 9; ++pos) {
            const int iy = y * a->conv_stride + pos / 3 - a->pad, ix = x * a->conv_stride + pos % 3 - a->pad;
            const bool inside = iy >= 0 && iy < a->h && ix >= 0 && ix < a->w;
            // past the last channel its weights are zeros of removed kernels, which meet nothing
            unsigned at = image + 2u * (unsigned)(step * 16 * plane + iy * a->w + ix);
            ushort8 bits;
            bool some = false;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                bits[j] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rsrc, inside ? (int)at : -1, 0, 0);
                at += 2u * (unsigned)plane;
                some |= (bits[j] & 0x7FFF) >= 0x7C00;
            }
            const NonFinite v = split_inputs(bits);
            const uint4 w = wt[(step * 9 + pos) * 64];
            if constexpr (PLAIN) {
                up = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, w), v.finite, up, 0, 0, 0);
            } else {
                if (!__any(some)) continue;
                half8 kept, sign;
                split_weights(__builtin_bit_cast(ushort8, w), kept, sign);
                up = __builtin_amdgcn_mfma_f32_32x32x16_f16(kept, v.any, up, 0, 0, 0);
                up = __builtin_amdgcn_mfma_f32_32x32x16_f16(sign, v.sign, up, 0, 0, 0);
                down = __builtin_amdgcn_mfma_f32_32x32x16_f16(kept, v.any, down, 0, 0, 0);
                down = __builtin_amdgcn_mfma_f32_32x32x16_f16(sign, -v.sign, down, 0, 0, 0);
            }
        }
}

// Blocks with a sum that is not finite (`odd`: a bit per block of the lane's pixels), once more; every
// wavefront of a block goes over all channels here.  Everything is worked out again from the kernel's
// arguments, read again, and one accumulator pair at a time, so that the kernel proper holds no register
// for it: the registers it needs decide how many wavefronts fit.
template <int FM, int PN, int WF, int WP, int WK>
static __device__ __forceinline__ void f16_again(unsigned odd, int wave)
{
    constexpr int PIX = 32 * PN * WP, RK = 16 / WK;
    F16ArgsPtr a = (F16ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    auto div = [](int n, const FastDiv __attribute__((address_space(4))) & d) { return (int)fast_div((uint32_t)n, FastDiv{d.m, d.shift}); };
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wk = wave % WK, wp = wave / WK % WP, wf = wave / (WK * WP);
    const int per_xcd = gridDim.x >> 3, rank = blockIdx.x >> 3;
    const int bid = rank < per_xcd ? (blockIdx.x & 7) * per_xcd + rank : blockIdx.x;
    const int tile_all = div(bid, a->div_fsets), fset = bid - tile_all * a->fsets;
    const int tile = div(tile_all, a->div_strips), strip = tile_all - tile * a->strips;
    const int pix0 = tile * PIX, last = min(pix0 + PIX, a->pixels) - 1;
    const int img0 = div(div(pix0, a->div_sw), a->div_ho);
    const int plane = a->h * a->w;
    const size_t oplane = (size_t)a->ho * a->wo, tail = (size_t)(a->n - img0) * a->c_in * plane * 2;
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(a->in + (size_t)img0 * a->c_in * plane), 0,
                                                                    (int)(unsigned)std::min<size_t>(tail, 0x80000000u), 0x00020000);
#pragma unroll 1
    for (int p = 0; p < PN; ++p) {
        const bool mine = odd >> p & 1;
        if (!__any(mine)) continue;
        const int q = min(pix0 + (wp * PN + p) * 32 + l32, last);
        const int row = div(q, a->div_sw), im = div(row, a->div_ho);
        const int y = row - im * a->ho, x = strip * a->sw + q - row * a->sw;
        const unsigned image = 2u * (unsigned)(((im - img0) * a->c_in + half * 8) * plane);
#pragma unroll 1
        for (int f = 0; f < FM; ++f) {
            const int block = (fset * WF + wf) * FM + f;
            if (block >= a->fblocks) break;
            const uint4* const wt = a->weights + (size_t)block * a->steps * (9 * 64) + lane;
            // `up` is positive where an infinity of positive product or a NaN met a kept weight, `down`
            // where one of negative product or a NaN did: sums of whole numbers that cancel exactly
            float16v up{}, down{};
            f16_walk<false>(a, rsrc, image, wt, y, x, up, down);
            unsigned plus = 0, minus = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                plus |= (unsigned)(up[r] > 0.0f) << r;
                minus |= (unsigned)(down[r] > 0.0f) << r;
            }
            float16v sum{};
            f16_walk<true>(a, rsrc, image, wt, y, x, sum, down);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                __builtin_amdgcn_sched_barrier(0);    // one store after the other
                const int s = block * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (mine && r / RK == (WK > 1 ? wk : 0) && s < a->c_out) {
                    const int co = a->reorder[s];
                    float v = sum[r];
                    if (minus >> r & 1) v = -__builtin_inff();
                    if (plus >> r & 1) v = minus >> r & 1 ? __builtin_nanf("") : __builtin_inff();
                    v += a->bias ? a->bias[co] : 0.0f;
                    if (a->relu) v = fmaxf(v, 0.0f);
                    a->out[((size_t)im * a->c_out + co) * oplane + (size_t)y * a->wo + x] = __float2half_rn(v);
                }
            }
        }
    }
}

// Wavefronts per SIMD that the registers of so many blocks allow.  Said to the compiler, which would
// otherwise save registers for more and wait for every load of the channel loop by itself (10 to 15 % on the
// splitting shapes).
constexpr int f16_waves(int blocks, bool most) { return blocks >= 8 ? 2 : blocks >= 4 ? 3 : !most ? 2 : blocks >= 2 ? 5 : 6; }

// Taps whose weights are on their way, as the registers allow.
constexpr int f16_hold(int blocks, int wk) { return wk > 1 ? 9 : blocks >= 4 ? 3 : 4; }

// Staging units whose loads are in flight while a chunk is computed: what the smaller tiles have for a wavefront, since
// those out of range cost as much as the others (four pairs, six pixels where wavefronts split the channels: 20 images of
// 200 -> 60 at 25 x 25 33 us for 22, 52 of 453 -> 108 at 16 x 16 46 for 33, 22 of 151 -> 260 at 24 x 26 30 for 22), and with two
// blocks, nine taps' weights and more of them a SIMD holds two wavefronts for three (28 of 280 -> 78 at 23 x 23 33 us for 28).
constexpr int f16_ahead(int blocks, int wk, bool pair) { return pair || (wk == 4 && blocks == 2) ? 2 : 4; }
// Where those that a wavefront does not have are branched around (20 images of 29 -> 239 at 36 x 36 15.6 us for 16.1, 20 of
// 32 -> 56 at 79 x 79 16.8 for 19.2; the others are slower for it: the loads of large tiles would end in the branches).
constexpr bool f16_branches(int blocks, int wk) { return wk == 1 && blocks == 2; }

// PAIR: rows of whole aligned pairs of pixels (see f16_tiles): staged two pixels per load, and
// stored two pixels at a time where the output's rows are the same.  FAR: a tile's outputs reach 2^30 elements past its
// first image's first one (3 -> 64 at 4200 x 4200), stores are through 64-bit addresses.
template <int FM, int PN, int WF, int WP, int WK, bool PAIR, bool FAR>
__global__ __launch_bounds__(64 * WF * WP * WK) __attribute__((amdgpu_waves_per_eu(f16_waves(FM * PN, false), f16_waves(FM * PN, true))))
void f16_conv_kernel(F16Args a)
{
    extern __shared__ uint4 lds4[];
    constexpr int WAVES = WF * WP * WK, PIX = 32 * PN * WP, G8 = 2 * WK;
    constexpr int UPX = PAIR ? 2 : 1, AHEAD = f16_ahead(FM * PN, WK, PAIR), BUFS = f16_buffers(WK);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave % WK, wp = wave / WK % WP, wf = wave / (WK * WP);
    // each XCD works on a contiguous range: the workgroups that stage the same tile share an L2
    const int per_xcd = gridDim.x >> 3, rank = blockIdx.x >> 3;
    const int bid = rank < per_xcd ? (blockIdx.x & 7) * per_xcd + rank : blockIdx.x;
    const int tile_all = (int)fast_div((uint32_t)bid, a.div_fsets);
    const int fset = bid - tile_all * a.fsets;
    const int tile = (int)fast_div((uint32_t)tile_all, a.div_strips), strip = tile_all - tile * a.strips;
    const int pix0 = tile * PIX;

    auto split_row = [&](int q, int& img, int& oy, int& sx) {
        const int r = (int)fast_div((uint32_t)q, a.div_sw);
        sx = q - r * a.sw;
        img = (int)fast_div((uint32_t)r, a.div_ho);
        oy = r - img * a.ho;
    };
    int img0, oy0, sx0;
    split_row(pix0, img0, oy0, sx0);
    const int vrow0 = img0 * a.vh + oy0 * a.conv_stride;
    const int plane = a.h * a.w;

    // ---- byte offset, from the tile's first image, of every staged pixel in its channel
    // (~0u: padding, reads as zero)
    const int last = min(pix0 + PIX, a.pixels) - 1;
    int img1, oy1, sx1;
    split_row(last, img1, oy1, sx1);
    // units (64 lanes) that this tile's rows take; the buffers are sized for the largest tile
    const int npb = (((img1 * a.vh + oy1 * a.conv_stride - vrow0 + 3) * a.pitch + 64 * UPX - 1) / (64 * UPX));
    unsigned* const voffs = reinterpret_cast<unsigned*>(lds4 + BUFS * G8 * a.npp);
    for (int e = threadIdx.x; e < npb * 64; e += 64 * WAVES) {
        const int rr = (int)fast_div((uint32_t)(e * UPX), a.div_pitch), cc = e * UPX - rr * a.pitch;
        const int v = vrow0 + rr, img = (int)fast_div((uint32_t)v, a.div_vh);
        const int y = v - img * a.vh - a.pad, x = strip * a.sw * a.conv_stride + cc - a.lead;
        const bool ok = img < a.n && y >= 0 && y < a.h && x >= 0 && x < a.w;
        voffs[e] = ok ? 2u * (unsigned)((img - img0) * a.c_in * plane + y * a.w + x) : ~0u;
    }

    // ---- this lane's pixels: where they lie in a staged group of eight channels (in 16-byte units)
    int base[PN];
#pragma unroll
    for (int p = 0; p < PN; ++p) {
        const int q = min(pix0 + (wp * PN + p) * 32 + l32, last);
        int img, oy, sx;
        split_row(q, img, oy, sx);
        base[p] = (img * a.vh + oy * a.conv_stride - vrow0) * a.pitch + sx * a.conv_stride + (a.lead - a.pad) + (2 * wk + half) * a.npp;
    }
    // channel and bias of the workgroup's filters, for the epilogue (which would wait for each by itself)
    const int behind = max(a.npp * (BUFS * G8 * 16 + 4), WK > 1 ? WAVES * 4096 : 0);
    int2* const slots = reinterpret_cast<int2*>(reinterpret_cast<char*>(lds4) + behind);
    for (int e = threadIdx.x; e < WF * FM * 32; e += 64 * WAVES) {
        const int s = fset * WF * FM * 32 + e;
        const int co = s < a.c_out ? a.reorder[s] : -1;
        slots[e] = make_int2(co, co >= 0 && a.bias ? __float_as_int(a.bias[co]) : 0);
    }
    int fb[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f) fb[f] = min((fset * WF + wf) * FM + f, a.fblocks - 1);

    float16v acc[FM][PN];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int p = 0; p < PN; ++p) acc[f][p] = float16v{};

    // ---- staging: unit u = 64 pixels (pairs) x 8 channels, units wave, wave + WAVES, ... of a chunk
    const int units = npb * G8;
    const size_t tail = (size_t)(a.n - img0) * a.c_in * plane * 2;
    const char* in_blk = (const char*)(a.in + (size_t)img0 * a.c_in * plane);
    // out of range (reads as zero) from the end of the tensor on, and for ~0u
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)in_blk, 0, (int)(unsigned)std::min<size_t>(tail, 0x80000000u), 0x00020000);
    // as loaded: whatever is done with them waits for them, so that is left to store_unit
    struct Unit { unsigned v[8]; };
    // unit u is block u / G8 of group u % G8
    auto load_unit = [&](int u, int off, int c0) __attribute__((always_inline)) -> Unit {
        const int cg = c0 + u % G8 * 8;
        Unit t;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // past the last channel its weights are zero; which pixel they meet does not matter
            const int soff = min(cg + j, a.c_in - 1) * plane * 2;
            if constexpr (PAIR) t.v[j] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, off, soff, 0);
            else t.v[j] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rsrc, off, soff, 0);
        }
        // the last load must not take the offset's register: that would part the eight loads (an s_nop between
        // them, 6 % on the splitting shapes of unpaired rows)
        asm volatile("" : : "v"(off));
        return t;
    };
    auto store_unit = [&](int u, int buf, const Unit& t) __attribute__((always_inline)) {
        uint4* dst = lds4 + (buf * G8 + u % G8) * a.npp + (u / G8 * 64 + lane) * UPX;
        const unsigned (&v)[8] = t.v;
        if constexpr (PAIR) {
            // low halves, then high halves, of two channels
            auto lo = [&](int j) { return __builtin_amdgcn_perm(v[j + 1], v[j], 0x05040100u); };
            auto hi = [&](int j) { return __builtin_amdgcn_perm(v[j + 1], v[j], 0x07060302u); };
            dst[0] = make_uint4(lo(0), lo(2), lo(4), lo(6));
            dst[1] = make_uint4(hi(0), hi(2), hi(4), hi(6));
        } else {
            dst[0] = make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16);
        }
    };
    __syncthreads();                                  // the offsets
    Unit ahead[AHEAD];
    unsigned off_ahead[AHEAD];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) off_ahead[k] = wave + k * WAVES < units ? voffs[(wave + k * WAVES) / G8 * 64 + lane] : ~0u;
    // where there is nothing more to fetch the loads are out of range
    auto fetch = [&](int c0) __attribute__((always_inline)) {
        const unsigned none = c0 < 16 * a.steps ? 0u : ~0u;
#pragma unroll
        for (int k = 0; k < AHEAD; ++k)
            if (!f16_branches(FM * PN, WK) || wave + k * WAVES < units) ahead[k] = load_unit(wave + k * WAVES, (int)(off_ahead[k] | none), c0);
    };
    // weights of a tap; loads come back in the order in which they were issued, so those of a step are all issued
    // before the next chunk's inputs, and the next step's first ones after them
    constexpr int HOLD = f16_hold(FM * PN, WK);
    half8 wv[9][FM];
    auto weights = [&](int step, int tap) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < FM; ++f)
            wv[tap][f] = __builtin_bit_cast(half8, a.weights[((size_t)fb[f] * a.steps + min(step, a.steps - 1)) * (9 * 64) + tap * 64 + lane]);
    };
    fetch(0);
#pragma unroll
    for (int tap = 0; tap < HOLD; ++tap) weights(wk, tap);
    int buf = 0;
    for (int c0 = 0; c0 < 16 * a.steps; c0 += 16 * WK) {
        if (BUFS == 1 && c0) __syncthreads();         // everyone has left the previous chunk
#pragma unroll
        for (int k = 0; k < AHEAD; ++k)
            if (wave + k * WAVES < units) store_unit(wave + k * WAVES, buf, ahead[k]);
        for (int u = wave + AHEAD * WAVES; u < units; u += WAVES) store_unit(u, buf, load_unit(u, (int)voffs[u / G8 * 64 + lane], c0));
        // with two buffers one barrier per chunk: whoever is past it has finished with the other one
        __syncthreads();
        const int step = (c0 >> 4) + wk;
        if (WK > 1 && step >= a.steps) break;         // only in the last chunk
        const uint4* src = lds4 + buf * G8 * a.npp;
        half8 x[PN];
        auto pixels = [&](int tap, int p) __attribute__((always_inline)) {
            x[p] = __builtin_bit_cast(half8, src[base[p] + tap / 3 * a.pitch + tap % 3]);
        };
        const bool more = c0 + 16 * WK < 16 * a.steps;
#pragma unroll
        for (int p = 0; p < PN; ++p) pixels(0, p);
        if (HOLD == 9 && more) fetch(c0 + 16 * WK);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
#pragma unroll
            for (int p = 0; p < PN; ++p) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int f = 0; f < FM; ++f) acc[f][p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wv[tap][f], x[p], acc[f][p], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (tap < 8) pixels(tap + 1, p);
            }
            if (tap + HOLD < 9) weights(step, tap + HOLD);
            else if (HOLD < 9) weights(step + WK, tap + HOLD - 9);
            __builtin_amdgcn_sched_barrier(0);
            if (tap + HOLD == 8) fetch(c0 + 16 * WK);
        }
        if (HOLD == 9 && more)
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) weights(step + WK, tap);
        if (BUFS == 2) buf ^= 1;
    }

    // ---- the wavefronts of a block add up their channels, in a fixed order; each keeps 16 / WK
    // of the registers of every block
    constexpr int RK = 16 / WK;
    if constexpr (WK > 1) {
        float* const sums = reinterpret_cast<float*>(lds4);
        __syncthreads();
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int p = 0; p < PN; ++p) {
                if (f + p) __syncthreads();
#pragma unroll
                for (int r = 0; r < 16; ++r) sums[(wave * 16 + r) * 64 + lane] = acc[f][p][r];
                __syncthreads();
#pragma unroll
                for (int r = 0; r < RK; ++r) {
                    float v = 0.0f;
#pragma unroll
                    for (int k = 0; k < WK; ++k) v += sums[((wave - wk + k) * 16 + wk * RK + r) * 64 + lane];
                    acc[f][p][r] = v;
                }
            }
    }

    // ---- epilogue: register r of a block is filter 8 * (r / 4) + 4 * half + r % 4, pixel lane % 32.  Byte offsets from
    // the tile's first image, those of pixels and filters that do not exist out of range whatever is added to them: no
    // branch and no 64-bit address a store (128 values a lane were 8 of a tile's 37 us at 128 -> 128, 6 of 15 at 24 -> 400).
    // us before -> after: 128 -> 128 at 56 x 56, 64 images 76 -> 72; 24 -> 400 at 46 x 33, 45 images 40 -> 32; 24 -> 408 at 51 x 69 45 -> 37;
    // 28 -> 416 at 193 x 224, 5 images 130 -> 120
    const size_t oplane = (size_t)a.ho * a.wo;
    const int reg0 = WK > 1 ? wk * RK : 0;
    const bool pair_out = PAIR && RK >= 2 && a.pair_out;
    float finite[PN];                                 // NaN where a sum is not
    unsigned off[PN];
    size_t pixel[PN];                                 // FAR: elements instead
    bool ok[PN];
#pragma unroll
    for (int p = 0; p < PN; ++p) {
        const int q = pix0 + (wp * PN + p) * 32 + l32;
        int img, oy, sx;
        split_row(min(q, last), img, oy, sx);
        const int ox = strip * a.sw + sx;
        ok[p] = q <= last && ox < a.wo;
        if constexpr (FAR) pixel[p] = (size_t)(img - img0) * a.c_out * oplane + (size_t)oy * a.wo + (ox - (pair_out ? lane & 1 : 0));
        off[p] = ok[p] ? 2u * ((unsigned)((img - img0) * a.c_out) * (unsigned)oplane + (unsigned)(oy * a.wo + ox - (pair_out ? lane & 1 : 0))) : 0x7FFFFFFFu;
        finite[p] = 0.0f;
    }
    const size_t out_tail = (size_t)(a.n - img0) * a.c_out * oplane * 2;
    __half* const out_blk = a.out + (size_t)img0 * a.c_out * oplane;
    __amdgpu_buffer_rsrc_t osrc = __builtin_amdgcn_make_buffer_rsrc((void*)out_blk, 0, (int)(unsigned)std::min<size_t>(out_tail, 0x7FFFFFFFu), 0x00020000);
    const float least = a.relu ? 0.0f : __builtin_nanf("");      // the maximum of a value and a NaN is the value
    // neighbouring pixels trade: the even one takes both of filter r, the odd one both of r + 1
    const unsigned trade = lane & 1 ? 0x03020706u : 0x05040100u;
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int r = 0; r < RK; r += 2) {
            int channel[2];
            unsigned co[2];
            float b[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int2 slot = slots[(wf * FM + f) * 32 + 8 * ((reg0 + r + k) >> 2) + 4 * half + ((reg0 + r + k) & 3)];
                channel[k] = slot.x;
                co[k] = slot.x >= 0 ? 2u * (unsigned)slot.x * (unsigned)oplane : 0x80000000u;
                b[k] = __int_as_float(slot.y);
            }
#pragma unroll
            for (int p = 0; p < PN; ++p) {
                __half v[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const float sum = acc[f][p][r + k];
                    finite[p] = fmaf(sum, 0.0f, finite[p]);
                    v[k] = __float2half_rn(fmaxf(sum + b[k], least));
                }
                if (pair_out) {
                    const unsigned mine = (unsigned)__half_as_ushort(v[0]) | (unsigned)__half_as_ushort(v[1]) << 16;
                    const unsigned next = (unsigned)__builtin_amdgcn_mov_dpp((int)mine, 0xB1, 0xf, 0xf, true);      // quad_perm [1,0,3,2]
                    const unsigned both = __builtin_amdgcn_perm(next, mine, trade);
                    if constexpr (FAR) {
                        const int c = lane & 1 ? channel[1] : channel[0];
                        if (ok[p] && c >= 0) *reinterpret_cast<unsigned*>(out_blk + pixel[p] + (size_t)c * oplane) = both;
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b32(both, osrc, (int)(off[p] + (lane & 1 ? co[1] : co[0])), 0, 0);
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        if constexpr (!FAR) __builtin_amdgcn_raw_buffer_store_b16((short)__half_as_ushort(v[k]), osrc, (int)(off[p] + co[k]), 0, 0);
                        else if (ok[p] && channel[k] >= 0) out_blk[pixel[p] + (size_t)channel[k] * oplane] = v[k];
                }
            }
        }
    unsigned odd = 0;                                 // pixels of this lane with a sum that is not finite
#pragma unroll
    for (int p = 0; p < PN; ++p) odd |= (unsigned)(ok[p] && finite[p] != 0.0f) << p;
    if (!__any(odd)) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // after the stores above, the neighbour's among them
    f16_again<FM, PN, WF, WP, WK>(odd, wave);
}

// One workgroup per stored filter: its kept weights to their places in the fragments, zeros as -0
// (removed ones stay +0).
__global__ __launch_bounds__(256) void f16_expand_kernel(const int32_t* offset, const int32_t* index, const int32_t* stride,
                                                         const __half* weight, const uint16_t* masks, int num_patterns,
                                                         int taps, int steps, __half* out)
{
    const int s = blockIdx.x;
    const int32_t* st = stride + (size_t)s * (num_patterns + 1);
    const int32_t k0 = offset[s], kn = offset[s + 1] - k0;
    for (int32_t k = threadIdx.x; k < kn; k += 256) {
        int p = 0;
        while (k >= st[p + 1]) ++p;
        unsigned m = masks[p];
        const int c = index[k0 + k];
        for (int t = 0; t < taps; ++t) {
            const int pos = __builtin_ctz(m);
            m &= m - 1;
            const size_t frag = ((size_t)(s >> 5) * steps + (c >> 4)) * 9 + pos;
            const unsigned short b = __half_as_ushort(weight[(size_t)(k0 + k) * taps + t]);
            out[(frag * 64 + ((c >> 3) & 1) * 32 + (s & 31)) * 8 + (c & 7)] = __ushort_as_half(b & 0x7FFF ? b : 0x8000);
        }
    }
}

size_t f16_expanded_halves(int32_t c_in, int32_t c_out)
{
    return (size_t)((c_out + 31) / 32) * ((c_in + 15) / 16) * 9 * 64 * 8;
}

hipError_t launch_f16_expand(const DevFkw& f, int32_t c_in, int32_t c_out, void* out, hipStream_t stream)
{
    hipLaunchKernelGGL(f16_expand_kernel, dim3((unsigned)c_out), dim3(256), 0, stream, f.offset, f.index, f.stride,
                       static_cast<const __half*>(f.weight_f16), f.masks, f.num_patterns, f.taps, (c_in + 15) / 16,
                       static_cast<__half*>(out));
    return hipGetLastError();
}

// How the pixels of an output are cut into tiles of `pix`; false where the kernel's 32-bit numbers
// do not reach.  `far`: see f16_conv_kernel.
static bool f16_tiles(const ConvShape& s, int pix, bool pair, F16Args& a, bool& far)
{
    a.strips = (s.wo + 31) / 32;
    a.sw = (s.wo + a.strips - 1) / a.strips;
    a.vh = s.h + 2 * s.pad;
    a.lead = s.pad;
    a.pitch = (a.sw - 1) * s.stride + 3;
    if (pair) {
        // strips and staged rows start at even columns
        a.sw = (a.sw + 1) / 2 * 2;
        a.lead = 2 * s.pad;
        a.pitch = ((a.sw - 1) * s.stride + 3 + s.pad + 1) / 2 * 2;
    }
    const long long pixels = (long long)s.n * s.ho * a.sw;
    if (pixels > INT32_MAX - pix || (long long)s.n * a.vh > INT32_MAX) return false;
    a.pixels = (int32_t)pixels;
    a.tiles = (int32_t)((pixels + pix - 1) / pix);
    // rows under a tile: of the output rows that `pix` pixels touch, and what lies between images
    const int rows_out = (int)std::min<long long>((pix - 1 + a.sw - 1) / a.sw + 1, (long long)s.n * s.ho);
    const int between = std::min(s.n - 1, (rows_out - 1 + s.ho - 1) / s.ho);
    const int rows = (rows_out - 1) * s.stride + between * (a.vh - s.ho * s.stride) + 3;
    a.npp = (rows * a.pitch + 127) / 128 * 128;
    // byte offsets from a tile's first image; its outputs lie in at most between + 1 images
    far = (long long)(between + 1) * s.c_out * s.ho * s.wo >= (1ll << 30);
    return (long long)(between + 2) * s.c_in * s.h * s.w < (1ll << 30);
}

template <int FM, int PN, int WF, int WP, int WK, bool PAIR, bool FAR>
static hipError_t launch_f16_t(const F16Args& args, const ConvShape& s, long long blocks, size_t lds, hipStream_t stream)
{
    F16Args a = args;
    a.div_fsets = make_fast_div((uint32_t)a.fsets);
    a.div_strips = make_fast_div((uint32_t)a.strips);
    a.div_sw = make_fast_div((uint32_t)a.sw);
    a.div_ho = make_fast_div((uint32_t)a.ho);
    a.div_vh = make_fast_div((uint32_t)a.vh);
    a.div_pitch = make_fast_div((uint32_t)a.pitch);
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};
        hipError_t e = allow_big_lds(reinterpret_cast<const void*>(&f16_conv_kernel<FM, PN, WF, WP, WK, PAIR, FAR>), allowed);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((f16_conv_kernel<FM, PN, WF, WP, WK, PAIR, FAR>), dim3((unsigned)blocks), dim3(64 * WF * WP * WK), lds, stream, a);
    return hipGetLastError();
}

// The compiled shapes, in the order in which they are tried: the first that gives the chip
// `min_blocks` workgroups.  Large blocks read every staged pixel and weight for more
// multiply-adds, small ones reach more CUs, and wavefronts that split the channels shorten
// the chain of the last layers of a network.  us per pass, largest to smallest shape (f2 p4, f2 p2,
// f1 p2, then the splitting ones):
//   128 -> 128 at 56x56, 64 images     94   99  103  147  188  232     (784 workgroups of the first; 78 since the loads are in
//                                                                       flight and the epilogue does not wait)
//    64 ->  64 at 112x112, 8 images    32   34   23   29   34   57     (784 of the third; half of the first idle)
//   128 -> 256 at 56x56 / 2, 16 images 37   32   47   58   83   --     (196 of the second)
//   512 -> 512 at 7x7, 64 images      136  146   95   52   68   69     (784 of the fourth)
//   256 -> 256 at 28x28, one image     47   42   28   12    9    9     (200 of the fifth and sixth)
//   512 -> 512 at 14x14, one image     81   75   50   21   22   16     (112)
//   328 -> 256 at 32x47, 5 images      58   46   37   43   53   50     (240 of the third)
//    89 ->  62 at 120x120, 2 images    23   17   13   17   24   23     (226)
//    32 -> 108 at 58x58 / 2, 17 images 17   12    9   19   --   28     (224)
struct F16Shape {
    int fm, pn, wf, wp, wk, min_blocks;
    bool strided;                    // only where every filter set's staging counts four times: stride 2
    hipError_t (*launch[2][2])(const F16Args&, const ConvShape&, long long, size_t, hipStream_t);       // far or not, pairs or not
};
// (outputs that need FAR are more than a hundred thousand workgroups of any of the shapes that do not split the channels)
#define PATDNN_F16(fm, pn, wf, wp, wk, min_blocks, strided) \
    {fm, pn, wf, wp, wk, min_blocks, strided, {{&launch_f16_t<fm, pn, wf, wp, wk, false, false>, &launch_f16_t<fm, pn, wf, wp, wk, true, false>}, \
                                               {&launch_f16_t<fm, pn, wf, wp, wk, false, wk == 1>, &launch_f16_t<fm, pn, wf, wp, wk, true, wk == 1>}}}
static const F16Shape kF16Shapes[] = {
    PATDNN_F16(2, 4, 2, 2, 1, 256, false),
    PATDNN_F16(2, 2, 2, 2, 1, 128, true),
    PATDNN_F16(1, 2, 1, 4, 1, 224, false),
    PATDNN_F16(1, 2, 1, 1, 4, 400, false),
    PATDNN_F16(1, 1, 1, 1, 8, 0, false),
    PATDNN_F16(1, 1, 1, 1, 4, 0, false),
};
#undef PATDNN_F16

// The shape that a launch takes, as an index of kF16Shapes (-1: beyond the kernel's 32-bit numbers).
struct F16Plan {
    int shape = -1;
    bool far = false;
    long long blocks = 0;
    size_t lds = 0;
};
static F16Plan f16_plan(const ConvShape& s, bool pair, F16Args& a)
{
    F16Plan plan;
    a.steps = (s.c_in + 15) / 16;
    a.fblocks = (s.c_out + 31) / 32;
    for (const F16Shape& v : kF16Shapes) {
        const int filters = v.fm * v.wf;
        if (filters >= 2 * a.fblocks) continue;                   // half of every workgroup idle
        if (v.strided && s.stride == 1) continue;
        if (v.wk == 8 && a.steps <= 4) continue;                  // four wavefronts hold all channels
        if (!f16_tiles(s, 32 * v.pn * v.wp, pair, a, plan.far) || (plan.far && v.wk > 1)) continue;
        a.fsets = (a.fblocks + filters - 1) / filters;
        plan.blocks = (long long)a.strips * a.tiles * a.fsets;
        plan.lds = std::max((size_t)a.npp * (f16_buffers(v.wk) * 2 * v.wk * 16 + 4), v.wk > 1 ? (size_t)v.wf * v.wp * v.wk * 4096 : 0) + (size_t)filters * 32 * 8;
        if (&v == kF16Shapes) {
            // Staged rows that leave a CU one workgroup of the first shape: the next one's are half of that (stride 2; 447 ->
            // 424 at 106 x 95, 9 images 249 us and 142, 39 -> 421 at 79 x 121, 24 images 95 and 65, 449 -> 264 at 163 x 224, 4 images 222
            // and 182).
            if (plan.lds > 80 * 1024) continue;
            // Filters that fill its sets badly: the third shape has sets of 32 filters and twice the workgroups a CU, each
            // of which takes 1.75 / 4 times as long per round, less with up to three channel steps.  What a launch has of an
            // unfinished round counts in part, most in the first.  us of the first and the third shape: 208 -> 272 at 32 x 32, 24
            // images 50.0 and 42.5, 48 -> 133 at 65 x 64, 16 images 30.8 and 23.8, 40 -> 88 at 54 x 55, 50 images 31.1 and 30.5; 48 -> 200 at 224
            // x 208, 4 images 56 and 78, 159 -> 272 at 66 x 66, 60 images 248 and 409.  Of 963 layers of 40 to 512 channels 233 are
            // taken, 7 % faster on average and 32 more than 3 % slower.  Layers of fewer channels stay with the first shape, as before there was
            // a rule: for 73 of 266 this one would save 10 %.
            const auto rounds = [](double n) {
                const double open = n <= 1 ? 0.6 : n <= 2 ? 0.3 : 0.1;
                return (1 - open) * n + open * std::ceil(n);
            };
            const double sets = (double)a.strips * a.tiles, part = a.steps > 3 ? 1.75 : pair ? 1.38 : 1.55;     // (both: tiles of 256 pixels)
            if (s.stride == 1 && s.c_in >= 40 && rounds(sets * a.fblocks / 1024) * part / 2 < rounds(sets * a.fsets / 512)) continue;
        }
        // (with so few channels to split that the wavefronts of the next shapes have one step each, a little earlier)
        const int least = &v == kF16Shapes + 2 && a.steps <= 4 ? 192 : v.min_blocks;
        if (plan.blocks < least || plan.blocks > INT32_MAX || plan.lds > 160 * 1024) continue;
        plan.shape = (int)(&v - kF16Shapes);
        break;
    }
    return plan;
}

// two pixels per load: rows of an even length and a 4-byte aligned tensor
static bool f16_pair(const ConvShape& s, const void* in) { return s.w % 2 == 0 && (reinterpret_cast<uintptr_t>(in) & 3) == 0; }

int f16_choice(const ConvShape& s, const void* in)
{
    F16Args a{};
    const bool pair = f16_pair(s, in);
    const int shape = f16_plan(s, pair, a).shape;
    return shape < 0 ? -1 : 2 * shape + pair;
}

hipError_t launch_f16(const DevFkw& f, const ConvShape& s, const void* in, const float* bias, void* out, hipStream_t stream)
{
    F16Args a{};
    a.in = static_cast<const __half*>(in); a.bias = bias; a.out = static_cast<__half*>(out);
    a.weights = static_cast<const uint4*>(f.expanded_f16);
    a.reorder = f.reorder;
    a.n = s.n; a.c_in = s.c_in; a.c_out = s.c_out; a.h = s.h; a.w = s.w; a.ho = s.ho; a.wo = s.wo;
    a.conv_stride = s.stride; a.pad = s.pad; a.relu = s.relu;
    // two pixels per store likewise
    a.pair_out = s.wo % 2 == 0 && (reinterpret_cast<uintptr_t>(out) & 3) == 0;
    const bool pair = f16_pair(s, in);
    const F16Plan plan = f16_plan(s, pair, a);
    if (plan.shape < 0) return launch_fkw_f16(f, s, in, bias, out, stream);
    return kF16Shapes[plan.shape].launch[plan.far][pair](a, s, plan.blocks, plan.lds, stream);
}

}  // namespace patdnn
