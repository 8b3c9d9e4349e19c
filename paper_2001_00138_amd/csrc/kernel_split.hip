// fp32 layers on the binary16 matrix cores: pruned layers, stride 1 or 2.
//
// An fp32 number is the sum of two binary16 numbers to within its last bit: 11 bits, and 11 bits of what
// is left, which are kept multiplied with 2^11 so that they have the same range.  Of the product of two such
// pairs three parts matter,
//     w x = w.high x.high + (w.high x.low + w.low x.high) / 2^11,
// each exact in fp32, and v_mfma_f32_16x16x32_f16 does 8192 of their multiply-adds in 16 cycles where the vector
// ALU does 64 in 4: even with the removed weights as zeros (a layer is expanded to all nine taps at encode time)
// and three products for one that is less work than the vector kernels' for layers that keep half of their kernels,
// and at stride 2, where those leave lanes idle.
//
// Range: each filter's weights are scaled to 2^14 .. 2^15 once, at encode time, and a tile's inputs to at most
// 2^15 as they come in, both by powers of two; sums are rescaled when later channels need it.  A scaled input of
// 2^-14 and more (some 2^-28 of the largest one beside it) keeps its 22 bits, smaller ones are off by up to 2^-36: a
// tile has one scale for pixels, channels and images that have nothing to do with each other.  The wavefronts that
// stage mark the pixels of such inputs, and where sums over marked pixels are so small that it could be seen in
// them (more than 2^-24 of the sum), they are worked out again in fp32 (see split_again).  128 -> 128 at 56 x 56 / 2, 64
// images: 87 us for normal numbers through a ReLU, 85 for three times normal ones through a GELU (marked pixels in every
// tile), 400 with one value of -1e30 in every image, 520 where all is worked out again (the stride-2 kernel: 100).
//
// Work decomposition
//   * Pixels are cut into strips, rows and tiles as in kernel_f16.hip; two rows are numbered together
//     where windows are pooled, so that a window lies in four neighbouring lanes.
//   * A workgroup is eight wavefronts, two per SIMD, and goes on to further tiles.  Four compute 64 filters x 64
//     (or 32) pixels each, four (or eight) stage the inputs: the loads of one step of 32 channels are in flight, the
//     largest magnitude of the next is found, and the one after it is split and put into LDS, while the matrix
//     cores work on a fourth; a barrier per step.  The matrix instructions leave the vector ALU to the other wavefront, and
//     loads of weights (from L2 in fragment order, a tap ahead) do not wait behind those of the inputs.
//   * The sums of a step's 32 channels start from zero and join those of the steps before at its end: fewer roundings
//     at the size of the whole (128 -> 128 at 56 x 56 / 2, kept 1/3.6: error against 64 bits 11.2e-8, 15.1e-8 in one sum;
//     98 -> 101 us on changing tensors).  Nine taps of 32 filters, then nine of the other 32, so that only half of
//     the step's sums are held.
//   * Sums that are not finite, or too small for the scale, are worked out again from the tensor (see split_again).
//
// What bounds it, 128 -> 128 at 56 x 56 / 2, 64 images: the tiles of 64 pixels that its strips allow are 784 units of work,
// three rounds of 256 CUs and a fourth of 16; a step of 32 channels takes 4.6 us while others are staged,
// 3.0 without, 1.4 of them matrix instructions: weights, 288 KB a step and CU through L1, and inputs share the texture
// addresser.  (LDS is busy 28 % of the cycles, half of that conflicts of windows two pixels apart; a layout
// without them is no faster.)  us, the vector kernels' -> this one's, on tensors in the last-level cache: that layer, kept
// 1/3.6, 99 -> 87 (114 -> 97 on changing ones); 256 -> 256 at 28 x 28 / 2 196 -> 74; 64 -> 64 at 112 x 112 / 1, 32 images, all kept
// 200 -> 124; 232 -> 96 at 95 x 95 / 2, three images, all kept 428 -> 46.
#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <iterator>

#include "kernels.hpp"

namespace patdnn {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef unsigned split_u2 __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));

struct SplitArgs {
    const float* in;
    const float* bias;
    float* out;
    const uint4* weights;            // fragments [64 filters][channel step][tap][16 of the filters][high, low][lane]
    const int2* filters;             // stored filter, to whole blocks of 64: channel (-1: none), power of two its weights were multiplied with (kSplitEmpty: it has none)
    float seen;                      // a sum over marked pixels may be that small (see split_filters)
    int32_t n, c_in, c_out, h, w, ho, wo, conv_stride, pad, relu, pool;
    int32_t vh, sw, strips, pitch, lead, npp, npb;       // rows per image, strip width, strips, staged columns, those before output column 0, staged pixels of a buffer, units of them
    int32_t rp, hr;                              // rows that are numbered together (2: pooling windows), ho / rp
    int32_t steps, fblocks, fsets, tiles, total; // channel steps of 32, blocks of 64 filters, filter sets, tiles of a strip, units of work
    int32_t pixels;                              // of a strip: n * hr * rp * sw
    FastDiv div_fsets, div_strips, div_sw, div_hr, div_vh, div_pitch;
};

typedef const SplitArgs __attribute__((address_space(4))) * SplitArgsPtr;
static __device__ __forceinline__ SplitArgsPtr split_args()
{
    SplitArgsPtr a = (SplitArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return a;
}
static __device__ __forceinline__ int div_by(int n, const FastDiv __attribute__((address_space(4))) & d)
{
    return (int)fast_div((uint32_t)n, FastDiv{d.m, d.shift});
}

// A unit of work: a tile of PIX pixels of a strip and a set of filters.
struct SplitUnit {
    int fset, strip, pix0, last, img0, vrow0;
};
template <int PIX>
static __device__ __forceinline__ SplitUnit split_unit(SplitArgsPtr a, int u)
{
    SplitUnit t;
    const int tile_all = div_by(u, a->div_fsets);
    t.fset = u - tile_all * a->fsets;
    const int tile = div_by(tile_all, a->div_strips);
    t.strip = tile_all - tile * a->strips;
    t.pix0 = tile * PIX;
    t.last = min(t.pix0 + PIX, a->pixels) - 1;
    const int r = div_by(a->rp == 2 ? t.pix0 >> 1 : t.pix0, a->div_sw);
    t.img0 = div_by(r, a->div_hr);
    t.vrow0 = t.img0 * a->vh + (r - t.img0 * a->hr) * a->rp * a->conv_stride;
    return t;
}
// pixel q of a strip: rows are numbered one by one, or (rp = 2) two at a time, column by column
static __device__ __forceinline__ void split_pixel(SplitArgsPtr a, int q, int& img, int& oy, int& sx)
{
    const int sub = a->rp == 2 ? q & 1 : 0, qq = a->rp == 2 ? q >> 1 : q;
    const int r = div_by(qq, a->div_sw);
    sx = qq - r * a->sw;
    img = div_by(r, a->div_hr);
    oy = (r - img * a->hr) * a->rp + sub;
}

// Wavefronts that stage: each of the four eights of a step's channels has one, or two that take every other unit of
// its pixels.  Tiles of few pixels are taken where those pixels lie two apart and four wavefronts cannot stage
// as fast as the others compute; the third wavefront of a SIMD leaves each 168 registers, enough for two blocks of
// sums, but for 14 that are spilled (some eight reloads a step of 32 channels), and not for four.  us with 4 / 8, 64 images of stride 2: 256 -> 256 at 28 x 28 80.8 / 74.5, 512 -> 512 at 14 x 14
// 76.3 / 70.4, 128 -> 128 at 56 x 56, whose weights come as fast as L1 gives them, 88.1 / 88.6 (kept 1/3.6 each).
constexpr int split_stagers(int pn) { return pn == 2 ? 8 : 4; }
constexpr int split_threads(int pn) { return 64 * (4 + split_stagers(pn)); }

// units of 64 lanes x 8 channels that the wavefronts of eight channels hold per step, a lane with one pixel or a pair
constexpr int split_units(bool pair) { return pair ? 5 : 9; }
constexpr int kSplitTop = 13;        // exponent that the largest input of a tile is brought to
constexpr int kSplitMost = 14;       // up to which exponent later channels are taken as they are
constexpr int kSplitLeast = -14;     // below it an input has not all of its bits
constexpr int kSplitDrop = 64;       // a scale that falls by more might take earlier channels' sums out of range

// Pixels of a unit of work under which inputs lie below the scale: one byte for each staged pixel, and whether
// there are any, or every pixel counts as one.  Three units have theirs at a time: the one that is computed, the
// next, whose inputs are coming in, and the last, whose bytes are cleared.
constexpr int kSplitMarks = 3;
enum { kSplitSome = 1, kSplitAll = 2 };

// LDS behind the staging buffers: largest input of three chunks, kSplitSome / kSplitAll of three units, exponents
// of two chunks, marks of three units.
constexpr int split_lds(int npp) { return npp * (16 * 16 + kSplitMarks) + 32; }

// The scale of a tile's inputs, a power of two, as its channels come in (every staging wavefront keeps
// the same).
struct SplitScale {
    int sx = 0, first = 0;
    bool set = false;
    // `top`: bits of the largest magnitude of the channels to come
    __device__ __forceinline__ void next(unsigned top)
    {
        if (!top) return;
        const int e = max((int)(top >> 23), 1) - 127;
        if (!set || e + sx > kSplitMost) sx = min(kSplitTop - e, 127);
        if (!set) first = sx;
        set = true;
    }
    // twice the bits of the smallest magnitude that keeps its own, less one (see split_low)
    __device__ __forceinline__ unsigned least() const
    {
        const int e = kSplitLeast - sx + 127;
        return ((e > 0 ? (unsigned)e << 23 : 1u << (e + 22)) << 1) - 1;
    }
};
// Orders magnitudes, with zero as the largest.
static __device__ __forceinline__ unsigned split_low(float v) { return (__float_as_uint(v) << 1) - 1; }

// Two inputs as the high and the low parts of their products with m (a power of two): mixed-precision
// multiply-adds scale, round and pack at once.
static __device__ __forceinline__ void split_pair(float a, float b, float m, unsigned& high, unsigned& low)
{
    unsigned h, l;
    float ra, rb;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(a), "v"(m));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(b), "v"(m));
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(ra) : "v"(a), "v"(m), "v"(h));
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(rb) : "v"(b), "v"(m), "v"(h));
    const float up = 2048.0f;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(l) : "v"(ra), "v"(up));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(l) : "v"(rb), "v"(up));
    high = h;
    low = l;
}

// Largest of the wavefront, in lane 63 (values that order like unsigned numbers: magnitudes).
static __device__ __forceinline__ float split_wave_max(float v)
{
#define PATDNN_MAX(ctrl, rows) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xf, false)))
    PATDNN_MAX(0x111, 0xf);          // row_shr:1, 2, 4, 8
    PATDNN_MAX(0x112, 0xf);
    PATDNN_MAX(0x114, 0xf);
    PATDNN_MAX(0x118, 0xf);
    PATDNN_MAX(0x142, 0xa);          // row_bcast:15, 31
    PATDNN_MAX(0x143, 0xc);
#undef PATDNN_MAX
    return v;
}

// The largest of a pooling window, which lies in four neighbouring lanes.
static __device__ __forceinline__ float split_pool(float v)
{
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true)));   // quad_perm [1,0,3,2]
    return fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, true)));   // quad_perm [2,3,0,1]
}

// ---- blocks that are worked out again
// The inputs of eight channels and a tap.  Those that are not finite: 1 in `any`, +-1 in `sign` for an infinity, 0
// in `v`.
struct SplitInputs {
    half8 any, sign;
    bool some;
    float v[8];
};
static __device__ __forceinline__ SplitInputs split_inputs(const unsigned (&bits)[8])
{
    SplitInputs r;
    r.some = false;
    unsigned any[4] = {}, sign[4] = {};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const unsigned b = bits[j], e = b & 0x7FFFFFFFu;
        const bool odd = e >= 0x7F800000u;
        any[j >> 1] |= (odd ? 0x3C00u : 0u) << (j & 1) * 16;
        sign[j >> 1] |= (e == 0x7F800000u ? 0x3C00u | (b >> 16 & 0x8000u) : 0u) << (j & 1) * 16;
        r.some |= odd;
        r.v[j] = odd ? 0.0f : __uint_as_float(b);
    }
    r.any = __builtin_bit_cast(half8, make_uint4(any[0], any[1], any[2], any[3]));
    r.sign = __builtin_bit_cast(half8, make_uint4(sign[0], sign[1], sign[2], sign[3]));
    return r;
}

// Blocks of 16 pixels with a sum that is not finite or too small (`again`: a bit per block), once more from the
// tensor: the sum over the finite inputs in fp32 (the weights are put together again, the matrix
// instruction takes one channel of each quarter of the lanes), and in two sums of whole numbers whether an
// infinity or a NaN met a kept weight, and with which sign (kept zeros are -0 in the high part).  The loads of the
// next eight channels and tap are in flight meanwhile.
template <int PN, int WF, int WP>
static __device__ __forceinline__ void split_again(unsigned again, int u, int wave)
{
    constexpr int PIX = 16 * PN * WP;
    const SplitArgsPtr a = split_args();
    const int lane = threadIdx.x & 63, quarter = lane >> 4;
    const int wp = wave % WP, wf = wave / WP;
    const SplitUnit t = split_unit<PIX>(a, u);
    const int block = t.fset * WF + wf;
    if (block >= a->fblocks) return;
    const int plane = a->h * a->w;
    const size_t tail = (size_t)(a->n - t.img0) * a->c_in * plane * 4;
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(a->in + (size_t)t.img0 * a->c_in * plane), 0,
                                                                    (int)(unsigned)std::min<size_t>(tail, 0x80000000u), 0x00020000);
    const int oh = a->pool ? a->ho >> 1 : a->ho, ow = a->pool ? a->wo >> 1 : a->wo;
    const int last = a->steps * 9 - 1;
    int scale[4];                                     // of the filter whose weights this lane holds
#pragma unroll
    for (int f = 0; f < 4; ++f) scale[f] = -a->filters[block * 64 + f * 16 + (lane & 15)].y;
#pragma unroll 1
    for (int p = 0; p < PN; ++p) {
        if (!__any(again >> p & 1)) continue;
        const int q = t.pix0 + (wp * PN + p) * 16 + (lane & 15);
        int img, oy, px;
        split_pixel(a, min(q, t.last), img, oy, px);
        const int ox = t.strip * a->sw + px;
        bool ok = q <= t.last && ox < a->wo;
        if (a->pool) ok = ok && !(lane & 3) && (ox >> 1) < ow && (oy >> 1) < oh;
        const size_t at = (size_t)img * a->c_out * oh * ow + (size_t)(a->pool ? oy >> 1 : oy) * ow + (a->pool ? ox >> 1 : ox);
        float4v sum[4], up[4], down[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) sum[f] = up[f] = down[f] = float4v{};
        struct Loads {
            unsigned x[8];
            uint4 w[4][2];
        } next;
        // `i`: tap i % 9 of channel step i / 9
        const auto load = [&](int i) __attribute__((always_inline)) {
            const int step = i / 9, tap = i - step * 9;
            const int y = oy * a->conv_stride + tap / 3 - a->pad, x = ox * a->conv_stride + tap % 3 - a->pad;
            const int c = step * 32 + quarter * 8;
            const bool inside = y >= 0 && y < a->h && x >= 0 && x < a->w && c < a->c_in;
            const int off = inside ? 4 * (((img - t.img0) * a->c_in + c) * plane + y * a->w + x) : -1;
            const uint4* const wt = a->weights + ((size_t)block * a->steps * 9 + i) * (4 * 2 * 64) + lane;
#pragma unroll
            for (int j = 0; j < 8; ++j) next.x[j] = (unsigned)__builtin_amdgcn_raw_buffer_load_b32(rsrc, j < a->c_in - c ? off : -1, j * plane * 4, 0);
#pragma unroll
            for (int f = 0; f < 4; ++f)
#pragma unroll
                for (int k = 0; k < 2; ++k) next.w[f][k] = wt[(f * 2 + k) * 64];
        };
        load(0);
#pragma unroll 1
        for (int i = 0; i <= last; ++i) {
            const Loads now = next;
            load(min(i + 1, last));
            const SplitInputs in = split_inputs(now.x);
            const bool some = __any(in.some);
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                const half8 wh = __builtin_bit_cast(half8, now.w[f][0]), wl = __builtin_bit_cast(half8, now.w[f][1]);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float w = ldexpf(fmaf((float)wl[j], 1.0f / 2048.0f, (float)wh[j]), scale[f]);
                    sum[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, in.v[j], sum[f], 0, 0, 0);
                }
                if (!some) continue;
                // 1 where a weight is kept; its sign, 0 for a kept zero
                const unsigned word[4] = {now.w[f][0].x, now.w[f][0].y, now.w[f][0].z, now.w[f][0].w};
                unsigned k[4] = {}, g[4] = {};
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const unsigned b = word[j >> 1] >> (j & 1) * 16 & 0xFFFFu;
                    k[j >> 1] |= (b ? 0x3C00u : 0u) << (j & 1) * 16;
                    g[j >> 1] |= (b & 0x7FFFu ? 0x3C00u | (b & 0x8000u) : 0u) << (j & 1) * 16;
                }
                const half8 kept = __builtin_bit_cast(half8, make_uint4(k[0], k[1], k[2], k[3]));
                const half8 sign = __builtin_bit_cast(half8, make_uint4(g[0], g[1], g[2], g[3]));
                up[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kept, in.any, up[f], 0, 0, 0);
                up[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(sign, in.sign, up[f], 0, 0, 0);
                down[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kept, in.any, down[f], 0, 0, 0);
                down[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(sign, -in.sign, down[f], 0, 0, 0);
            }
        }
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = a->filters[block * 64 + f * 16 + quarter * 4 + r].x;
                float v = sum[f][r];
                if (down[f][r] > 0.0f) v = -__builtin_inff();
                if (up[f][r] > 0.0f) v = down[f][r] > 0.0f ? __builtin_nanf("") : __builtin_inff();
                v += a->bias ? a->bias[max(co, 0)] : 0.0f;
                if (a->pool) v = split_pool(v);
                if (a->relu) v = fmaxf(v, 0.0f);
                if (ok && co >= 0) a->out[at + (size_t)co * oh * ow] = v;
            }
    }
}

template <int PN, int WF, int WP, bool PAIR>
__global__ __launch_bounds__(split_threads(PN)) __attribute__((amdgpu_waves_per_eu(split_threads(PN) / 256, split_threads(PN) / 256)))
void split_conv_kernel(SplitArgs)
{
    extern __shared__ uint4 lds4[];
    constexpr int PARTS = split_stagers(PN) / 4;      // staging wavefronts of eight channels
    constexpr int PIX = 16 * PN * WP, UPX = PAIR ? 2 : 1, UNITS = (split_units(PAIR) + PARTS - 1) / PARTS;
    static_assert(WF * WP == 4, "four wavefronts compute");
    const int lane = threadIdx.x & 63, quarter = lane >> 4, l16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_xcd = gridDim.x >> 3, rank = blockIdx.x >> 3;
    const int u0 = rank < per_xcd ? (blockIdx.x & 7) * per_xcd + rank : blockIdx.x;
    SplitArgsPtr a = split_args();
    unsigned* const top_bits = reinterpret_cast<unsigned*>(lds4 + 16 * a->npp);       // see split_lds
    unsigned* const marked = top_bits + 3;
    int* const exps = reinterpret_cast<int*>(marked + kSplitMarks);
    unsigned char* const marks = reinterpret_cast<unsigned char*>(top_bits + 8);
    if (threadIdx.x < 3 + kSplitMarks) top_bits[threadIdx.x] = 0;
    for (int e = threadIdx.x; e < kSplitMarks * a->npp / 4; e += split_threads(PN)) reinterpret_cast<unsigned*>(marks)[e] = 0;
    __syncthreads();
    const int steps = a->steps;
    const int my_units = (a->total - u0 + (int)gridDim.x - 1) / (int)gridDim.x;
    const int chunks = my_units * steps;

    if (wave >= 4) {
        // ---- staging: of iteration g the inputs of chunk g + 1 into LDS, the loads of chunk g + 3, the largest
        // input of chunk g + 2; the smallest one beside zero stays with the lane until its chunk's scale is known
        const int w4 = wave & 3, part = (wave >> 2) - 1;
        auto unit = [&](int k) __attribute__((always_inline)) -> int { return k * PARTS + part; };
        const int plane = a->h * a->w, c_in = a->c_in, npp = a->npp;
        unsigned off[UNITS];
        const char* in_blk = nullptr;
        unsigned range = 0;
        auto enter = [&](int u) {
            const SplitArgsPtr b = split_args();
            const SplitUnit t = split_unit<PIX>(b, u);
            in_blk = (const char*)(b->in + (size_t)t.img0 * c_in * plane);
            const size_t tail = (size_t)(b->n - t.img0) * c_in * plane * 4;
            range = (unsigned)std::min<size_t>(tail, 0x80000000u);
#pragma unroll
            for (int k = 0; k < UNITS; ++k) {
                const int e = (unit(k) * 64 + lane) * UPX;
                const int rr = div_by(e, b->div_pitch), cc = e - rr * b->pitch;
                const int v = t.vrow0 + rr, img = div_by(v, b->div_vh);
                const int y = v - img * b->vh - b->pad, x = t.strip * b->sw * b->conv_stride + cc - b->lead;
                const bool ok = img < b->n && y >= 0 && y < b->h && x >= 0 && x < b->w;
                off[k] = ok ? 4u * (unsigned)((img - t.img0) * c_in * plane + y * b->w + x) : ~0u;
            }
        };
        const int units = (a->npb - part + PARTS - 1) / PARTS;   // this wavefront's: eight channels of each
        float raw[2][UNITS][UPX][8];
        unsigned low[2];
        int lu = u0, ls = 0;                          // what is loaded next
        auto load_unit = [&](float (&dst)[UPX][8], __amdgpu_buffer_rsrc_t rsrc, unsigned at, int c0) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                // past the last channel its weights are zero; which pixel they meet does not matter
                const int c = min(c0 + j, c_in - 1);
                if constexpr (PAIR) {
                    const split_u2 v = __builtin_bit_cast(split_u2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)at, c * plane * 4, 0));
                    dst[0][j] = __uint_as_float(v.x);
                    dst[1][j] = __uint_as_float(v.y);
                } else {
                    dst[0][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)at, c * plane * 4, 0));
                }
            }
        };
        SplitScale scale;
        int cs = 0, slot = kSplitMarks - 1;           // step of the chunk that is put into LDS next, marks of its unit
        // the scale of a chunk that is put into LDS, as a factor; marks its pixels
        auto begin_put = [&](int chunk, const float (&src)[UNITS][UPX][8], unsigned lowest) __attribute__((always_inline)) -> float {
            if (cs == 0) {
                scale = SplitScale{};
                slot = slot == kSplitMarks - 1 ? 0 : slot + 1;
            }
            if (++cs == steps) cs = 0;
            scale.next((unsigned)__builtin_amdgcn_readfirstlane((int)top_bits[chunk % 3]));
            if (threadIdx.x == 256) {
                exps[chunk & 1] = scale.sx;
                if (scale.first - scale.sx > kSplitDrop) atomicOr(&marked[slot], kSplitAll);
            }
            if (__any(lowest < scale.least())) {
                const unsigned least = scale.least();
#pragma unroll
                for (int k = 0; k < UNITS; ++k)
                    if (k < units)
#pragma unroll
                        for (int q = 0; q < UPX; ++q) {
                            unsigned v = ~0u;
#pragma unroll
                            for (int j = 0; j < 8; ++j) v = min(v, split_low(src[k][q][j]));
                            if (v < least) marks[slot * npp + (unit(k) * 64 + lane) * UPX + q] = 1;
                        }
                if (lane == 0) atomicOr(&marked[slot], kSplitSome);
            }
            return __int_as_float((scale.sx + 127) << 23);
        };
        auto put_unit = [&](int chunk, int k, const float (&src)[UPX][8], float m) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < UPX; ++q) {
                uint4 hi, lo;
                unsigned* const ph = &hi.x;
                unsigned* const pl = &lo.x;
#pragma unroll
                for (int j = 0; j < 8; j += 2) split_pair(src[q][j], src[q][j + 1], m, ph[j >> 1], pl[j >> 1]);
                uint4* dst = lds4 + ((chunk & 1) * 4 + w4) * 2 * npp + (unit(k) * 64 + lane) * UPX + q;
                dst[0] = hi;
                dst[npp] = lo;
            }
        };
        // largest and, beside zero, smallest magnitude; the maximum of two passes over a NaN
        auto top_unit = [&](const float (&src)[UPX][8], float& m, unsigned& lowest) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8 * UPX; j += 2) {
                m = fmaxf(fmaxf(fabsf(src[j >> 3][j & 7]), fabsf(src[j >> 3][(j + 1) & 7])), m);
                lowest = min(min(split_low(src[j >> 3][j & 7]), split_low(src[j >> 3][(j + 1) & 7])), lowest);
            }
        };
        auto end_top = [&](int chunk, const float (&src)[UNITS][UPX][8], float m) __attribute__((always_inline)) {
            if (__any(m > 3.402823466e38f)) {
                m = 0.0f;
#pragma unroll
                for (int k = 0; k < UNITS; ++k)
                    if (k < units)
#pragma unroll
                        for (int j = 0; j < 8 * UPX; ++j) {
                            const float v = fabsf(src[k][j >> 3][j & 7]);
                            m = fmaxf(m, v <= 3.402823466e38f ? v : 0.0f);
                        }
            }
            m = split_wave_max(m);
            if (lane == 63) atomicMax(&top_bits[chunk % 3], __float_as_uint(m));
        };
        // When the first chunk of a unit is computed, the marks of the one before have been read.  (The next that
        // are written, even of a unit of one step, are those of the unit after the one computed.)
        int gs = 0, old = kSplitMarks - 1;            // step of chunk g, marks of the unit before its own
        auto clear = [&]() __attribute__((always_inline)) {
            if (gs == 0) {
                if (wave == 4 && marked[old]) {
                    for (int e = lane; e < npp; e += 64) marks[old * npp + e] = 0;
                    if (lane == 0) marked[old] = 0;
                }
                old = old == kSplitMarks - 1 ? 0 : old + 1;
            }
            if (++gs == steps) gs = 0;
        };
        // set c & 1 holds chunk c
        auto iteration = [&](int g, float (&near)[UNITS][UPX][8], float (&far)[UNITS][UPX][8], unsigned& low_near, unsigned& low_far) __attribute__((always_inline)) {
            // near: chunk g + 1, then g + 3; far: chunk g + 2.  Unit by unit: the loads of one, which wait for their turn
            // in the addresser, are issued between the arithmetic of others (128 -> 128 at 56 x 56 / 2, 64 images: all of
            // one kind, then the next, 100.8 us, this way 98.0; 64 -> 64 at 224 x 224, 4 images, all kept 121 -> 116)
            if (g >= 0) {
                if (threadIdx.x == 256) top_bits[g % 3] = 0;
                clear();
            }
            const bool puts = g + 1 >= 0 && g + 1 < chunks, loads = g + 3 < chunks, tops = g + 2 >= 0 && g + 2 < chunks;
            float m = 0.0f, most = 0.0f;
            unsigned lowest = ~0u;
            if (puts) m = begin_put(g + 1, near, low_near);
            if (loads && ls == 0) enter(lu);
            __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)in_blk, 0, (int)range, 0x00020000);
#pragma unroll
            for (int k = 0; k < UNITS; ++k) {
                if (k < units) {
                    if (tops) top_unit(far[k], most, lowest);
                    if (puts) put_unit(g + 1, k, near[k], m);
                    if (loads) load_unit(near[k], rsrc, off[k], ls * 32 + w4 * 8);
                }
            }
            if (loads && ++ls == steps) { ls = 0; lu += gridDim.x; }
            if (tops) {
                low_far = lowest;
                end_top(g + 2, far, most);
            }
            __syncthreads();
        };
        for (int g = -3; g < chunks; g += 2) {
            iteration(g, raw[0], raw[1], low[0], low[1]);
            if (g + 1 < chunks) iteration(g + 1, raw[1], raw[0], low[1], low[0]);
        }
        return;
    }

    // ---- computing
    const int wp = wave % WP, wf = wave / WP;
    for (int g = -3; g < 0; ++g) __syncthreads();
    int chunk = 0, slot = 0;
    for (int u = u0; u < a->total; u += gridDim.x, slot = slot == kSplitMarks - 1 ? 0 : slot + 1) {
        a = split_args();
        const int npp = a->npp, pitch = a->pitch;
        int base[PN];
        // (by their number in a buffer: pointers would take two registers for each load)
        const __amdgpu_buffer_rsrc_t wsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a->weights, 0, (a->fblocks * steps * 9 + 2) * (8 * 1024), 0x00020000);
        unsigned wt;
        {
            const SplitUnit t = split_unit<PIX>(a, u);
#pragma unroll
            for (int p = 0; p < PN; ++p) {
                int img, oy, sx;
                split_pixel(a, min(t.pix0 + (wp * PN + p) * 16 + l16, t.last), img, oy, sx);
                base[p] = (img * a->vh + oy * a->conv_stride - t.vrow0) * pitch + sx * a->conv_stride + (a->lead - a->pad) + quarter * 2 * npp;
            }
            wt = (unsigned)min(t.fset * WF + wf, a->fblocks - 1) * (unsigned)steps * (9 * 8 * 1024);
        }
        float4v sum[4][PN];
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int p = 0; p < PN; ++p) sum[f][p] = float4v{};
        int sx = 0;
        // a stage is a tap of 32 filters: nine of the first 32, nine of the others; weights come two stages ahead
        half8 wv[3][2][2];
        auto weights = [&](int stage) __attribute__((always_inline)) {
            // the last step's last two look one step further: there is room behind the weights
            const int step = stage / 18, f0 = stage % 18 / 9 * 2, tap = step * 9 + stage % 9;
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int k = 0; k < 2; ++k) wv[stage % 3][f][k] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(wsrc, lane * 16, (int)(wt + (((unsigned)tap * 4 + f0 + f) * 2 + k) * 1024), 0));
        };
        weights(0);
        weights(1);
#pragma unroll 1
        for (int step = 0; step < steps; ++step, ++chunk) {
            const uint4* src = lds4 + (chunk & 1) * 8 * npp;
            half8 x[PN][2];
            int row = 0;
            auto inputs = [&](int tap, int p) __attribute__((always_inline)) {
                if (tap % 3 == 0 && p == 0) {
                    row = tap / 3 * pitch;
                    asm volatile("" : "+s"(row));     // or the first half's addresses are held for the second one
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) x[p][k] = __builtin_bit_cast(half8, src[base[p] + row + tap % 3 + k * npp]);
            };
#pragma unroll
            for (int p = 0; p < PN; ++p) inputs(0, p);
            const int e = __builtin_amdgcn_readfirstlane(exps[chunk & 1]);
            const float rescale = ldexpf(1.0f, e - sx);
            sx = e;
            float4v high[2][PN], low[2][PN];
            // sums of a step by themselves, and what they are together: fewer roundings at the size of the whole
            auto join = [&](int f0, int p) __attribute__((always_inline)) {
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    const float4v part = __builtin_elementwise_fma(low[f][p], float4v{} + 1.0f / 2048.0f, high[f][p]);
                    sum[f0 + f][p] = __builtin_elementwise_fma(sum[f0 + f][p], float4v{} + rescale, part);
                    // here: at the step's end, where the compiler would put it, both halves' parts are held
                    asm volatile("" : "+v"(sum[f0 + f][p]));
                }
            };
#pragma unroll
            for (int stage = 0; stage < 18; ++stage) {
                const int tap = stage % 9, f0 = stage / 9 * 2;
                weights(stage + 2);
                const half8 (&w)[2][2] = wv[stage % 3];
#pragma unroll
                for (int p = 0; p < PN; ++p) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int f = 0; f < 2; ++f) high[f][p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[f][0], x[p][0], tap ? high[f][p] : float4v{}, 0, 0, 0);
#pragma unroll
                    for (int f = 0; f < 2; ++f) low[f][p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[f][0], x[p][1], tap ? low[f][p] : float4v{}, 0, 0, 0);
#pragma unroll
                    for (int f = 0; f < 2; ++f) low[f][p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[f][1], x[p][0], low[f][p], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (stage < 17) inputs((tap + 1) % 9, p);
                    if (tap == 8 && p > 0) join(f0, p - 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (tap == 8) join(f0, PN - 1);
            }
            wt += 9 * 8 * 1024;
            if (step + 1 < steps) __syncthreads();
        }

        // ---- epilogue: register r of a block is filter 4 * (lane / 16) + r, pixel lane % 16
        a = split_args();
        const SplitUnit t = split_unit<PIX>(a, u);
        bool ok[PN];
        size_t at[PN];
        const int oh = a->pool ? a->ho >> 1 : a->ho, ow = a->pool ? a->wo >> 1 : a->wo;
        const size_t oplane = (size_t)oh * ow;
#pragma unroll
        for (int p = 0; p < PN; ++p) {
            const int q = t.pix0 + (wp * PN + p) * 16 + l16;
            int img, oy, px;
            split_pixel(a, min(q, t.last), img, oy, px);
            const int ox = t.strip * a->sw + px;
            ok[p] = q <= t.last && ox < a->wo;
            if (a->pool) ok[p] = ok[p] && !(lane & 3) && (ox >> 1) < ow && (oy >> 1) < oh;
            at[p] = (size_t)img * a->c_out * oplane + (size_t)(a->pool ? oy >> 1 : oy) * ow + (a->pool ? ox >> 1 : ox);
        }
        const bool pool = a->pool, relu = a->relu;
        unsigned again = 0;                           // blocks of pixels that are worked out again
        unsigned low_px = 0;                          // ... for small sums: pixels over marked ones
        const unsigned some = (unsigned)__builtin_amdgcn_readfirstlane((int)marked[slot]);
        if (some) {
            if (some & kSplitAll) again = ~0u;
#pragma unroll
            for (int p = 0; p < PN; ++p) {
                int img, oy, px;
                split_pixel(a, min(t.pix0 + (wp * PN + p) * 16 + l16, t.last), img, oy, px);
                const unsigned char* const under = marks + slot * a->npp + (img * a->vh + oy * a->conv_stride - t.vrow0) * a->pitch + px * a->conv_stride + (a->lead - a->pad);
                unsigned any = 0;
#pragma unroll
                for (int tap = 0; tap < 9; ++tap) any |= under[tap / 3 * a->pitch + tap % 3];
                low_px |= (unsigned)(any != 0) << p;
            }
        }
        int2 filter[4][4];
        float bias[4][4];
        const int2* const mine = a->filters + (size_t)min(t.fset * WF + wf, a->fblocks - 1) * 64 + quarter * 4;
        const bool used = t.fset * WF + wf < a->fblocks;
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) filter[f][r] = mine[f * 16 + r];
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (!used) filter[f][r].x = -1;
                bias[f][r] = a->bias ? a->bias[max(filter[f][r].x, 0)] : 0.0f;
            }
        if (some)
#pragma unroll
            for (int f = 0; f < 4; ++f)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float seen = filter[f][r].x >= 0 && filter[f][r].y != kSplitEmpty ? a->seen : 0.0f;
#pragma unroll
                    for (int p = 0; p < PN; ++p)
                        again |= fabsf(sum[f][p][r]) < seen ? low_px & 1u << p : 0u;
                }
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = filter[f][r].x, ex = -(sx + filter[f][r].y);
                const float b = bias[f][r];
                const bool has = co >= 0;
                float* const dst = a->out + (size_t)co * oplane;
#pragma unroll
                for (int p = 0; p < PN; ++p) {
                    float v = ldexpf(sum[f][p][r], ex);
                    again |= (unsigned)!(fabsf(v) < __builtin_inff()) << p;
                    v += b;
                    if (pool) v = split_pool(v);
                    if (relu) v = fmaxf(v, 0.0f);
                    if (ok[p] && has) dst[at[p]] = v;
                }
            }
        if (__any(again)) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // after the stores above
            split_again<PN, WF, WP>(again, u, wave);
        }
        __syncthreads();
    }
}

// One workgroup per stored filter: its kept weights, brought to the filter's scale, to their places in the
// fragments, zeros as -0 in the high part (removed ones stay +0).
__global__ __launch_bounds__(256) void split_expand_kernel(const int32_t* offset, const int32_t* index, const int32_t* stride,
                                                           const float* weight, const uint16_t* masks, const int32_t* filters,
                                                           int num_patterns, int taps, int steps, __half* out)
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
            const float w = ldexpf(weight[(size_t)(k0 + k) * taps + t], filters[2 * s + 1]);
            const __half hi = __float2half_rn(w), lo = __float2half_rn((w - __half2float(hi)) * 2048.0f);
            const unsigned short b = __half_as_ushort(hi);
            __half* frag = out + ((((size_t)(s >> 6) * steps + (c >> 5)) * 9 + pos) * 4 + ((s >> 4) & 3)) * (2 * 64 * 8) + (((c >> 3) & 3) * 16 + (s & 15)) * 8 + (c & 7);
            frag[0] = __ushort_as_half(b & 0x7FFF ? b : 0x8000);
            frag[64 * 8] = lo;
        }
    }
}

// Two taps more than the layer has: the kernel looks two stages ahead.
size_t split_expanded_halves(int32_t c_in, int32_t c_out)
{
    return ((size_t)((c_out + 63) / 64) * ((c_in + 31) / 32) * 9 + 2) * 8 * 64 * 8;
}

hipError_t launch_split_expand(const DevFkw& f, int32_t c_in, int32_t c_out, void* out, hipStream_t stream)
{
    hipLaunchKernelGGL(split_expand_kernel, dim3((unsigned)c_out), dim3(256), 0, stream, f.offset, f.index, f.stride, f.weight, f.masks,
                       f.split_filters, f.num_patterns, f.taps, (c_in + 31) / 32, static_cast<__half*>(out));
    return hipGetLastError();
}

// How the pixels of an output are cut into tiles of `pix`; false where the kernel's numbers do not reach.
static bool split_tiles(const ConvShape& s, int pix, int widest, bool pair, SplitArgs& a)
{
    a.rp = s.pool ? 2 : 1;
    a.hr = s.ho / a.rp;
    const int wo = s.pool ? s.wo & ~1 : s.wo;
    a.strips = (wo + widest - 1) / widest;
    a.sw = (wo + a.strips - 1) / a.strips;
    if (s.pool || pair) a.sw = (a.sw + 1) & ~1;
    a.vh = s.h + 2 * s.pad;
    a.lead = pair ? 2 * s.pad : s.pad;               // pairs start at even columns
    a.pitch = (a.sw - 1) * s.stride + 3 + a.lead - s.pad;
    if (pair) a.pitch = (a.pitch + 1) & ~1;
    const long long pixels = (long long)s.n * a.hr * a.rp * a.sw;
    if (pixels > INT32_MAX - pix || (long long)s.n * a.vh > INT32_MAX) return false;
    a.pixels = (int32_t)pixels;
    a.tiles = (int32_t)((pixels + pix - 1) / pix);
    // row groups that `pix` pixels touch, and the rows under them
    const int group = a.rp * a.sw;
    const int groups = (int)std::min<long long>((pix - 1 + group - 1) / group + 1, (long long)s.n * a.hr);
    const int between = std::min(s.n - 1, (groups - 1 + a.hr - 1) / a.hr);
    const int rows = (groups * a.rp - 1) * s.stride + between * (a.vh - a.hr * a.rp * s.stride) + 3;
    const int unit = pair ? 128 : 64;
    a.npb = (rows * a.pitch + unit - 1) / unit;
    a.npp = a.npb * unit;
    // byte offsets from a tile's first image, and a staging wavefront's registers
    return (long long)(between + 2) * s.c_in * s.h * s.w < (1ll << 29) && a.npb <= split_units(pair) && split_lds(a.npp) <= 160 * 1024;
}

template <int PN, int WF, int WP, bool PAIR>
static hipError_t launch_split_t(SplitArgs a, hipStream_t stream)
{
    a.div_fsets = make_fast_div((uint32_t)a.fsets);
    a.div_strips = make_fast_div((uint32_t)a.strips);
    a.div_sw = make_fast_div((uint32_t)a.sw);
    a.div_hr = make_fast_div((uint32_t)a.hr);
    a.div_vh = make_fast_div((uint32_t)a.vh);
    a.div_pitch = make_fast_div((uint32_t)a.pitch);
    const size_t lds = (size_t)split_lds(a.npp);
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> allowed{0};
        hipError_t e = allow_big_lds(reinterpret_cast<const void*>(&split_conv_kernel<PN, WF, WP, PAIR>), allowed);
        if (e != hipSuccess) return e;
    }
    const int grid = std::min(a.total, 256);
    hipLaunchKernelGGL((split_conv_kernel<PN, WF, WP, PAIR>), dim3((unsigned)grid), dim3(split_threads(PN)), lds, stream, a);
    return hipGetLastError();
}

struct SplitShape {
    int pn, wf, wp;
    hipError_t (*launch[2])(SplitArgs, hipStream_t);
};
#define PATDNN_SPLIT(pn, wf, wp) {pn, wf, wp, {&launch_split_t<pn, wf, wp, false>, &launch_split_t<pn, wf, wp, true>}}
static const SplitShape kSplitShapes[] = {
    PATDNN_SPLIT(4, 1, 4),
    PATDNN_SPLIT(4, 2, 2),
    PATDNN_SPLIT(2, 1, 4),
    PATDNN_SPLIT(2, 2, 2),
};
#undef PATDNN_SPLIT

static int split_plan(const ConvShape& s, bool pair, bool narrow, SplitArgs& a)
{
    a.steps = (s.c_in + 31) / 32;
    a.fblocks = (s.c_out + 63) / 64;
    for (const SplitShape& v : kSplitShapes) {
        // (half of the last shape's wavefronts idle for 64 filters: narrow images of many rows only)
        const bool last = &v == std::end(kSplitShapes) - 1;
        if ((v.wf > 1) != (a.fblocks > 1) && !last) continue;
        const int pix = 16 * v.pn * v.wp;
        if (narrow ? !(last && split_tiles(s, pix, 8, pair, a)) : !split_tiles(s, pix, 32, pair, a) && !split_tiles(s, pix, 16, pair, a)) continue;
        a.fsets = (a.fblocks + v.wf - 1) / v.wf;
        const long long total = (long long)a.strips * a.tiles * a.fsets;
        if (total > INT32_MAX / 2 || total * a.steps > INT32_MAX / 2) continue;
        a.total = (int32_t)total;
        return (int)(&v - kSplitShapes);
    }
    return -1;
}

// two pixels per load: rows of an even length and an 8-byte aligned tensor
static bool split_pair_rows(const ConvShape& s, const void* in) { return s.w % 2 == 0 && (reinterpret_cast<uintptr_t>(in) & 7) == 0; }

bool split_cost(const ConvShape& s, int& rounds, int& steps, int& pixels)
{
    SplitArgs a{};
    int shape = split_plan(s, false, false, a);
    if (shape < 0 && s.pool) shape = split_plan(s, false, true, a);
    if (shape < 0) return false;
    rounds = (a.total + 255) / 256;
    steps = a.steps;
    pixels = 16 * kSplitShapes[shape].pn;
    return true;
}

// Number of the launch shape, twice, plus one with pairs; -1 where none fits.
static int split_launch_plan(const ConvShape& s, const void* in, SplitArgs& a)
{
    // (rows two at a time stage more: narrow strips then, so that a pooled call runs the kernel that the plain one does)
    for (const bool narrow : {false, true})
        for (const bool pair : {true, false}) {
            if ((pair && !split_pair_rows(s, in)) || (narrow && !s.pool)) continue;
            const int shape = split_plan(s, pair, narrow, a);
            if (shape >= 0) return 2 * shape + pair;
        }
    return -1;
}

int split_choice(const ConvShape& s, const void* in, int& units)
{
    SplitArgs a{};
    const int choice = split_launch_plan(s, in, a);
    units = a.total;
    return choice;
}

hipError_t launch_split(const DevFkw& f, const ConvShape& s, const float* in, const float* bias, float* out, hipStream_t stream)
{
    SplitArgs a{};
    a.in = in; a.bias = bias; a.out = out;
    a.weights = static_cast<const uint4*>(f.split_f16);
    a.filters = reinterpret_cast<const int2*>(f.split_filters);
    a.seen = f.split_seen;
    a.n = s.n; a.c_in = s.c_in; a.c_out = s.c_out; a.h = s.h; a.w = s.w; a.ho = s.ho; a.wo = s.wo;
    a.conv_stride = s.stride; a.pad = s.pad; a.relu = s.relu; a.pool = s.pool;
    const int choice = split_launch_plan(s, in, a);
    return choice < 0 ? hipErrorInvalidValue : kSplitShapes[choice >> 1].launch[choice & 1](a, stream);
}

}  // namespace patdnn
