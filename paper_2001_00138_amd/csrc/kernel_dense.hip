// Dense 3x3 layers of few input channels (the first layer of a pruned network) on the matrix cores in fp32.
//
// Such a layer writes much more than it reads - 64 output channels from three - and has so few products per
// output (27) that what matters is to keep the stores going.  v_mfma_f32_32x32x2_f32 does them at twice the
// vector ALU's rate, from registers alone: the weights of a wavefront's filters stay there, and the input values of 32
// pixels are read by the lanes where they are needed, from the caches, with no LDS and no barrier.
//
//   * Output pixels are numbered through all images; a block is 32 consecutive ones, and a wavefront computes FM x 32
//     filters of a block: lane (half, i) supplies weight and input value 2 * step + half of filter i and pixel i
//     for the matrix instruction of that step.  The value after the last tap is a one that meets the bias.
//   * Workgroups stay and go on to further blocks, those of an XCD side by side, so that rows are read from
//     memory by one L2; the inputs of the next block are loaded before this one is multiplied.
//   * Where windows are pooled a block is eight of them, each in four neighbouring lanes, which store a fourth of the
//     filters each (3 -> 64 at 224 x 224, 64 images, 168 us where atomics on a cleared output took 2383 and the
//     vector ALU's kernel 1338; 4 -> 88 at 100 x 100, 32 images, 49, 420 and 257).
//
// What bounds it: the output's way to memory (3 -> 64 at 224 x 224, 64 images: 165 to 176 us, 5 TB/s, where the vector
// ALU's kernel took 233), small launches the chain of loads, 28 steps of 64 cycles and stores (one image of it 10.5
// us for 15.9; 4 -> 88 at 100 x 100, 32 images, 44 to 51 for 69; 3 -> 32 at 112 x 112 / 2, 64 images, 13.4 where the walk over
// the weights took 117).  Errors against 64 bits are those of the kernels before (9.35e-8 of the result's norm).
#include <algorithm>

#include "kernels.hpp"

namespace patdnn {

struct DenseArgs {
    const float* in;
    const float* weight;             // [c_out][c_in][9]
    const float* bias;
    float* out;
    int32_t n, c_out, h, w, pad, relu;
    int32_t wo, oplane;              // columns and pixels of an output plane, or of a pooled one
    int32_t blocks, pixels;          // those of all images (pooled: four times as many), and blocks of 32 of them
    FastDiv div_wo, div_plane;       // wo, oplane
};

// Steps of two values: nine taps of every channel, and the bias.
constexpr int dense_steps(int c_in) { return (9 * c_in + 2) / 2; }

// STREAM: stores that leave nothing in the caches (see launch_dense; the compiler makes one of two kinds of store in one kernel).
enum DenseOut { kDensePlain, kDenseStream, kDensePool };
// Each of a window's four lanes has its largest value afterwards.
static __device__ __forceinline__ float dense_window(float v)
{
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true)));      // quad_perm [1,0,3,2]
    return fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, true)));   // quad_perm [2,3,0,1]
}

template <int C, int FM, int STRIDE, DenseOut OUT>
__global__ __launch_bounds__(256) void dense_conv_kernel(DenseArgs a)
{
    constexpr int K = 9 * C, STEPS = dense_steps(C);
    typedef float float16v __attribute__((ext_vector_type(16)));
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int f0 = (int)blockIdx.y * FM * 32;

    float wv[FM][STEPS];
#pragma unroll
    for (int f = 0; f < FM; ++f) {
        const int s = f0 + f * 32 + l32;
        const float* const row = a.weight + (size_t)min(s, a.c_out - 1) * K;
        const float last = a.bias ? a.bias[min(s, a.c_out - 1)] : 0.0f;
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const int k = 2 * i + half;
            const float v = row[min(k, K - 1)];
            wv[f][i] = k < K ? v : k == K ? last : 0.0f;
        }
    }
    // where value 2 * step + half lies from a window's first one, in bytes
    const int plane = a.h * a.w;
    int tap[STEPS];
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        const int k = min(2 * i + half, K - 1), c = k / 9, pos = k - 9 * c;
        tap[i] = 4 * (c * plane + pos / 3 * a.w + pos % 3);
    }

    const size_t image = (size_t)C * plane;
    const int oplane = a.oplane;
    constexpr int PER = OUT == kDensePool ? 4 : 1;    // lanes of an output pixel
    // blocks of a step of the whole grid: an XCD's eighth of them side by side
    const int per_xcd = gridDim.x >> 3, share = (a.blocks + 31) / 32 * 4;
    const bool whole = (gridDim.x & 7) == 0;
    const int first = whole ? (int)(blockIdx.x & 7) * share + (int)(blockIdx.x >> 3) * 4 + wave : (int)blockIdx.x * 4 + wave;
    const int past = whole ? min(a.blocks, ((int)(blockIdx.x & 7) + 1) * share) : a.blocks;
    const int stride = whole ? per_xcd * 4 : (int)gridDim.x * 4;

    // the lane's pixel of a block (or its window), and that pixel's inputs
    struct Pixel { int img0, img, at; };
    auto locate = [&](int block) __attribute__((always_inline)) -> Pixel {
        const int q = min(block * 32 + l32, a.pixels - 1) / PER;
        Pixel p;
        p.img0 = (int)fast_div((uint32_t)(block * (32 / PER)), a.div_plane);
        p.img = (int)fast_div((uint32_t)q, a.div_plane);
        p.at = q - p.img * oplane;
        return p;
    };
    auto load = [&](int block, float (&x)[STEPS]) __attribute__((always_inline)) {
        const Pixel p = locate(block);
        int oy = (int)fast_div((uint32_t)p.at, a.div_wo), ox = p.at - oy * a.wo;
        if constexpr (OUT == kDensePool) {
            oy = 2 * oy + (lane & 1);
            ox = 2 * ox + (lane >> 1 & 1);
        }
        const int y = oy * STRIDE - a.pad, xx = ox * STRIDE - a.pad;
        unsigned cols = 0, outside = 0;               // bit t: tap column, then tap, outside the image
#pragma unroll
        for (int t = 0; t < 3; ++t) cols |= (unsigned)((unsigned)(xx + t) >= (unsigned)a.w) << t;
#pragma unroll
        for (int t = 0; t < 3; ++t) outside |= ((unsigned)(y + t) >= (unsigned)a.h ? 7u : cols) << (3 * t);
        const int base = 4 * ((p.img - p.img0) * C * plane + y * a.w + xx);
        __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(a.in + p.img0 * image), 0, (int)(unsigned)std::min<size_t>((size_t)(a.n - p.img0) * image * 4, 0x80000000u), 0x00020000);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            // (out of range reads as zero; what follows the last tap does too)
            const unsigned bit = half ? 1u << (2 * i + 1) % 9 : 1u << 2 * i % 9;
            const bool none = (outside & bit) || 2 * i + half >= K;
            x[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, none ? -1 : base + tap[i], 0, 0));
        }
    };

    float x[STEPS];
    if (first < past) load(first, x);
    for (int block = first; block < past; block += stride) {
        if (K & 1) x[STEPS - 1] = half ? 1.0f : x[STEPS - 1];
        else x[STEPS - 1] = half ? 0.0f : 1.0f;
        float next[STEPS];
        load(min(block + stride, past - 1), next);
        float16v acc[FM];
#pragma unroll
        for (int f = 0; f < FM; ++f) acc[f] = float16v{};
#pragma unroll
        for (int i = 0; i < STEPS; ++i)
#pragma unroll
            for (int f = 0; f < FM; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[f][i], x[i], acc[f], 0, 0, 0);

        // register r is filter 8 * (r / 4) + 4 * half + r % 4, pixel lane % 32
        const Pixel p = locate(block);
        const bool ok = block * 32 + l32 < a.pixels;
        const int left = a.c_out - f0 - 4 * half;     // filters from this lane's first one on
        char* const dst = reinterpret_cast<char*>(a.out + ((size_t)p.img0 * a.c_out + f0) * oplane);
        const unsigned at = 4u * (((unsigned)(p.img - p.img0) * (unsigned)a.c_out + 4u * half) * (unsigned)oplane + (unsigned)p.at);
        if constexpr (OUT == kDensePool) {
            const int mine = lane & 3;                // registers 4 i + mine
#pragma unroll
            for (int f = 0; f < FM; ++f)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float m[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) m[k] = dense_window(acc[f][4 * i + k]);
                    const float v = fmaxf(mine < 2 ? mine ? m[1] : m[0] : mine == 2 ? m[2] : m[3], 0.0f);
                    const int s = f * 32 + 8 * i + mine;
                    if (ok && s < left) *reinterpret_cast<float*>(dst + (size_t)s * oplane * 4 + at) = v;
                }
        } else {
            auto store = [&](bool some) __attribute__((always_inline)) {
#pragma unroll
                for (int f = 0; f < FM; ++f)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int s = f * 32 + 8 * (r >> 2) + (r & 3);
                        const float v = a.relu ? fmaxf(acc[f][r], 0.0f) : acc[f][r];
                        float* const to = reinterpret_cast<float*>(dst + (size_t)s * oplane * 4 + at);
                        if (some && s >= left) continue;
                        if constexpr (OUT == kDenseStream) __builtin_nontemporal_store(v, to);
                        else *to = v;
                    }
            };
            if (ok) {
                if (f0 + 32 * FM > a.c_out) store(true);
                else store(false);
            }
        }
#pragma unroll
        for (int i = 0; i < STEPS; ++i) x[i] = next[i];
    }
}

// Up to four input channels, whose weights fit in registers; 32-bit pixel numbers, and byte offsets from a block's first
// image.
bool dense_fits(const ConvShape& s)
{
    if (s.c_in > kDenseChannels || s.stride > 2) return false;
    // (images that a block spans: the more where windows are pooled; both have to fit, so that both kinds of call
    // run the same kernel)
    const long long oplane = (long long)s.ho * s.wo, whole = std::max(1ll, (long long)(s.ho / 2) * (s.wo / 2) * 4);
    const long long between = std::min<long long>(s.n - 1, 31 / std::min(oplane, whole) + 1);
    return (long long)s.n * oplane <= INT32_MAX - 64 && (between + 1) * s.c_in * s.h * s.w < (1ll << 29) &&
           (between + 1) * s.c_out * oplane < (1ll << 29) && s.c_out <= 32 * 65535;
}

template <int C, int FM, int STRIDE>
static hipError_t launch_dense_t(const DenseArgs& a, DenseOut out, hipStream_t stream)
{
    const unsigned sets = (unsigned)((a.c_out + 32 * FM - 1) / (32 * FM));
    // as many workgroups as their registers let a CU hold
    const unsigned most = std::max(8u, (C == 4 && FM == 2 ? 512u : 768u) / sets / 8 * 8);
    const unsigned grid = std::min((unsigned)((a.blocks + 3) / 4), most);
    if (out == kDensePool) hipLaunchKernelGGL((dense_conv_kernel<C, FM, STRIDE, kDensePool>), dim3(grid, sets), dim3(256), 0, stream, a);
    else if (out == kDenseStream) hipLaunchKernelGGL((dense_conv_kernel<C, FM, STRIDE, kDenseStream>), dim3(grid, sets), dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((dense_conv_kernel<C, FM, STRIDE, kDensePlain>), dim3(grid, sets), dim3(256), 0, stream, a);
    return hipGetLastError();
}
template <int C>
static hipError_t launch_dense_c(const DenseArgs& a, int stride, DenseOut out, hipStream_t stream)
{
    // 64 filters at a time unless all fit in 32: what is read is read once more for the next ones
    const bool two = a.c_out > 32;
    if (stride == 2) return two ? launch_dense_t<C, 2, 2>(a, out, stream) : launch_dense_t<C, 1, 2>(a, out, stream);
    return two ? launch_dense_t<C, 2, 1>(a, out, stream) : launch_dense_t<C, 1, 1>(a, out, stream);
}

hipError_t launch_dense(const DevFkw& f, const ConvShape& s, const float* in, const float* bias, float* out, hipStream_t stream)
{
    DenseArgs a{};
    a.in = in; a.weight = f.weight; a.bias = bias; a.out = out;
    a.n = s.n; a.c_out = s.c_out; a.h = s.h; a.w = s.w; a.pad = s.pad; a.relu = s.relu;
    a.wo = s.pool ? s.wo / 2 : s.wo;
    a.oplane = s.pool ? s.ho / 2 * a.wo : s.ho * s.wo;
    a.pixels = s.n * a.oplane * (s.pool ? 4 : 1);
    // Beyond the 256 MB of the last-level cache, and where a block's stores are whole cache lines (3 -> 64 at 224 x 224, 64
    // images, 822 MB: 230 us without, 176 to 187 with; 4 -> 88 at 100 x 100, 32 images, 113 MB, 47 and 46; 4 -> 24 at 150 x 133,
    // 30 images, which are not whole lines, 27 and 37).
    const bool stream_out = (size_t)a.pixels * s.c_out * 4 > ((size_t)256 << 20) && s.ho * s.wo % 32 == 0 && (reinterpret_cast<uintptr_t>(out) & 127) == 0;
    a.blocks = (a.pixels + 31) / 32;
    a.div_wo = make_fast_div((uint32_t)a.wo);
    a.div_plane = make_fast_div((uint32_t)a.oplane);
    const DenseOut kind = s.pool ? kDensePool : stream_out ? kDenseStream : kDensePlain;
    switch (s.c_in) {
    case 1: return launch_dense_c<1>(a, s.stride, kind, stream);
    case 2: return launch_dense_c<2>(a, s.stride, kind, stream);
    case 3: return launch_dense_c<3>(a, s.stride, kind, stream);
    case 4: return launch_dense_c<4>(a, s.stride, kind, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace patdnn
