// Depthwise pattern-pruned 3x3 convolution (the MobileNet-V2 layers the paper evaluates,
// section 6.1): one four-tap kernel per channel, so the layer does about one flop per byte
// and is bound by HBM bandwidth, not by arithmetic.
//
// Design for that bound: one pass over the input and one over the output.  A lane owns
// four consecutive output pixels of one row (one 16-byte store); per input row that its
// channel's pattern touches it loads 16-byte vectors plus the one or two halo elements
// (predicated, zero outside the image).  Rows are re-read by the lanes of the rows above
// and below, which sit next to each other in the grid and hit the same cache lines, so the
// traffic that reaches HBM is the tensor once.  Channels are walked in the stored filter
// order of the FKW arrays; for one-kernel filters the filter reorder of section 5.2 sorts
// them by pattern, so the lanes of a wavefront share one pattern and skip the same rows
// and taps together (the `if`s on the pattern mask below are then uniform branches).
// Bias and ReLU are fused; the result goes to the original channel `reorder[f]`.
// The same kernel runs on fp32 tensors and on half-precision storage (binary16 weights, input
// and output, fp32 arithmetic in between - the paper's GPU runs keep weights and intermediate
// results in 16 bits, section 6.1): there the bytes, and with them the time, halve.
#include <hip/hip_fp16.h>

#include <algorithm>

#include "kernels.hpp"

namespace patdnn {

// LDS that dw_planes_kernel may take: three workgroups on a CU
constexpr long long kDwPlanesLds = 52 * 1024;

template <class T>
struct DwArgs {
    const int32_t* reorder;      // [c] stored filter -> channel
    const int32_t* dw_mask;      // [c] pattern mask of the stored filter's kernel (0: removed)
    const T* dw_weight;          // [c][4] its weights, ascending position
    const T* in;
    const float* bias;
    T* out;
    int32_t c, h, w, ho, wo, wq, pad, relu;
    long long total;             // n * c * ho * wq lanes
    FastDiv div_wq, div_ho, div_c;   // for lane numbers below 2^31 (every realistic launch)
};

// element access: one value, or four consecutive ones with one 16-byte (fp32) / 8-byte
// (binary16) access at an address aligned to that size
__device__ __forceinline__ float ld1(const float* p) { return *p; }
__device__ __forceinline__ float ld1(const __half* p) { return __half2float(*p); }
__device__ __forceinline__ void ld4(const float* p, float& a, float& b, float& c, float& d)
{
    const float4 m = *reinterpret_cast<const float4*>(p);
    a = m.x; b = m.y; c = m.z; d = m.w;
}
__device__ __forceinline__ void ld4(const __half* p, float& a, float& b, float& c, float& d)
{
    const uint2 m = *reinterpret_cast<const uint2*>(p);
    const __half2 lo = *reinterpret_cast<const __half2*>(&m.x), hi = *reinterpret_cast<const __half2*>(&m.y);
    a = __low2float(lo); b = __high2float(lo); c = __low2float(hi); d = __high2float(hi);
}
__device__ __forceinline__ void st1(float* p, float v) { *p = v; }
__device__ __forceinline__ void st1(__half* p, float v) { *p = __float2half_rn(v); }
// NP consecutive elements at an address aligned to NP elements: 16-byte accesses for four
// floats or eight binary16 values
template <int NP>
__device__ __forceinline__ void ldv(const float* p, float* v)
{
#pragma unroll
    for (int k = 0; k < NP; k += 4) ld4(p + k, v[k], v[k + 1], v[k + 2], v[k + 3]);
}
template <int NP>
__device__ __forceinline__ void ldv(const __half* p, float* v)
{
    if constexpr (NP == 8) {
        const uint4 m = *reinterpret_cast<const uint4*>(p);
        const unsigned w[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const __half2 h = *reinterpret_cast<const __half2*>(&w[k]);
            v[2 * k] = __low2float(h);
            v[2 * k + 1] = __high2float(h);
        }
    } else {
        ld4(p, v[0], v[1], v[2], v[3]);
    }
}
// STREAM: stores that do not stay in the L2s
template <bool STREAM, int NP>
__device__ __forceinline__ void stv(float* p, const float (&v)[NP])
{
    typedef float float4s __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int k = 0; k < NP; k += 4) {
        const float4s q = {v[k], v[k + 1], v[k + 2], v[k + 3]};
        if constexpr (STREAM) __builtin_nontemporal_store(q, reinterpret_cast<float4s*>(p + k));
        else *reinterpret_cast<float4s*>(p + k) = q;
    }
}
template <bool STREAM, int NP>
__device__ __forceinline__ void stv(__half* p, const float (&v)[NP])
{
    unsigned w[NP / 2];
#pragma unroll
    for (int k = 0; k < NP / 2; ++k) {
        const __half2 h = __floats2half2_rn(v[2 * k], v[2 * k + 1]);
        w[k] = *reinterpret_cast<const unsigned*>(&h);
    }
    if constexpr (NP == 8) *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
    else *reinterpret_cast<uint2*>(p) = make_uint2(w[0], w[1]);
}

// S: stride.  NP: outputs per lane (4, or 8 where the rows allow and the launcher finds it faster).  VEC: rows start aligned to NP elements (w % NP == 0,
// aligned base) -> vector loads.  VST: output rows aligned to NP elements -> one vector store.
template <int S, int NP, bool VEC, bool VST, class T, bool STREAM>
__global__ __launch_bounds__(256) void dw_conv_kernel(DwArgs<T> a)
{
    constexpr int NC = (NP - 1) * S + 3;           // input columns under NP outputs
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= a.total) return;
    // lane number -> (image n, stored channel f, output row oy, group of NP columns xq).  A
    // thread has a dozen FMAs to do, so three 64-bit divisions would be most of its
    // instructions and the kernel would be bound by them instead of by HBM: below 2^31 lanes
    // they are multiplications by launch-time constants.
    int xq, oy, f;
    long long n;
    if (a.total <= 0x7FFFFFFFll) {
        const uint32_t t32 = (uint32_t)t;
        const uint32_t r1 = fast_div(t32, a.div_wq);
        xq = (int)(t32 - r1 * (uint32_t)a.wq);
        const uint32_t r2 = fast_div(r1, a.div_ho);
        oy = (int)(r1 - r2 * (uint32_t)a.ho);
        const uint32_t r3 = fast_div(r2, a.div_c);
        f = (int)(r2 - r3 * (uint32_t)a.c);
        n = r3;
    } else {
        xq = (int)(t % a.wq);
        long long r = t / a.wq;
        oy = (int)(r % a.ho);
        r /= a.ho;
        f = (int)(r % a.c);
        n = r / a.c;
    }
    const int co = a.reorder[f];
    const unsigned mask = (unsigned)a.dw_mask[f];
    float4 wv;
    ld4(a.dw_weight + (size_t)f * 4, wv.x, wv.y, wv.z, wv.w);
    const T* plane = a.in + ((size_t)n * a.c + co) * ((size_t)a.h * a.w);
    const int ox0 = xq * NP;
    const int ix0 = ox0 * S - a.pad;               // input column under (output ox0, tap 0)

    float acc[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
        const unsigned rowbits = (mask >> (3 * dy)) & 7u;
        if (rowbits == 0) continue;
        const int iy = oy * S + dy - a.pad;
        if (iy < 0 || iy >= a.h) continue;         // zero padding: the row contributes nothing
        const T* row = plane + (size_t)iy * a.w;
        float v[NC];
        if constexpr (VEC) {
            // pad is 0 or 1: columns ix0 + pad .. start a vector
            if (a.pad == 1) {
                v[0] = ((rowbits & 1u) && ix0 >= 0) ? ld1(row + ix0) : 0.0f;
#pragma unroll
                for (int q = 0; q < (NC - 1) / NP; ++q) {
                    const int ix = ix0 + 1 + NP * q;
                    float m[NP];
#pragma unroll
                    for (int k = 0; k < NP; ++k) m[k] = 0.0f;
                    if (ix < a.w) ldv<NP>(row + ix, m);
#pragma unroll
                    for (int k = 0; k < NP; ++k) v[1 + NP * q + k] = m[k];
                }
                if constexpr (S == 1) {
                    const int ix = ix0 + NP + 1;
                    v[NP + 1] = ((rowbits & 4u) && ix < a.w) ? ld1(row + ix) : 0.0f;
                }
            } else {
#pragma unroll
                for (int q = 0; q < (NC + NP - 1) / NP; ++q) {
                    const int ix = ix0 + NP * q;
                    float m[NP];
#pragma unroll
                    for (int k = 0; k < NP; ++k) m[k] = 0.0f;
                    if (ix < a.w) ldv<NP>(row + ix, m);
#pragma unroll
                    for (int k = 0; k < NP; ++k)
                        if (NP * q + k < NC) v[NP * q + k] = m[k];
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const int ix = ix0 + j;
                v[j] = (ix >= 0 && ix < a.w) ? ld1(row + ix) : 0.0f;
            }
        }
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            if (!((rowbits >> dx) & 1u)) continue;
            // rank of this position among the kept ones = index of its stored weight
            const int rank = __builtin_popcount(mask & ((1u << (3 * dy + dx)) - 1u));
            const float wt = rank == 0 ? wv.x : rank == 1 ? wv.y : rank == 2 ? wv.z : wv.w;
#pragma unroll
            for (int i = 0; i < NP; ++i) acc[i] = fmaf(wt, v[i * S + dx], acc[i]);
        }
    }
    const float b = a.bias ? a.bias[co] : 0.0f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        acc[i] += b;
        if (a.relu) acc[i] = fmaxf(acc[i], 0.0f);
    }
    T* dst = a.out + (((size_t)n * a.c + co) * a.ho + oy) * (size_t)a.wo + ox0;
    if constexpr (VST) {
        stv<STREAM, NP>(dst, acc);
    } else {
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (ox0 + i < a.wo) st1(dst + i, acc[i]);
    }
}

template <class T>
struct DwPlanesArgs {
    const int32_t* taps;         // [c] by channel: four positions in nibbles, ascending; -1: kernel removed
    const float4* weight;        // [c] its weights in fp32
    const T* in;
    const float* bias;
    T* out;
    int32_t c, h, w, ho, wo, pad, relu;
    int32_t total, planes;       // n * c; planes of a workgroup, a multiple of the elements of 16 bytes
    int32_t in_units, out_units; // LDS for the staged planes and the results, in 16 bytes
    FastDiv div_c, div_hw, div_w, div_px, div_wo;
};

// Planes whose rows are no whole vectors.  Planes lie one after the other in memory, through
// channels and images, so a workgroup takes a run of them that starts at a multiple of 16 bytes,
// reads it with 16-byte loads whatever the row length, and lays the rows out in LDS with one zero
// column and one zero row between neighbours: that is every plane's padding, so a tap is an LDS
// read at a constant distance and a multiply-add.  A thread keeps one output pixel and walks the
// planes; results leave through LDS with 16-byte stores.  Channels stay in memory order (tap
// positions and weights are looked up per plane), since nothing here branches on the pattern.
// The sums are those of dw_conv_kernel, term by term.
// What bounds it: below about 12 MB of tensors the launch (9 us a pass); above, address arithmetic of
// the LDS layout on both sides, 2.0 to 2.7 TB/s.  The row kernel's lanes load single elements of such rows.
// us per pass, row kernel -> this one, 64 images: 960 channels of 7x7 binary16 15.9 -> 9.2, fp32
// 15.2 -> 9.7; 576 of 14x14 binary16 28.0 -> 15.5, fp32 26.1 -> 17.5, stride 2 17.8 -> 12.5; 96 of 37x35
// binary16 27.9 -> 18.3, fp32 33.9 -> 22.6.
template <int S, class T>
__global__ __launch_bounds__(256) void dw_planes_kernel(DwPlanesArgs<T> a)
{
    extern __shared__ uint4 lds4[];
    constexpr int V = 16 / sizeof(T), AHEAD = 2;
    T* const staged = reinterpret_cast<T*>(lds4);
    T* const result = reinterpret_cast<T*>(lds4 + a.in_units);
    float4* const weights = reinterpret_cast<float4*>(lds4 + a.in_units + a.out_units);
    int4* const info = reinterpret_cast<int4*>(weights + a.planes);   // tap distances (four times 16 bits), bias, removed
    const int tid = threadIdx.x;
    const int g0 = (int)blockIdx.x * a.planes, np = min(a.planes, a.total - g0);
    const int hw = a.h * a.w, px = a.ho * a.wo, pitch = a.w + 1, in_count = np * hw, out_count = np * px;
    const T* src = a.in + (size_t)g0 * hw;
    union Vec { uint4 u; T t[V]; };
    auto load = [&](int i) __attribute__((always_inline)) -> uint4 {
        if ((i + 1) * V <= in_count) return reinterpret_cast<const uint4*>(src)[i];
        Vec v;
        v.u = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int k = 0; k < V; ++k)
            if (i * V + k < in_count) v.t[k] = src[i * V + k];
        return v.u;
    };
    auto scatter = [&](int i, uint4 u) __attribute__((always_inline)) {
        Vec v;
        v.u = u;
        const int e = i * V;
        const int p = (int)fast_div((uint32_t)e, a.div_hw), r = e - p * hw;
        int y = (int)fast_div((uint32_t)r, a.div_w), x = r - y * a.w;
        int at = (p * (a.h + 1) + y + 1) * pitch + x + 1;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (e + k < in_count) staged[at] = v.t[k];
            ++at;
            if (++x == a.w) {
                x = 0;
                ++at;
                if (++y == a.h) { y = 0; at += pitch; }
            }
        }
    };
    const int vecs = (in_count + V - 1) / V;
    uint4 ahead[AHEAD];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k)
        if (tid + k * 256 < vecs) ahead[k] = load(tid + k * 256);
    for (int p = tid; p < np; p += 256) {
        const int co = g0 + p - (int)fast_div((uint32_t)(g0 + p), a.div_c) * a.c;
        const int taps = a.taps[co];
        float4 wv = a.weight[co];
        if constexpr (sizeof(T) == 2) {
            wv.x = __half2float(__float2half_rn(wv.x)); wv.y = __half2float(__float2half_rn(wv.y));
            wv.z = __half2float(__float2half_rn(wv.z)); wv.w = __half2float(__float2half_rn(wv.w));
        }
        auto dist = [&](int k) { const int pos = (taps >> (4 * k)) & 15; return taps < 0 ? 0 : pos / 3 * pitch + pos % 3; };
        weights[p] = wv;
        info[p] = make_int4(dist(0) | dist(1) << 16, dist(2) | dist(3) << 16, __float_as_int(a.bias ? a.bias[co] : 0.0f), taps < 0);
    }
    for (int i = tid; i < a.in_units; i += 256) lds4[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < AHEAD; ++k)
        if (tid + k * 256 < vecs) scatter(tid + k * 256, ahead[k]);
    for (int i = tid + AHEAD * 256; i < vecs; i += 256) scatter(i, load(i));
    __syncthreads();

    // planes with at most 256 outputs: as many at a time as there are threads for
    const int side = px <= 256 ? 256 / px : 1;
    const int mine = px <= 256 ? (int)fast_div((uint32_t)tid, a.div_px) : 0;
    for (int q0 = 0; q0 < px; q0 += 256) {
        const int q = px <= 256 ? tid - mine * px : q0 + tid;
        if (mine < side && q < px) {
            const int oy = (int)fast_div((uint32_t)q, a.div_wo), ox = q - oy * a.wo;
            const int base = (oy * S - a.pad + 1) * pitch + ox * S - a.pad + 1;
#pragma unroll 2
            for (int p = mine; p < np; p += side) {
                const float4 wv = weights[p];
                const int4 in = info[p];
                const T* at = staged + base + p * (a.h + 1) * pitch;
                float acc = fmaf(wv.x, ld1(at + (in.x & 0xFFFF)), 0.0f);
                acc = fmaf(wv.y, ld1(at + (int)((unsigned)in.x >> 16)), acc);
                acc = fmaf(wv.z, ld1(at + (in.y & 0xFFFF)), acc);
                acc = fmaf(wv.w, ld1(at + (int)((unsigned)in.y >> 16)), acc);
                acc = (in.w ? 0.0f : acc) + __int_as_float(in.z);
                if (a.relu) acc = fmaxf(acc, 0.0f);
                st1(result + p * px + q, acc);
            }
        }
    }
    __syncthreads();
    T* dst = a.out + (size_t)g0 * px;
    for (int i = tid; i * V < out_count; i += 256) {
        if ((i + 1) * V <= out_count) {
            reinterpret_cast<uint4*>(dst)[i] = lds4[a.in_units + i];
        } else {
            for (int e = i * V; e < out_count; ++e) dst[e] = result[e];
        }
    }
}

// True where dw_planes_kernel took the layer.
template <class T>
static bool launch_dw_planes(const DevFkw& f, const ConvShape& s, const T* in, const float* bias, T* out, hipStream_t stream)
{
    constexpr int V = 16 / sizeof(T);
    if (!f.dw_taps || s.pad > 1 || ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) != 0) return false;
    const long long hw = (long long)s.h * s.w, px = (long long)s.ho * s.wo, total = (long long)s.n * s.c_out;
    if (total > INT32_MAX - 4096 || hw > 4096) return false;
    // about 6 KB of input: six workgroups and more on a CU at a time, whose loads overlap; fewer
    // planes where that leaves CUs without work
    const long long most = std::max(1ll, std::min({256ll, 6144 / (hw * (long long)sizeof(T)), total / 1024}));
    const long long planes = (most + V - 1) / V * V;
    const long long in_units = (((planes * (s.h + 1) + 1) * (s.w + 1) + 1) * (long long)sizeof(T) + 15) / 16;
    const long long out_units = planes * px / V;
    const long long lds = (in_units + out_units + 2 * planes) * 16;
    // Planes are not cut up: too few workgroups leave CUs idle while the others walk large planes (96
    // channels of 37x35 binary16: 16 images, 192 workgroups 12.7 us against the row kernel's 9.3;
    // 44 images, 528 workgroups 17.4 against 20.8).  Small planes are equal from 256 on
    // (21x21, 384 workgroups: 9.3 and 9.2) and ahead above.
    if (lds > kDwPlanesLds || (total + planes - 1) / planes < (lds > 16 * 1024 ? 512 : 256)) return false;
    DwPlanesArgs<T> a{};
    a.taps = f.dw_taps; a.weight = reinterpret_cast<const float4*>(f.dw_tap_weight);
    a.in = in; a.bias = bias; a.out = out;
    a.c = s.c_out; a.h = s.h; a.w = s.w; a.ho = s.ho; a.wo = s.wo; a.pad = s.pad; a.relu = s.relu;
    a.total = (int32_t)total; a.planes = (int32_t)planes; a.in_units = (int32_t)in_units; a.out_units = (int32_t)out_units;
    a.div_c = make_fast_div((uint32_t)s.c_out);
    a.div_hw = make_fast_div((uint32_t)hw);
    a.div_w = make_fast_div((uint32_t)s.w);
    a.div_px = make_fast_div((uint32_t)px);
    a.div_wo = make_fast_div((uint32_t)s.wo);
    const dim3 grid((unsigned)((total + planes - 1) / planes)), block(256);
    if (s.stride == 1) hipLaunchKernelGGL((dw_planes_kernel<1, T>), grid, block, (size_t)lds, stream, a);
    else hipLaunchKernelGGL((dw_planes_kernel<2, T>), grid, block, (size_t)lds, stream, a);
    return true;
}

template <class T>
static hipError_t launch_dw_t(const DevFkw& f, const T* weights, const ConvShape& s, const T* in, const float* bias,
                              T* out, hipStream_t stream)
{
    DwArgs<T> a{};
    a.reorder = f.reorder; a.dw_mask = f.dw_mask; a.dw_weight = weights;
    a.in = in; a.bias = bias; a.out = out;
    a.c = s.c_out; a.h = s.h; a.w = s.w; a.ho = s.ho; a.wo = s.wo;
    // eight outputs per lane where every row, in and out, is whole vectors of eight elements
    // (more bytes in flight per lane and half the index arithmetic: 3.0 -> 3.5 TB/s from HBM on
    // the 112x112 fp32 layer); not for fp32 at stride 2, where the seventeen columns under
    // eight outputs made the lanes slower; four otherwise
    constexpr uintptr_t kAlign8 = 8 * sizeof(T) - 1;
    const bool wide = (sizeof(T) == 2 || s.stride == 1) && s.w % 8 == 0 && s.wo % 8 == 0 &&
                      ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & kAlign8) == 0;
    const int np = wide ? 8 : 4;
    a.wq = (s.wo + np - 1) / np; a.pad = s.pad; a.relu = s.relu;
    a.total = (long long)s.n * s.c_out * s.ho * a.wq;
    a.div_wq = make_fast_div((uint32_t)a.wq);
    a.div_ho = make_fast_div((uint32_t)a.ho);
    a.div_c = make_fast_div((uint32_t)a.c);
    const long long blocks = (a.total + 255) / 256;
    if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
    // vector loads need every row to start aligned to four elements and to be read in whole
    // vectors: the columns a lane reads beyond its last tap stay inside the row when w % 4 == 0
    constexpr uintptr_t kAlign = 4 * sizeof(T) - 1;
    const bool vec = s.w % 4 == 0 && (reinterpret_cast<uintptr_t>(in) & kAlign) == 0;
    const bool vst = s.wo % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & kAlign) == 0;
    // rows that are whole vectors on the way in stay with the row kernel (192 channels of 28x28 at
    // stride 2, binary16: 11.0 us, 11.3 with planes in LDS)
    if (!vec && launch_dw_planes<T>(f, s, in, bias, out, stream)) return hipGetLastError();
    const dim3 grid((unsigned)blocks), block(256);
    // fp32 outputs that leave nothing in the L2s, and the inputs more room: where both tensors are at most twice the 32 MB of
    // those, and where what this layer and the next one touch exceeds the 256 MB of the last-level cache anyway.  Between
    // them the next layer would find its input there.  us without and with such stores, alone and followed by a layer that
    // reads the output: 144 channels of 56 x 56, 30 MB of output 16.3 and 14.1, 33.8 both; 60 MB 26 both, 52.7 and 58.8; 115 MB
    // on changing tensors 63.3 and 59.4, 120 MB and the next one 112 and 108; 240 MB 127 and 88, 256 and 245.  144 channels of
    // 112 x 112 / 2, 30 MB 28 both, 44.5 and 46.2; 60 MB 60.9 and 48.4, 91.8 and 84.9.
    const size_t in_bytes = (size_t)s.n * s.c_out * s.h * s.w * sizeof(T), out_bytes = (size_t)s.n * s.c_out * s.ho * s.wo * sizeof(T);
    constexpr size_t kMB = (size_t)1 << 20;
    const bool stream_out = sizeof(T) == 4 && out_bytes > 16 * kMB && (in_bytes + out_bytes <= 64 * kMB || in_bytes + 2 * out_bytes > 256 * kMB);
#define PATDNN_DW_LAUNCH(S, NP, V, W) \
    if (W && stream_out) hipLaunchKernelGGL((dw_conv_kernel<S, NP, V, W, T, W && sizeof(T) == 4>), grid, block, 0, stream, a); \
    else hipLaunchKernelGGL((dw_conv_kernel<S, NP, V, W, T, false>), grid, block, 0, stream, a)
    if (wide && s.stride == 1) { PATDNN_DW_LAUNCH(1, 8, true, true); }
    else if (wide) { PATDNN_DW_LAUNCH(2, 8, true, true); }
    else if (s.stride == 1) {
        if (vec && vst) { PATDNN_DW_LAUNCH(1, 4, true, true); }
        else if (vec) { PATDNN_DW_LAUNCH(1, 4, true, false); }
        else if (vst) { PATDNN_DW_LAUNCH(1, 4, false, true); }
        else { PATDNN_DW_LAUNCH(1, 4, false, false); }
    } else {
        if (vec && vst) { PATDNN_DW_LAUNCH(2, 4, true, true); }
        else if (vec) { PATDNN_DW_LAUNCH(2, 4, true, false); }
        else if (vst) { PATDNN_DW_LAUNCH(2, 4, false, true); }
        else { PATDNN_DW_LAUNCH(2, 4, false, false); }
    }
#undef PATDNN_DW_LAUNCH
    return hipGetLastError();
}

hipError_t launch_dw(const DevFkw& f, const ConvShape& s, const float* in, const float* bias,
                     float* out, hipStream_t stream)
{
    return launch_dw_t<float>(f, f.dw_weight, s, in, bias, out, stream);
}

hipError_t launch_dw_f16(const DevFkw& f, const ConvShape& s, const void* in, const float* bias,
                         void* out, hipStream_t stream)
{
    return launch_dw_t<__half>(f, static_cast<const __half*>(f.dw_weight_f16), s, static_cast<const __half*>(in), bias,
                               static_cast<__half*>(out), stream);
}

}  // namespace patdnn
