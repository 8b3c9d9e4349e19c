// Depthwise pattern-pruned 3x3 convolution (the MobileNet-V2 layers the paper evaluates,
// section 6.1): one four-tap kernel per channel, so the layer does about one flop per byte
// and is bound by HBM bandwidth, not by arithmetic.
//
// Design for that bound: one pass over the input and one over the output.  A lane owns
// some neighbouring outputs of two rows (dw_rows_kernel).  Channels are walked in the stored filter
// order of the FKW arrays; for one-kernel filters the filter reorder of section 5.2 sorts
// them by pattern, so the lanes of a wavefront share one pattern and skip the same
// taps together (the `if`s on the pattern mask below are then uniform branches).  Small planes whose rows are
// no whole vectors are taken several at a time through LDS (dw_planes_kernel).
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
    uint32_t div_rows;               // dw_rows_kernel: groups of rows (what div_ho divides by there)
};

// element access: one value, a filter's four weights, or the outputs of a lane at an address aligned to them
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
    typedef unsigned Words __attribute__((ext_vector_type(NP / 2)));
    Words q;
#pragma unroll
    for (int k = 0; k < NP / 2; ++k) q[k] = w[k];
    if constexpr (STREAM) __builtin_nontemporal_store(q, reinterpret_cast<Words*>(p));
    else *reinterpret_cast<Words*>(p) = q;
}

// Any layer: a lane owns four outputs of one row and reads element by element, its row's neighbours again for each of
// three rows.  For what the kernels below leave out: weights that are not finite (rows outside the image are left out
// here, and columns there zeros), rows of fewer than four outputs' columns, 2^31 lanes and more.
template <int S, class T>
__global__ __launch_bounds__(256) void dw_conv_kernel(DwArgs<T> a)
{
    constexpr int NP = 4, NC = (NP - 1) * S + 3;   // outputs, input columns under them
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
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int ix = ix0 + j;
            v[j] = (ix >= 0 && ix < a.w) ? ld1(row + ix) : 0.0f;
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
    T* dst = a.out + (((size_t)n * a.c + co) * a.ho + oy) * (size_t)a.wo + ox0;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        acc[i] += b;
        if (a.relu) acc[i] = fmaxf(acc[i], 0.0f);
        if (ox0 + i < a.wo) st1(dst + i, acc[i]);
    }
}

// A lane owns R rows of V neighbouring outputs and reads the rows under them once, where dw_conv_kernel reads three for
// every row, in vectors of its own columns, and takes the columns beside them from the lanes beside it, which hold
// them.  (A load for each of those is 64 accesses of the texture addresser, as many as two of a row's vectors: that and
// not HBM was the bound of a row kernel of vectors, at 3.9 TB/s.)  WHOLE: padding 1 and rows of whole aligned vectors; otherwise
// rows start anywhere, vectors are accessed at the elements' alignment, and the last lane of a row reads its vector where it ends
// with the row and shifts it.  What bounds it: HBM at the rate of a copy, 144 channels of 56 x 56, 64 images, fp32 on
// changing tensors 231 MB in 47 us, of 112 x 112 / 2 578 MB in 103; binary16 at stride 1 (34 us for 116 MB) conversions and the tap
// branches of eight columns.  R = 2: us of one, two, three and four rows 58, 47, 55, 57 and, of binary16, 37, 34, 34, 36.  (Branches on
// one pattern after the other of a wavefront: 38.)  The sums are those of dw_conv_kernel, term by term; weights are finite
// (rows outside the image are zeros here, not left out).
constexpr int kDwRows = 2;
template <int S, int R, int V, bool WHOLE, class T, bool STREAM>
__global__ __launch_bounds__(256) void dw_rows_kernel(DwArgs<T> a)
{
    constexpr int C = S * V, ROWS = (R - 1) * S + 3;          // own columns, input rows
    constexpr int E = C * (int)sizeof(T) < 16 ? C : 16 / (int)sizeof(T);      // elements of a load
    // (rows that start anywhere: 16- and 8-byte accesses want no more than the elements' alignment)
    typedef unsigned Raw __attribute__((ext_vector_type(E * sizeof(T) / 4), aligned(WHOLE ? E * sizeof(T) : sizeof(T))));
    typedef unsigned RawOut __attribute__((ext_vector_type(V * sizeof(T) / 4), aligned(sizeof(T))));
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    if (t >= (uint32_t)a.total) return;            // whole rows of lanes: the last lane that stays ends one
    const uint32_t r1 = fast_div(t, a.div_wq);
    const int xq = (int)(t - r1 * (uint32_t)a.wq);
    const uint32_t r2 = fast_div(r1, a.div_ho);    // groups of R rows
    const int y0 = (int)(r1 - r2 * a.div_rows) * R;
    const uint32_t n = fast_div(r2, a.div_c);
    const int f = (int)(r2 - n * (uint32_t)a.c);
    const int co = a.reorder[f];
    const unsigned mask = (unsigned)a.dw_mask[f];
    float4 wv;
    ld4(a.dw_weight + (size_t)f * 4, wv.x, wv.y, wv.z, wv.w);
    const int pad = WHOLE ? 1 : a.pad;
    // its first input column, that of tap column 1, and how far before it the columns start that lie in the row
    const int x = xq * C + 1 - pad, shift = WHOLE ? 0 : max(x + C - a.w, 0);
    const size_t plane = (size_t)n * a.c + co;
    const T* const src = a.in + plane * ((size_t)a.h * a.w) + x;
    const int lane = threadIdx.x & 63;
    // the ends of a wavefront have no neighbour, and those of a row none that holds what is there without padding
    const bool left_own = x > 0 && (lane == 0 || xq == 0), right_own = S == 1 && x + C < a.w && (lane == 63 || xq == a.wq - 1);

    // as loaded: a conversion where a row is loaded would wait for each row by itself
    Raw raw[ROWS][C / E];
    T before[ROWS], behind[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int y = y0 * S + r - pad;
#pragma unroll
        for (int k = 0; k < C / E; ++k) raw[r][k] = Raw{};
        before[r] = behind[r] = T(0.0f);
        if (y >= 0 && y < a.h) {
            const T* const row = src + (size_t)y * a.w;
#pragma unroll
            for (int k = 0; k < C / E; ++k) raw[r][k] = *reinterpret_cast<const Raw*>(row - shift + k * E);
            if (left_own) before[r] = row[-1];
            if (right_own) behind[r] = row[C];
        }
    }
    float v[ROWS][C + 2];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
#pragma unroll
        for (int k = 0; k < C / E; ++k) {
            union { Raw u; T t[E]; } m;
            m.u = raw[r][k];
#pragma unroll
            for (int e = 0; e < E; ++e) v[r][k * E + e + 1] = ld1(&m.t[e]);
        }
        if constexpr (!WHOLE) {
#pragma unroll
            for (int d = 1; d < C; d *= 2)
#pragma unroll
                for (int k = 1; k <= C; ++k) v[r][k] = shift & d ? (k + d <= C ? v[r][k + d <= C ? k + d : 0] : 0.0f) : v[r][k];
        }
        const float left = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[r][C]), 0x138, 0xf, 0xf, false));       // wave_shr:1
        v[r][0] = xq == 0 || left_own ? ld1(&before[r]) : left;
        if constexpr (S == 1) {
            const float right = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[r][1]), 0x130, 0xf, 0xf, false));  // wave_shl:1
            v[r][C + 1] = xq == a.wq - 1 || right_own ? ld1(&behind[r]) : right;
        }
    }
    float acc[R][V];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < V; ++i) acc[r][i] = 0.0f;
#pragma unroll
    for (int pos = 0; pos < 9; ++pos) {
        if (!(mask >> pos & 1u)) continue;
        const int rank = __builtin_popcount(mask & ((1u << pos) - 1u));
        const float wt = rank == 0 ? wv.x : rank == 1 ? wv.y : rank == 2 ? wv.z : wv.w;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < V; ++i) acc[r][i] = fmaf(wt, v[r * S + pos / 3][i * S + pos % 3], acc[r][i]);
    }
    const float b = a.bias ? a.bias[co] : 0.0f;
    T* const dst = a.out + plane * ((size_t)a.ho * a.wo) + xq * V;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (y0 + r >= a.ho) break;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            acc[r][i] += b;
            if (a.relu) acc[r][i] = fmaxf(acc[r][i], 0.0f);
        }
        T* const row = dst + (size_t)(y0 + r) * a.wo;
        if (WHOLE) {
            stv<STREAM, V>(row, acc[r]);
        } else if (xq * V + V <= a.wo) {
            union { RawOut u; T t[V]; } m;
#pragma unroll
            for (int i = 0; i < V; ++i) st1(&m.t[i], acc[r][i]);
            *reinterpret_cast<RawOut*>(row) = m.u;
        } else {
#pragma unroll
            for (int i = 0; i < V - 1; ++i)
                if (xq * V + i < a.wo) st1(row + i, acc[r][i]);
        }
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
// What bounds it: below about 12 MB of tensors the launch (8 us a pass); above, address arithmetic of
// the LDS layout on both sides, 2.0 to 2.7 TB/s.
// us per pass, a kernel of single elements -> this one, 64 images: 960 channels of 7x7 binary16 15.9 -> 9.2, fp32
// 15.2 -> 9.7 (7.8 and 8.2 since a call from Python makes no Stream object).
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

// True where dw_planes_kernel takes the layer, with no more than `most_lds` bytes a workgroup, which it then does if `run`.
template <class T>
static bool launch_dw_planes(const DevFkw& f, const ConvShape& s, const T* in, const float* bias, T* out, long long most_lds, hipStream_t stream, bool run)
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
    // Planes are not cut up: too few workgroups leave CUs idle while the others walk large planes.  Against single elements, us
    // of this kernel over those: up to 16 KB from 512 workgroups on (fewer take no longer than a launch) 0.59 to 1.01 times, 16 to 32 KB from
    // 512 on 0.42 to 1.11, 384 to 511 0.86 to 1.25; 32 to 52 KB from 512 on 0.66 to 1.05, below 0.77 to 1.47 (174 layers of up to
    // seven columns).
    if (lds > most_lds || (total + planes - 1) / planes < (lds > 16 * 1024 ? 512 : 256)) return false;
    if (!run) return true;
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

// Not 0 where dw_rows_kernel, or dw_planes_kernel in its place, takes the layer (see dw_choice).  us of the kernels before -> of this one, on changing tensors, 64 images unless
// said: fp32 144 channels of 56 x 56 60 -> 47, 8 images 9.5 -> 7.2, one 6.8 both; 96 of 112 x 112 156 -> 106; 96 of 37 x 35 23.7 ->
// 15.0; 144 of 57 x 61, 16 images 40 -> 12.8; 144 of 112 x 112 / 2 120 -> 103; 75 x 110 / 2 9.7 -> 7.4; binary16 56 x 56 42 -> 33, 60 x 58 120 ->
// 52, 112 x 112 / 2 77 -> 59.  Rows of up to 12 elements that are not whole stay with dw_planes_kernel, whose 16-byte loads they
// leave idle less (400 channels of 9 x 9 7.7 there, 8.0 here, 10 x 10 9.3 and 10.0, 11 x 11 10.8 and 11.9, 13 x 13 13.6 and 10.3),
// where a workgroup's planes take up to 18 KB of LDS: of 491 layers that take more than a launch the two are even there (0.70 to 1.33),
// from 24 to 40 KB, tall planes, dw_planes_kernel takes 1.18 times as long (0.79 to 1.59), above 1.36 (0.89 to 2.01).
template <class T>
static int launch_dw_rows(const DevFkw& f, const ConvShape& s, DwArgs<T> a, hipStream_t stream, bool run)
{
    constexpr int kWide = 16 / sizeof(T);
    const uintptr_t at = reinterpret_cast<uintptr_t>(a.in) | reinterpret_cast<uintptr_t>(a.out);
    if (!(sizeof(T) == 4 ? f.dw_finite : f.dw_taps != nullptr) || s.stride > 2 || s.pad > 1 || s.w < 4 * s.stride) return 0;
    // outputs of a lane: four, or a whole vector; at stride 2 the columns of four are one or two
    const int v = s.stride == 1 && s.pad == 1 && s.w % kWide == 0 && (at & 15) == 0 ? kWide : 4;
    const bool whole = s.pad == 1 && s.w % (v * s.stride) == 0 && (at & std::min<size_t>(15, v * s.stride * sizeof(T) - 1)) == 0;
    if (!whole && s.w <= 12 && launch_dw_planes<T>(f, s, a.in, a.bias, a.out, 18 * 1024, stream, run)) return 1;
    a.wq = (s.wo + v - 1) / v;
    a.div_rows = (uint32_t)(s.ho + kDwRows - 1) / kDwRows;
    a.total = (long long)s.n * s.c_out * a.div_rows * a.wq;
    if (a.total > INT32_MAX - 256) return 0;
    a.div_wq = make_fast_div((uint32_t)a.wq);
    a.div_ho = make_fast_div(a.div_rows);
    a.div_c = make_fast_div((uint32_t)a.c);
    // Outputs that leave nothing in the L2s, where both tensors exceed the last-level cache and rows are most of two cache lines:
    // 96 channels of 112 x 112, alone / followed by a layer that reads the output, 109 / 219 us without, 106 / 211 with, binary16
    // 72.7 / 148 and 70.8 / 142; below that size 144 channels of 56 x 56, 64 images 47.6 / 91.6 and 46.9 / 94.2; 576 of 28 x 28 54 / 96
    // and 60 / 120.
    const size_t bytes = (size_t)s.n * s.c_out * s.h * s.w * sizeof(T);
    const bool past = s.stride == 1 && whole && 2 * bytes > (size_t)256 << 20 && s.w * sizeof(T) >= 224;
    const int choice = 2 + whole + 2 * (v == 8) + 4 * past;
    if (!run) return choice;
    const dim3 grid((unsigned)((a.total + 255) / 256)), block(256);
    const auto kernel = s.stride == 2 ? (whole ? &dw_rows_kernel<2, kDwRows, 4, true, T, false> : &dw_rows_kernel<2, kDwRows, 4, false, T, false>)
                        : !whole      ? &dw_rows_kernel<1, kDwRows, 4, false, T, false>
                        : v == kWide  ? (past ? &dw_rows_kernel<1, kDwRows, kWide, true, T, true> : &dw_rows_kernel<1, kDwRows, kWide, true, T, false>)
                                      : (past ? &dw_rows_kernel<1, kDwRows, 4, true, T, true> : &dw_rows_kernel<1, kDwRows, 4, true, T, false>);
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, a);
    return choice;
}

template <class T>
static hipError_t launch_dw_t(const DevFkw& f, const T* weights, const ConvShape& s, const T* in, const float* bias,
                              T* out, hipStream_t stream, bool run, int& choice)
{
    DwArgs<T> a{};
    a.reorder = f.reorder; a.dw_mask = f.dw_mask; a.dw_weight = weights;
    a.in = in; a.bias = bias; a.out = out;
    a.c = s.c_out; a.h = s.h; a.w = s.w; a.ho = s.ho; a.wo = s.wo; a.pad = s.pad; a.relu = s.relu;
    choice = launch_dw_rows<T>(f, s, a, stream, run);
    if (!choice && s.w % 4 != 0 && launch_dw_planes<T>(f, s, in, bias, out, kDwPlanesLds, stream, run)) choice = 1;
    if (choice || !run) return run ? hipGetLastError() : hipSuccess;
    a.wq = (s.wo + 3) / 4;
    a.total = (long long)s.n * s.c_out * s.ho * a.wq;
    a.div_wq = make_fast_div((uint32_t)a.wq);
    a.div_ho = make_fast_div((uint32_t)a.ho);
    a.div_c = make_fast_div((uint32_t)a.c);
    const long long blocks = (a.total + 255) / 256;
    if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
    const auto kernel = s.stride == 1 ? &dw_conv_kernel<1, T> : &dw_conv_kernel<2, T>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_dw(const DevFkw& f, const ConvShape& s, const float* in, const float* bias,
                     float* out, hipStream_t stream)
{
    int choice = 0;
    return launch_dw_t<float>(f, f.dw_weight, s, in, bias, out, stream, true, choice);
}

hipError_t launch_dw_f16(const DevFkw& f, const ConvShape& s, const void* in, const float* bias,
                         void* out, hipStream_t stream)
{
    int choice = 0;
    return launch_dw_t<__half>(f, static_cast<const __half*>(f.dw_weight_f16), s, static_cast<const __half*>(in), bias,
                               static_cast<__half*>(out), stream, true, choice);
}

int dw_choice(const DevFkw& f, const ConvShape& s, const void* in, const void* out, bool half)
{
    int choice = 0;
    if (half) launch_dw_t<__half>(f, nullptr, s, static_cast<const __half*>(in), nullptr, static_cast<__half*>(const_cast<void*>(out)), nullptr, false, choice);
    else launch_dw_t<float>(f, nullptr, s, static_cast<const float*>(in), nullptr, static_cast<float*>(const_cast<void*>(out)), nullptr, false, choice);
    return choice;
}

}  // namespace patdnn
