// C ABI of the library (see include/patdnn.h): handle management, upload of the
// encoded layouts, variant selection, launch, decode, tuning.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iterator>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "kernels.hpp"
#include "layout.hpp"

using namespace patdnn;

namespace {

thread_local std::string g_err;

// Nothing leaves the C interface as an exception: a text that finds no memory is dropped, ...
template <class... Parts>
patdnn_status_t fail(patdnn_status_t s, const Parts&... parts)
{
    try {
        g_err.clear();
        (g_err.append(parts), ...);
    } catch (const std::bad_alloc&) {
        g_err.clear();
    }
    return s;
}

patdnn_status_t hip_fail(hipError_t e, const char* what) { return fail(PATDNN_EHIP, what, ": ", hipGetErrorString(e)); }

// ... and an entry point whose work allocates runs it in here.
template <class F>
patdnn_status_t guarded(F&& work)
{
    try {
        return work();
    } catch (const std::bad_alloc&) {
        return fail(PATDNN_ENOMEM, "out of host memory");
    }
}

}  // namespace

namespace patdnn {
void set_last_error(const std::string& msg) { g_err = msg; }     // for the other translation units
}

namespace {

struct TiledOnDevice {
    Tiled host;
    DevTiled dev;
    std::vector<void*> allocations;       // device arrays of this layout
    ~TiledOnDevice()
    {
        for (void* p : allocations) (void)hipFree(p);
    }
};

struct TapsOnDevice {
    Taps host;                            // its arrays are on the device only
    size_t bytes = 0;                     // of the arrays
    DevTaps dev;
    std::vector<void*> allocations;
    ~TapsOnDevice()
    {
        for (void* p : allocations) (void)hipFree(p);
    }
};

}  // namespace

struct patdnn_layer {
    LayerHost L;
    bool on_device = false;
    bool dense_mfma = false;                               // the kernel of dense layers of few channels runs this one
    bool split = false;                                    // the weights as pairs of binary16 numbers exist
    std::vector<int32_t> split_filters;                    // of those
    int device = -1;
    DevFkw dfkw;
    // by (variant index, ck); dense variants use ck = 0
    std::map<std::pair<int, int>, std::unique_ptr<TiledOnDevice>> tiled;
    std::map<int, std::unique_ptr<TapsOnDevice>> taps;     // tap-product layouts by ck
    std::vector<int32_t> tap_groups;                       // the filter groups they share
    std::vector<int> order;                                // tiled variants that can run the layer, as they are tried
    std::vector<void*> allocations;
    // the comparison kernels' layouts (built when such a variant is first selected)
    struct CompareHost {
        std::vector<int32_t> row_ptr, col, kmask;
        std::vector<float> val;
    } noopt_host, csr_host;
    DevCompare noopt_dev, csr_dev;
    bool compare_built = false, compare_on_device = false;
    patdnn_config_t cfg{-1, 0, 0, 1};                      // variant -1: choose per call
    bool cfg_tuned = false;                                // cfg came from patdnn_tune (for one input size)

    ~patdnn_layer()
    {
        for (void* p : allocations) (void)hipFree(p);
    }
};

namespace {

// Host arrays on their way to the device: one allocation for all of them, and one copy where they are
// small - an allocation and a copy take some 15 us whatever their size, and a layer has two dozen arrays.
class Upload {
public:
    // `v` must stay as it is until commit(), which sets *out (NULL for an empty array)
    template <class T>
    void add(const std::vector<T>& v, const T** out)
    {
        place(v.data(), v.size() * sizeof(T), out);
    }
    // room for `count` elements that a kernel will write
    template <class T>
    void room(size_t count, const T** out)
    {
        place(nullptr, count * sizeof(T), out);
    }
    hipError_t commit(std::vector<void*>& owner)
    {
        if (!total) return hipSuccess;
        owner.reserve(owner.size() + 1);
        void* p = nullptr;
        hipError_t e = hipMalloc(&p, total);
        if (e != hipSuccess) return e;
        owner.push_back(p);
        char* const dev = static_cast<char*>(p);
        const bool together = copied <= 256 * 1024;
        std::vector<char> stage(together ? copied : 0);
        for (const Item& i : items) {
            if (i.src && together) std::memcpy(&stage[i.at], i.src, i.bytes);
            else if (i.src && (e = hipMemcpy(dev + i.at, i.src, i.bytes, hipMemcpyHostToDevice)) != hipSuccess) return e;
            i.set(i.out, dev + i.at);
        }
        return stage.empty() ? hipSuccess : hipMemcpy(dev, stage.data(), stage.size(), hipMemcpyHostToDevice);
    }

private:
    struct Item {
        const void* src;
        size_t bytes, at;
        void* out;
        void (*set)(void* out, void* device);
    };
    template <class T>
    void place(const void* src, size_t bytes, const T** out)
    {
        *out = nullptr;
        if (!bytes) return;
        items.push_back(Item{src, bytes, total, out, [](void* o, void* d) { *static_cast<const T**>(o) = static_cast<const T*>(d); }});
        if (src) copied = total + bytes;
        total = (total + bytes + 255) / 256 * 256;
    }
    std::vector<Item> items;
    size_t total = 0, copied = 0;             // bytes of the allocation; up to the end of the last array that is copied
};

bool variant_fits_layer(const patdnn_layer* h, const TiledVariant& v)
{
    const LayerHost& L = h->L;
    if (L.depthwise) return false;
    if (v.dense != L.dense) return false;
    if (v.S != L.desc.stride) return false;
    if (!L.dense && !L.all_in_universe) return false;
    if (L.desc.c_in > 65535) return false;
    return true;
}

// Variants marked experimental have passed the host model of the interpreter but have not
// been measured on hardware; they run only when the caller asks for them by number AND the
// environment carries PATDNN_EXPERIMENTAL=1.
bool experimental_allowed()
{
    const char* e = std::getenv("PATDNN_EXPERIMENTAL");
    return e && e[0] == '1' && e[1] == 0;
}

bool variant_selectable(const patdnn_layer* h, const TiledVariant& v)
{
    return variant_fits_layer(h, v) && !v.experimental;
}

// Variant numbers: 0 the FKW walk, 1..T the tiled variants, then the kernels below.
enum ExtraVariant { kExtraDepthwise = 0, kExtraNoopt, kExtraCsr, kExtraTaps8, kExtraTaps16, kExtraSplit, kExtraDense, kNumExtra };
int extra_variant(int variant) { return variant - 1 - num_tiled_variants(); }     // < 0: not one
int variant_of_extra(int extra) { return 1 + num_tiled_variants() + extra; }
const char* const kExtraNames[kNumExtra] = {"dw_p1x4", "noopt", "csr", "taps_f8", "taps_f16", "split_f16", "dense_mfma"};
// filters per wavefront of a tap-product variant, 0 for any other
int taps_filters(int variant)
{
    return extra_variant(variant) == kExtraTaps8 ? 8 : extra_variant(variant) == kExtraTaps16 ? 16 : 0;
}

constexpr int kMaxLdsBytes = 160 * 1024;      // LDS of one CU; two staging buffers must fit
constexpr int kMaxWaves = 8;

int default_ck(const TiledVariant& v, int c_in)
{
    const int max_ck = kMaxLdsBytes / (4 * v.lds_buffers * v.lds_floats_per_channel);
    return std::max(1, std::min(std::min(8, max_ck), c_in));
}

// Smallest / default launch parameters of a tiled variant for this layer; false if
// the variant cannot run at all.
bool resolve_tiled_params(const patdnn_layer* h, const TiledVariant& v, const ConvShape& s,
                          int32_t& ck, int32_t& waves)
{
    const int num_groups = (h->L.desc.c_out + v.G - 1) / v.G;
    const int min_waves = (v.stage_elems + 64 * v.max_slots - 1) / (64 * v.max_slots);
    if (min_waves > kMaxWaves) return false;
    if (waves <= 0) waves = std::max(min_waves, std::min(num_groups, 4));
    if (waves < min_waves || waves > kMaxWaves) return false;
    const int max_ck = kMaxLdsBytes / (4 * v.lds_buffers * v.lds_floats_per_channel);
    if (max_ck < 1) return false;
    if (ck <= 0) ck = default_ck(v, s.c_in);
    if (ck < 1 || ck > max_ck) return false;
    // staging offsets are 32-bit byte offsets relative to the first image of a tile
    const int nb = 64 / v.TGX;
    const long long span = (long long)(nb + 1) * s.c_in * s.h * s.w;
    if (span >= (1ll << 30)) return false;
    return true;
}

patdnn_status_t ensure_tiled(patdnn_layer* h, int vi, int ck, const DevTiled** out)
{
    const TiledVariant& v = tiled_variant(vi);
    if (v.dense) ck = 0;
    const std::pair<int, int> key(vi, ck);
    auto it = h->tiled.find(key);
    if (it == h->tiled.end()) {
        if (v.threaded && h->on_device) {
            std::string why;
            if (!movrel_selftest(why)) return fail(PATDNN_EUNSUPPORTED, "threaded variants are off: ", why);
        }
        std::unique_ptr<TiledOnDevice> t(new (std::nothrow) TiledOnDevice());
        if (!t) return fail(PATDNN_ENOMEM, "out of host memory");
        TiledParams prm;
        prm.G = v.G;
        prm.ck = ck;
        prm.block_bytes = v.block_bytes;
        prm.table_off = v.table_off;
        prm.ctrl_bytes = v.ctrl_bytes;
        prm.records = v.records;
        prm.double_window = v.double_window;
        prm.threaded = v.threaded;
        prm.channel_bytes = 4u * (uint32_t)v.lds_floats_per_channel;
        build_tiled(h->L, prm, t->host);
        if (t->host.overflow) return fail(PATDNN_EUNSUPPORTED, "layer has too many steps for this variant");
        t->dev.G = v.G;
        t->dev.num_groups = t->host.num_groups;
        t->dev.ck = ck;
        t->dev.num_chunks = t->host.num_chunks;
        if (h->on_device) {
            Upload up;
            up.add(t->host.slot_channel, &t->dev.slot_channel);
            up.add(t->host.chunk_ptr, &t->dev.chunk_ptr);
            up.add(t->host.steps, &t->dev.steps);
            up.add(t->host.w9, &t->dev.w9);
            const hipError_t e = up.commit(t->allocations);
            if (e != hipSuccess) return hip_fail(e, "uploading the tiled layout");
        }
        it = h->tiled.emplace(key, std::move(t)).first;
    }
    if (out) *out = &it->second->dev;
    return PATDNN_OK;
}

constexpr int kMaxTapWaves = 16;

bool taps_fit_layer(const patdnn_layer* h)
{
    const LayerHost& L = h->L;
    return !L.depthwise && !L.dense && L.all_in_universe && L.desc.stride == 1;
}

// The chunk sizes whose layouts every handle holds: equal chunks of at most 128 channels (a flush
// per filter and pattern in every chunk, so the fewer chunks the better; 128 KB of LDS), half and a
// quarter of that for launches that split the channels over workgroups.
int taps_ck(int c_in, int level)
{
    const int chunks = ((c_in + 127) / 128) << level;
    return (c_in + chunks - 1) / chunks;
}
constexpr int kTapLevels = 3, kMinTapChunk = 8;

patdnn_status_t ensure_taps(patdnn_layer* h, int ck, const DevTaps** out)
{
    auto it = h->taps.find(ck);
    if (it == h->taps.end()) {
        std::unique_ptr<TapsOnDevice> t(new (std::nothrow) TapsOnDevice());
        if (!t) return fail(PATDNN_ENOMEM, "out of host memory");
        if (h->tap_groups.empty()) h->tap_groups = taps_groups(h->L, taps_ck(h->L.desc.c_in, 1));
        build_taps(h->L, ck, h->tap_groups, t->host);
        t->dev.num_groups = t->host.num_groups;
        t->dev.ck = ck;
        t->dev.num_chunks = t->host.num_chunks;
        if (h->on_device) {
            Upload up;
            up.add(t->host.slot_channel, &t->dev.slot_channel);
            up.add(t->host.chunk_ptr, &t->dev.chunk_ptr);
            up.add(t->host.records, &t->dev.records);
            up.add(t->host.weights, &t->dev.weights);
            const hipError_t e = up.commit(t->allocations);
            if (e != hipSuccess) return hip_fail(e, "uploading the tap-product layout");
        }
        t->bytes = t->host.bytes();
        // the planner needs the numbers only
        t->host.slot_channel = std::vector<int32_t>();
        t->host.chunk_ptr = t->host.records = std::vector<uint32_t>();
        t->host.weights = std::vector<float>();
        it = h->taps.emplace(ck, std::move(t)).first;
    }
    if (out) *out = &it->second->dev;
    return PATDNN_OK;
}

// The layer before filter-kernel reorder (filters in original order, kernels by input
// channel, a pattern mask per kernel) and as a CSR matrix [c_out][c_in*9], both derived from
// the FKW arrays by undoing the reorder.
patdnn_status_t ensure_compare(patdnn_layer* h)
{
    if (h->L.depthwise || h->L.dense) return fail(PATDNN_EUNSUPPORTED, "the comparison kernels run pruned, non-depthwise layers");
    if (!h->compare_built) {
        const Fkw& f = h->L.fkw;
        const int c_out = h->L.desc.c_out, P = f.num_patterns;
        struct K { int32_t ci; int32_t mask; const float* w; };
        std::vector<std::vector<K>> per_filter((size_t)c_out);
        for (int s = 0; s < c_out; ++s) {
            const int32_t* st = &f.stride[(size_t)s * (P + 1)];
            for (int p = 0; p < P; ++p)
                for (int32_t k = f.offset[s] + st[p]; k < f.offset[s] + st[p + 1]; ++k)
                    per_filter[(size_t)f.reorder[s]].push_back(K{f.index[k], (int32_t)f.masks[p], &f.weight[(size_t)k * 4]});
        }
        auto& no = h->noopt_host = patdnn_layer::CompareHost();
        auto& cs = h->csr_host = patdnn_layer::CompareHost();
        no.row_ptr.assign(1, 0);
        cs.row_ptr.assign(1, 0);
        for (int co = 0; co < c_out; ++co) {
            auto& ks = per_filter[(size_t)co];
            std::sort(ks.begin(), ks.end(), [](const K& a, const K& b) { return a.ci < b.ci; });
            for (const K& k : ks) {
                no.col.push_back(k.ci);
                no.kmask.push_back(k.mask);
                int t = 0;
                for (int pos = 0; pos < 9; ++pos)
                    if ((k.mask >> pos) & 1) {
                        no.val.push_back(k.w[t]);
                        cs.col.push_back(k.ci * 9 + pos);
                        cs.val.push_back(k.w[t]);
                        ++t;
                    }
            }
            no.row_ptr.push_back((int32_t)no.col.size());
            cs.row_ptr.push_back((int32_t)cs.col.size());
        }
        h->compare_built = true;
    }
    if (h->on_device && !h->compare_on_device) {
        Upload up;
        up.add(h->noopt_host.row_ptr, &h->noopt_dev.row_ptr);
        up.add(h->noopt_host.col, &h->noopt_dev.col);
        up.add(h->noopt_host.kmask, &h->noopt_dev.kmask);
        up.add(h->noopt_host.val, &h->noopt_dev.val);
        up.add(h->csr_host.row_ptr, &h->csr_dev.row_ptr);
        up.add(h->csr_host.col, &h->csr_dev.col);
        up.add(h->csr_host.val, &h->csr_dev.val);
        const hipError_t e = up.commit(h->allocations);
        if (e != hipSuccess) return hip_fail(e, "uploading the comparison layouts");
        h->compare_on_device = true;
    }
    return PATDNN_OK;
}

patdnn_status_t shape_of(const patdnn_layer* h, int32_t n, int32_t h_in, int32_t w_in, ConvShape& s)
{
    if (!h) return fail(PATDNN_EINVAL, "handle is NULL");
    if (n < 0 || h_in <= 0 || w_in <= 0) return fail(PATDNN_EINVAL, "n must be >= 0 and h_in, w_in positive");
    const auto& d = h->L.desc;
    s.n = n; s.c_in = d.c_in; s.c_out = d.c_out; s.h = h_in; s.w = w_in;
    s.stride = d.stride; s.pad = d.pad;
    s.ho = (h_in + 2 * d.pad - 3) / d.stride + 1;
    s.wo = (w_in + 2 * d.pad - 3) / d.stride + 1;
    s.relu = 0;
    if (h_in + 2 * d.pad < 3 || w_in + 2 * d.pad < 3 || s.ho <= 0 || s.wo <= 0)
        return fail(PATDNN_EINVAL, "input smaller than the 3x3 kernel");
    if ((long long)d.c_in * h_in * w_in > INT32_MAX || (long long)d.c_out * s.ho * s.wo > INT32_MAX)
        return fail(PATDNN_EUNSUPPORTED, "more than 2^31-1 elements per image");
    return PATDNN_OK;
}

int taps_parts(const patdnn_layer* h, const Taps& t, const ConvShape& s, int waves, int ksplit);

// Launch with an explicit configuration (variant >= 0).
patdnn_status_t run_config(patdnn_layer* h, const patdnn_config_t& c, const ConvShape& s,
                           const float* in, const float* bias, float* out, hipStream_t stream,
                           float* scratch = nullptr, size_t scratch_floats = 0)
{
    if (c.variant == PATDNN_VARIANT_FKW) {
        hipError_t e = launch_fkw(h->dfkw, s, in, bias, out, stream);
        return e == hipSuccess ? PATDNN_OK : hip_fail(e, "launching the FKW kernel");
    }
    if (extra_variant(c.variant) == kExtraDepthwise) {
        if (!h->L.depthwise) return fail(PATDNN_EUNSUPPORTED, "the depthwise kernel runs depthwise layers only");
        hipError_t e = launch_dw(h->dfkw, s, in, bias, out, stream);
        return e == hipSuccess ? PATDNN_OK : hip_fail(e, "launching the depthwise kernel");
    }
    if (extra_variant(c.variant) == kExtraNoopt || extra_variant(c.variant) == kExtraCsr) {
        if (!h->compare_on_device) return fail(PATDNN_EUNSUPPORTED, "select the comparison kernel with patdnn_set_config first");
        if (s.pool) return fail(PATDNN_EUNSUPPORTED, "the comparison kernels have no pooled epilogue");
        const bool csr = extra_variant(c.variant) == kExtraCsr;
        hipError_t e = launch_compare(csr, csr ? h->csr_dev : h->noopt_dev, s, in, bias, out, stream);
        return e == hipSuccess ? PATDNN_OK : hip_fail(e, "launching a comparison kernel");
    }
    if (extra_variant(c.variant) == kExtraSplit) {
        if (!h->dfkw.split_f16) return fail(PATDNN_EUNSUPPORTED, "variant cannot run this layer");
        int rounds = 0, steps = 0, pixels = 0;
        if (!split_cost(s, rounds, steps, pixels)) return fail(PATDNN_EUNSUPPORTED, "input too large for the split kernel");
        hipError_t e = launch_split(h->dfkw, s, in, bias, out, stream);
        return e == hipSuccess ? PATDNN_OK : hip_fail(e, "launching the split kernel");
    }
    if (extra_variant(c.variant) == kExtraDense) {
        if (!h->dense_mfma) return fail(PATDNN_EUNSUPPORTED, "variant cannot run this layer");
        if (!dense_fits(s)) return fail(PATDNN_EUNSUPPORTED, "input too large for the dense kernel");
        hipError_t e = launch_dense(h->dfkw, s, in, bias, out, stream);
        return e == hipSuccess ? PATDNN_OK : hip_fail(e, "launching the dense kernel");
    }
    if (const int filters = taps_filters(c.variant)) {
        auto it = h->taps.find(c.ck);
        if (it == h->taps.end()) return fail(PATDNN_EUNSUPPORTED, "no layout for this ck: choose it with patdnn_set_config");
        if (!taps_fit_input(s)) return fail(PATDNN_EUNSUPPORTED, "input too large for the tap-product kernel");
        const int parts = filters == 16 ? 1 : taps_parts(h, it->second->host, s, c.waves, c.ksplit);
        hipError_t e = launch_taps(filters / parts, it->second->dev, s, in, bias, out, c.waves * parts, c.ksplit, scratch, scratch_floats, stream);
        return e == hipSuccess ? PATDNN_OK : hip_fail(e, "launching the tap-product kernel");
    }
    const int vi = c.variant - 1;
    if (vi < 0 || vi >= num_tiled_variants()) return fail(PATDNN_EINVAL, "no such variant");
    const TiledVariant& v = tiled_variant(vi);
    if (!variant_fits_layer(h, v)) return fail(PATDNN_EUNSUPPORTED, "variant cannot run this layer");
    if (v.experimental && !experimental_allowed())
        return fail(PATDNN_EUNSUPPORTED, "experimental variant: set PATDNN_EXPERIMENTAL=1 to run it");
    if (c.ksplit > 1 && v.dense) return fail(PATDNN_EUNSUPPORTED, "ksplit is for sparse variants");
    int32_t ck = c.ck, waves = c.waves;
    if (!resolve_tiled_params(h, v, s, ck, waves))
        return fail(PATDNN_EUNSUPPORTED, "launch parameters outside the variant's limits");
    const DevTiled* t = nullptr;
    // the layout of (variant, ck) is built by encode / set_config / tune, never here
    auto it = h->tiled.find(std::make_pair(vi, v.dense ? 0 : ck));
    if (it == h->tiled.end())
        return fail(PATDNN_EUNSUPPORTED, "no layout for this ck: choose it with patdnn_set_config");
    t = &it->second->dev;
    DevTiled dt = *t;
    if (v.dense) { dt.ck = ck; dt.num_chunks = (s.c_in + ck - 1) / ck; }
    if (c.ksplit > dt.num_chunks) return fail(PATDNN_EUNSUPPORTED, "ksplit exceeds the number of channel chunks");
    hipError_t e = v.launch(dt, s, in, bias, out, waves, c.ksplit, scratch, scratch_floats, stream);
    return e == hipSuccess ? PATDNN_OK : hip_fail(e, "launching a tiled kernel");
}

// Tiled variants that can run the layer, in the order in which it tries them when nothing is
// configured: first the variant that the tuner prefers on most measured layers (threaded dispatch,
// 7x2 patch, one staging buffer; it needs the scalar relative moves that the self-test checks on the
// device), then the order of variants.def, whose first line (call dispatch) has no such requirement.
// Worked out once per handle: a call allocates nothing.
std::vector<int> default_variant_order(const patdnn_layer* h)
{
    std::vector<int> order;
    for (int vi = 0; vi < num_tiled_variants(); ++vi)
        if (std::string(tiled_variant(vi).name) == "t_g8_p7x2_s1_x8_thw1b") {
            std::string why;
            if (variant_selectable(h, tiled_variant(vi)) && (!h->on_device || movrel_selftest(why))) order.push_back(vi);
        }
    for (int vi = 0; vi < num_tiled_variants(); ++vi)
        if (variant_selectable(h, tiled_variant(vi)) && (order.empty() || vi != order[0])) order.push_back(vi);
    return order;
}

// Partial sums that the library asks room for by itself: 512 MB.
constexpr size_t kMaxSliceFloats = (size_t)128 << 20;

// ---- the configuration used when the caller has not chosen or tuned one: the candidate with the
// smallest estimate of its time.  The estimates are a few products; their constants were fitted to
// measurements of layers from 16 to 512 channels, 7x7 to 224x224 pixels and 1 to 64 images in every
// candidate configuration; on 80 layers of 6 to 56 patterns (profiles/planner_choice.txt) the
// chosen candidate is 5.0 % slower than the fastest one on average (median 1.2 %) without a workspace, 7.0 % (3.2 %) with one,
// and at most 2.1 times as slow, a layer of 56 patterns in 43 small images that the split kernel would run, less exactly.

// Tap-product kernel, microseconds, for workgroups of `waves` wavefronts of `filters` filters.  Workgroups of one round
// share a CU as far as LDS and registers allow; `share` is what a wavefront's work costs when so many sit on a SIMD (one alone
// leaves the matrix core waiting for it), where more than three of a workgroup are counted from the first SIMD on.  What a
// workgroup reads and writes is not hidden by its own computation, only by another workgroup on the CU, and few wavefronts
// stage a chunk longer.  (770 layers in every configuration, on the same tensors each time: the one with the smallest estimate is
// 2.5 % behind the fastest on average, with five wavefronts of 98 registers on a SIMD and five chunks of 32 KB in LDS 3.6 %; 440
// of them on changing tensors, which cost large chunks most, 1.8 %, and at most 24 %.)
struct TapsEstimate {
    double groups, tiles, kernels, in_mb, again_mb, out_mb;
    int ck, num_chunks, chunks_in_lds;
    TapsEstimate(const patdnn_layer* h, const Taps& t, const ConvShape& s, double tiles_)
        : groups(t.num_groups), tiles(tiles_), kernels((46.7 * h->L.kept + 92.0 * t.segments) / s.c_out / t.num_chunks + 93.0),
          in_mb(4e-6 * s.n * s.c_in * s.h * s.w), again_mb(0.665 * in_mb * in_mb / (in_mb + 3.0)),    // few megabytes come from the L2s
          out_mb(4e-6 * s.n * s.c_out * s.ho * s.wo), ck(t.ck), num_chunks(t.num_chunks),
          chunks_in_lds(128 / ((4 * t.ck + 4) / 5))                       // of 1 KB a channel, in units of 1280 bytes: four of 32 channels, not five
    {
    }
    double sets(int filters, int waves) const { return (double)(((int)groups * kTapGroup + waves * filters - 1) / (waves * filters)); }
    // of a launch whose wavefronts have a whole group
    double wavefronts(int waves, int ksplit) const { return tiles * sets(kTapGroup, waves) * ksplit * waves; }
    // (a hundred of these in a call: no 64-bit divisions, no library calls)
    double operator()(int filters, int waves, int ksplit) const
    {
        const double sets = this->sets(filters, waves), blocks = tiles * sets * ksplit;
        // wavefronts that a SIMD has registers for: 128 each, or 98 for eight and four filters (five fit with 96, and those whose slices
        // leave bias and pooling to another kernel need no more)
        const int simd = filters == 16 || (filters != 2 && ksplit == 1) ? 4 : 5;
        const int resident = std::max(1, std::min(chunks_in_lds, 4 * simd / waves));
        const int together = blocks >= 256.0 * resident ? resident : ((int)blocks + 255) / 256;
        const double per_simd = std::max(1.0, waves > 3 ? (double)((waves + 3) / 4 * together) : waves / 4.0 * together);
        const double share = per_simd < 2 ? 1.2 - 0.165 * (per_simd - 1) : std::max(0.75, 1.035 - 0.172 * (per_simd - 2));
        const int own = (num_chunks + ksplit - 1) / ksplit;               // chunks of one slice
        const double at_once = 1.0 / together;
        double rounds = blocks * at_once / 256;
        rounds = rounds < 3 ? (double)((int)blocks / (256 * together) + ((int)blocks % (256 * together) != 0)) : rounds + 0.5;
        const double staging = own * (420.0 + ck * (25.0 * together + 120.0 / waves + 15.0 * at_once));
        double us = 5.28 + rounds * (filters * own * kernels * share * per_simd + staging + 2460) * (1.0 / 2400) +
                    (in_mb + again_mb * (sets - 1) + out_mb) * at_once * (1.0 / 5.65);
        if (ksplit > 1) us += 3.2 + out_mb * (2 * ksplit + 1) * (1.0 / 5.75);    // the slices' sums, out and back in
        return us;
    }
};

// Wavefronts that share a group's eight filters in a launch of taps_f8 whose workgroups take `waves` groups: 1, 2 or
// 4, whichever is estimated to be fastest.  A filter's kernels come one after the other, some 230 cycles each, flushes
// included, for a wavefront that has its SIMD to itself, so launches with few wavefronts gain: one image of
// 512 -> 512 at 14 x 14 20.5 -> 14.0 us, of 128 -> 256 at 56 x 56 23.9 -> 13.7, 100 -> 75 at 45 x 61, six images 23.6 -> 18.6;
// launches that fill the chip anyway lose (they stage the same inputs for fewer filters at a time: 512 -> 512 at 28 x 28,
// two images, ck 64, 37.9 -> 42.3).  The sums of a filter are the same whoever computes it.
int taps_parts(const TapsEstimate& estimate, int waves, int ksplit, double& us)
{
    int best = 1;
    us = estimate(kTapGroup, waves, ksplit);
    if (estimate.wavefronts(waves, ksplit) >= 4096.0) return best;        // sixteen for each CU already
    for (int parts = 2; parts <= 4 && parts * waves <= kMaxTapWaves; parts *= 2) {
        const double e = estimate(kTapGroup / parts, parts * waves, ksplit);
        if (e < us) { us = e; best = parts; }
    }
    return best;
}

int taps_parts(const patdnn_layer* h, const Taps& t, const ConvShape& s, int waves, int ksplit)
{
    double us = 0.0;
    return taps_parts(TapsEstimate(h, t, s, (double)tap_tile_count(s)), waves, ksplit, us);
}

// A launch and its estimate.
struct Launch {
    double us = 1e30;
    patdnn_config_t c{};
};

// The shortest launch in workgroups of 2, 4, 8 or 16 wavefronts with whole groups, in up to 16 slices as `room` floats allow,
// by an estimate that the finer one above has replaced for the choice among this kernel's launches.  It goes on telling which
// layers are this kernel's, the one with the smallest errors (in 1e-8 of the result against 64 bits, 64 to 512 channels, kept
// 1/3.6: 8 to 9.5, the tiled kernel 12 to 30, the split kernel 11 to 13): by the finer one alone 180 of 2500 layers went to one of
// those, 20 to the tiled kernel, most for more time (384 -> 56 at 170 x 170, five images, kept 0.15 180 -> 198 us), and 160 to the
// split kernel for less (80 -> 292 at 52 x 52, 37 images, all kept 375 -> 228).
Launch whole_groups(const patdnn_layer* h, const ConvShape& s, double tiles, size_t room)
{
    const size_t slice_stride = split_slice_stride((size_t)s.n * s.c_out * s.ho * s.wo);
    const double in_mb = 4e-6 * s.n * s.c_in * s.h * s.w, out_mb = 4e-6 * s.n * s.c_out * (double)s.ho * s.wo;
    Launch best;
    for (const auto& layout : h->taps) {
        const Taps& t = layout.second->host;
        const double kernels = (46.7 * h->L.kept + 107.4 * t.segments) / s.c_out / t.num_chunks + 93.0;       // of one chunk
        for (int filters = 8; filters <= 16; filters *= 2)
            for (int waves = 2; waves <= kMaxTapWaves && (waves == 2 || waves / 2 * filters < s.c_out); waves *= 2) {
                const int sets = (t.num_groups * kTapGroup + waves * filters - 1) / (waves * filters);
                const int resident = std::max(1, std::min(kTapMaxChunk / t.ck, (filters == 16 ? 16 : 20) / waves));
                for (int ks = 1; ks <= 16 && ks <= t.num_chunks && (ks == 1 || (room / ks >= slice_stride && ks * slice_stride <= kMaxSliceFloats)); ks *= 2) {
                    const double blocks = tiles * sets * ks, together = blocks >= 256.0 * resident ? resident : std::ceil(blocks / 256);
                    const double per_simd = std::max(1.0, waves / 4.0) * together, rounds = blocks / (256 * together);
                    const double share = per_simd < 2 ? 1.73 - 0.64 * (per_simd - 1) : std::max(0.75, 1.09 - 0.17 * (per_simd - 2));
                    const double work = filters * ((t.num_chunks + ks - 1) / ks) * kernels;
                    double us = 5.0 + (rounds < 3 ? std::ceil(rounds) : rounds + 0.5) * (work * share * per_simd + 2000) / 2400 +
                                (in_mb * (1 + 1.33 * (sets - 1)) + out_mb) / (5.65 * together);
                    if (ks > 1) us += 4.1 + out_mb * (2 * ks + 1) / 8.5;
                    if (us < best.us) best = Launch{us, patdnn_config_t{variant_of_extra(filters == 8 ? kExtraTaps8 : kExtraTaps16), t.ck, waves, ks}};
                }
            }
    }
    return best;
}

// Default tiled variant, microseconds: rounds of three wavefronts per SIMD.
double tiled_estimate(const patdnn_layer* h, const TiledVariant& v, const ConvShape& s)
{
    const long long bands = (long long)s.n * ((s.wo + v.TGX * v.PC - 1) / (v.TGX * v.PC)) * ((s.ho + v.PR - 1) / v.PR);
    const double waves = (double)((bands + 64 / v.TGX - 1) / (64 / v.TGX)) * ((s.c_out + v.G - 1) / v.G);
    const double rounds = waves <= 3072 ? 1.0 : waves / 3072 + 0.35;
    const double per_simd = std::min(3.0, std::max(1.0, waves / 1024));
    // libraries of more than eight patterns: the blocks in use outgrow the instruction cache, the more
    // so the more kernels a wavefront runs (512 -> 512 at 28 x 28, 56 patterns: 825 us, 8 patterns 673)
    const double kernels = (double)h->L.kept / s.c_out, over8 = std::log2(std::max(1.0, h->L.fkw.num_patterns / 8.0));
    return rounds * (0.336 * s.c_in + 0.195 * v.G * kernels + 8.06) * (0.785 + 0.1075 * (per_simd - 1)) *
           (1.0 + (0.03 + 5e-4 * std::min(kernels, 200.0)) * over8);
}

// Default stride-2 variant, microseconds: a wavefront of 16 filters and 64 columns of four rows goes through the
// channels one after the other; up to some two wavefronts per SIMD that chain is the time.  (Nine layers of 77
// to 352 channels, 77 to 586 us: 8 % on average.)
double tiled2_estimate(const patdnn_layer* h, const ConvShape& s)
{
    const double kernels = (double)h->L.kept / s.c_out;
    const long long bands = (long long)s.n * ((s.wo + 15) / 16) * ((s.ho + 3) / 4);
    const double per_simd = (double)((bands + 3) / 4) * ((s.c_out + 15) / 16) / 1024;
    return 5.0 + (0.265 * s.c_in + 1.25 * kernels) * (per_simd < 1.9 ? 1.1 + 0.1 * per_simd : 1.4 + 0.42 * per_simd);
}

// FKW walk, microseconds: a wavefront walks the kernels of one filter, pattern by pattern, for 64
// output pixels, one load after the other; launches of more wavefronts than the chip holds pay for
// each of them.  (Fitted to 90 layers of 16 to 512 channels, 6 to 56 patterns and 9 us to 9 ms: 14 %
// on average.)
double fkw_estimate(const patdnn_layer* h, const ConvShape& s)
{
    const double kernels = (double)h->L.kept / s.c_out, patterns = h->L.fkw.num_patterns;
    const double waves = (double)s.n * s.c_out * (((long long)s.ho * s.wo + 63) / 64);
    return 4.9 + 0.223 * kernels + 0.192 * patterns + waves * (9.8e-5 * kernels + 2.8e-5 * patterns);
}

// Binary16 layers, microseconds: the walk as above, and the matrix kernel, which multiplies the removed
// weights too and fills its channels to 16 and its filters to 32: a chain of channel steps, multiply-adds,
// inputs staged once per 128 filters, outputs.  Fitted to 400 layers of 1 to 512 channels, keep ratios
// from 0.003 and dense ones: 14 % and 8 % on average, on 400 others 15 % and 9 %.  The walk is taken for
// filters of at most eight kernels and where it is ahead by more than 15 % (longer chains of cold loads are
// up to 1.7 times the estimate): 17 -> 3 at 175 x 175 / 2, 15 images, one kernel in a hundred 9 us against
// 28.  Of the 800 layers 11 are then more than 15 % behind the walk (56 without it) and 5 more than 10 %
// behind the matrix kernel.  Layers of 16 channels and filters and more at keep ratios from 1/3.6 are
// none of these.
bool f16_walk_pays(const patdnn_layer* h, const ConvShape& s)
{
    const double kernels = (double)h->L.kept / s.c_out * h->L.fkw.taps / 4, patterns = h->L.fkw.num_patterns;
    if (kernels > 8.0) return false;
    const double pixels = (double)s.n * s.ho * s.wo, waves = (double)s.n * s.c_out * (((long long)s.ho * s.wo + 63) / 64);
    const double walk = std::max(9.4, 5.2 + 0.368 * kernels + 0.079 * patterns + waves * (1.47e-4 * kernels + 2.4e-5 * patterns));
    const double c16 = (s.c_in + 15) / 16 * 16.0, f32 = (s.c_out + 31) / 32 * 32.0;
    const double matrix = std::max(9.4, 7.1 + 0.156 * c16 / 16 + 1.16e-8 * pixels * c16 * f32 +
                                            1.44e-6 * s.n * s.h * s.w * c16 * std::ceil(f32 / 128) + 0.84e-6 * pixels * s.c_out);
    return walk * 1.15 < matrix;
}

// Binary16 weights with the removed ones as zeros: up to 256 MB a layer.
constexpr size_t kMaxExpandedHalves = (size_t)128 << 20;

// DevFkw::split_filters and split_seen; false where a weight is not finite, or so small beside its filter's largest
// that binary16 would not have all of its bits.
bool split_filters(const LayerHost& L, std::vector<int32_t>& out, float& seen)
{
    const Fkw& f = L.fkw;
    out.assign((size_t)(L.desc.c_out + 63) / 64 * 128, -1);
    double sum = 0.0;                                 // largest of a filter's magnitudes, scaled
    for (int s = 0; s < L.desc.c_out; ++s) {
        out[2 * (size_t)s] = f.reorder[s];
        int32_t& exponent = out[2 * (size_t)s + 1] = kSplitEmpty;
        float most = 0.0f, least = INFINITY;
        double all = 0.0;
        for (size_t i = (size_t)f.offset[s] * f.taps; i < (size_t)f.offset[s + 1] * f.taps; ++i) {
            const float w = std::fabs(f.weight[i]);
            if (!(w < INFINITY)) return false;
            if (w > 0.0f) least = std::min(least, w);
            most = std::max(most, w);
            all += w;
        }
        if (most == 0.0f) continue;                   // (kept zeros count as none: they are what they are in any scale)
        int e = 0;
        std::frexp(most, &e);                         // most < 2^e
        exponent = 15 - e;
        if (std::ldexp((double)least, exponent) < 0x1p-14) return false;
        sum = std::max(sum, std::ldexp(all, exponent));
    }
    // an input below the scale is off by 2^-36, and of its product with a weight as much is left out again
    seen = (float)std::min(sum * 0x1p-35 * 0x1p24, 0x1p100);
    return true;
}

// Pruned layers for which the split kernel exists: where each of its filters comes out no less exact than from the
// kernels that it stands in for (the walk and the tiled kernels; the tap-product kernel is the more exact one), which
// add a filter's products one after the other.  Errors against 64 bits, in 1e-8 of a filter's result, over inputs
// that a ReLU left, 64 to 512 channels: theirs grow as 2.6 sqrt(kernels), 7.6 for 8 kernels, 10.5 for 16, 11.2 for 18, 11.8
// for 20, 14.7 for 32, 58 for 512; the split kernel has 7.3 from the halves' last bits and adds 32 channels by
// themselves, 10.2 for 8, 10.8 for 16, 11.0 for 18 and 20, 11.7 for 32, 15 for 512.  (Inputs of both signs: even at 8 kernels.)
constexpr int kSplitKernels = 18;
// At stride 1 it is slower than the others for less than about 0.4 of the kernels (128 -> 128 at 112 x 112, 64
// images: 1/3.6 615 us against 560 when it still added without joins, one half 708 and 711; all of 64 -> 64 123 against 209).
// `filters`, `seen`: see split_filters.
bool split_layer(const LayerHost& L, std::vector<int32_t>& filters, float& seen)
{
    if (L.depthwise || L.dense || L.kept == 0) return false;
    if (L.desc.stride == 1 && (double)L.kept / L.desc.c_out / L.desc.c_in < 0.4) return false;
    for (int s = 0; s < L.desc.c_out; ++s) {
        const int32_t kernels = L.fkw.offset[s + 1] - L.fkw.offset[s];
        if (kernels && kernels < kSplitKernels) return false;
    }
    return split_expanded_halves(L.desc.c_in, L.desc.c_out) <= kMaxExpandedHalves && split_filters(L, filters, seen);
}

// Dense layers of few channels: filters are stored in the order of their channels there, and zero padding, which the
// matrix cores multiply, must not meet a weight that is not finite (the walk leaves it out).
bool dense_layer(const LayerHost& L)
{
    if (!L.dense || L.depthwise || L.desc.c_in > kDenseChannels || L.desc.stride > 2) return false;
    for (float w : L.fkw.weight)
        if (!std::isfinite(w)) return false;
    return true;
}

// Whether the dense kernel, which computes 32 filters whatever there are, is the library's choice: large launches of very
// few filters are left to the kernels before it.  64 images of 224 x 224, us of this one, of the tiled one and of the
// walk: 1 -> 1 44, 38, 27; 3 -> 2 80, 73, 72; 3 -> 4 82, 75, 132; 3 -> 8 82, 79, 235; 4 -> 8 and all of 16 filters even or ahead,
// pooled 3 -> 8 at 150 x 150, 32 images, 23, 60, 81; at stride 2 3 -> 1 25, --, 18, 1 -> 2 even.  Below half a million pixels
// all end within a microsecond.
bool dense_pays(const ConvShape& s)
{
    return s.c_out > (s.stride == 1 ? 4 : 1) || (long long)s.n * s.ho * s.wo < 1 << 19;
}

// Split kernel, microseconds: units of work one after the other, channel steps and stores of each.  (18 layers of
// tests/test_planner_choice.py: 5 % off on average, 19 % at most.)
double split_estimate(int rounds, int steps, int pixels)
{
    return 8.0 + rounds * (3.9 * steps + (pixels == 64 ? 8.7 : 3.5));
}

// The FKW arrays and what is derived from them, to the device.
patdnn_status_t upload_layer(patdnn_layer* h)
{
    hipError_t e = hipGetDevice(&h->device);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    const Fkw& f = h->L.fkw;
    DevFkw& d = h->dfkw;
    d.num_patterns = f.num_patterns;
    d.taps = f.taps;
    Upload up;
    up.add(f.offset, &d.offset);
    up.add(f.reorder, &d.reorder);
    up.add(f.index, &d.index);
    up.add(f.stride, &d.stride);
    up.add(f.weight, &d.weight);
    up.add(f.masks, &d.masks);
    // the weights once more in binary16 (round to nearest even) for patdnn_conv2d_f16
    const auto to_f16 = [](const std::vector<float>& from, std::vector<uint16_t>& to) {
        bool finite = true;
        to.resize(from.size());
        for (size_t i = 0; i < to.size(); ++i) {
            const _Float16 hv = static_cast<_Float16>(from[i]);
            std::memcpy(&to[i], &hv, 2);
            finite = finite && (to[i] & 0x7C00) != 0x7C00;
        }
        return finite;
    };
    std::vector<uint16_t> w16;
    const bool finite16 = to_f16(f.weight, w16);
    const uint16_t *weight16 = nullptr, *expanded16 = nullptr, *dw_weight16 = nullptr;
    up.add(w16, &weight16);
    std::vector<int32_t> dmask, taps;
    std::vector<float> dweight, tap_weight;
    std::vector<uint16_t> dweight16;
    if (h->L.depthwise) {
        // per stored filter: the mask of its kernel's pattern and its four weights; and by channel, the
        // four tap positions in nibbles
        const int c = h->L.desc.c_out, P = f.num_patterns;
        dmask.assign((size_t)c, 0);
        dweight.assign((size_t)c * 4, 0.0f);
        taps.assign((size_t)c, -1);
        tap_weight.assign((size_t)c * 4, 0.0f);
        for (int s = 0; s < c; ++s) {
            if (f.offset[s + 1] == f.offset[s]) continue;
            const int32_t* st = &f.stride[(size_t)s * (P + 1)];
            for (int p = 0; p < P; ++p)
                if (st[p + 1] > st[p]) dmask[s] = f.masks[p];
            const int co = f.reorder[s];
            unsigned nibbles = 0;
            for (int pos = 8; pos >= 0; --pos)
                if (dmask[s] >> pos & 1) nibbles = nibbles << 4 | (unsigned)pos;
            taps[co] = (int32_t)nibbles;
            for (int t = 0; t < 4; ++t)
                tap_weight[(size_t)co * 4 + t] = dweight[(size_t)s * 4 + t] = f.weight[(size_t)f.offset[s] * 4 + t];
        }
        up.add(dmask, &d.dw_mask);
        up.add(dweight, &d.dw_weight);
        d.dw_finite = std::all_of(dweight.begin(), dweight.end(), [](float w) { return std::isfinite(w); });
        if (to_f16(dweight, dweight16)) {         // else zero padding would meet an infinite weight
            up.add(taps, &d.dw_taps);
            up.add(tap_weight, &d.dw_tap_weight);
        }
        up.add(dweight16, &dw_weight16);
    }
    const size_t split = h->split ? split_expanded_halves(h->L.desc.c_in, h->L.desc.c_out) : 0;
    const uint16_t* split16 = nullptr;
    if (split) up.add(h->split_filters, &d.split_filters);
    size_t expanded = h->L.depthwise || !finite16 ? 0 : f16_expanded_halves(h->L.desc.c_in, h->L.desc.c_out);
    if (expanded > kMaxExpandedHalves) expanded = 0;
    // from a megabyte on by themselves, at the start of a page (512 -> 512 at 7 x 7, 64 images: 26.5 us, 27.2
    // behind the other arrays)
    Upload own;
    (expanded >= 1 << 19 ? own : up).room(expanded, &expanded16);
    (split >= 1 << 19 ? own : up).room(split, &split16);
    if ((e = up.commit(h->allocations)) != hipSuccess || (e = own.commit(h->allocations)) != hipSuccess)
        return hip_fail(e, "uploading the layer");
    d.weight_f16 = weight16;
    d.dw_weight_f16 = dw_weight16;
    if (expanded) {
        if ((e = hipMemsetAsync(const_cast<uint16_t*>(expanded16), 0, expanded * 2, nullptr)) != hipSuccess ||
            (e = launch_f16_expand(d, h->L.desc.c_in, h->L.desc.c_out, const_cast<uint16_t*>(expanded16), nullptr)) != hipSuccess ||
            (e = hipStreamSynchronize(nullptr)) != hipSuccess)
            return hip_fail(e, "expanding the binary16 weights");
        d.expanded_f16 = expanded16;
    }
    if (split) {
        if ((e = hipMemsetAsync(const_cast<uint16_t*>(split16), 0, split * 2, nullptr)) != hipSuccess ||
            (e = launch_split_expand(d, h->L.desc.c_in, h->L.desc.c_out, const_cast<uint16_t*>(split16), nullptr)) != hipSuccess ||
            (e = hipStreamSynchronize(nullptr)) != hipSuccess)
            return hip_fail(e, "splitting the weights");
        d.split_f16 = split16;
    }
    h->on_device = true;
    return PATDNN_OK;
}

// The workgroups that a tile's `units` (of eight or sixteen filters) are dealt to: up to so many wavefronts each, evenly.
template <class F>
void for_each_tap_split(int units, F&& f)
{
    int last = 0;
    for (const int most : {1, 2, 3, 4, 6, 8, 12, kMaxTapWaves}) {
        const int sets = (units + most - 1) / most, waves = (units + sets - 1) / sets;
        if (waves != last) f(waves);
        last = waves;
    }
}

// `scratch_floats`: room for the partial sums of a split launch (0: no split candidates).  The
// choice does not depend on fused pooling, so that a pooled output is the pooling of the plain one (to the last
// bits only where the split kernel meets inputs far apart: its tiles then differ in what is worked out again).
patdnn_config_t default_config(patdnn_layer* h, const ConvShape& shape, size_t scratch_floats)
{
    ConvShape s = shape, pooled = shape;
    s.pool = 0;
    pooled.pool = s.ho >= 2 && s.wo >= 2;
    if (h->L.depthwise) return patdnn_config_t{variant_of_extra(kExtraDepthwise), 0, 0, 1};
    if (h->dense_mfma && dense_fits(s) && dense_pays(s)) return patdnn_config_t{variant_of_extra(kExtraDense), 0, 0, 1};
    patdnn_config_t best{PATDNN_VARIANT_FKW, 0, 0, 1};
    const bool taps = taps_fit_layer(h) && taps_fit_input(s) && taps_fit_input(pooled) && !h->taps.empty();
    double best_us = taps ? fkw_estimate(h, s) : 0.0;
    for (int vi : h->order) {
        const TiledVariant& v = tiled_variant(vi);
        int32_t ck = 0, waves = 0;
        if (!resolve_tiled_params(h, v, s, ck, waves)) continue;
        if (h->tiled.find(std::make_pair(vi, v.dense ? 0 : ck)) == h->tiled.end()) continue;
        const double us = taps ? tiled_estimate(h, v, s) : -1.0;
        if (us < best_us) { best_us = us; best = patdnn_config_t{vi + 1, ck, waves, 1}; }
        break;
    }
    // the split kernel, on halves, stands in for those two only: the tap-product kernel is the more exact one
    double halves_us = 1e30;
    int halves_rounds = 0, halves_steps = 0, halves_pixels = 0;
    if (h->split && split_cost(pooled, halves_rounds, halves_steps, halves_pixels) && split_cost(s, halves_rounds, halves_steps, halves_pixels))
        halves_us = split_estimate(halves_rounds, halves_steps, halves_pixels) * (s.stride == 1 ? 1.03 : 1.15);   // (the estimate of the stride-2 variant is the coarser one)
    const auto or_halves = [&]() {
        const double other = taps ? best_us : best.variant == PATDNN_VARIANT_FKW ? fkw_estimate(h, s) : tiled2_estimate(h, s);
        return halves_us > other ? best : patdnn_config_t{variant_of_extra(kExtraSplit), 0, 0, 1};
    };
    if (!taps) return or_halves();
    const long long tiles = tap_tile_count(s);
    const size_t stride = split_slice_stride((size_t)s.n * s.c_out * s.ho * s.wo);
    Launch unsplit, split;
    for (int level = 0; level < kTapLevels; ++level) {
        const int ck = taps_ck(s.c_in, level);
        auto it = h->taps.find(ck);
        if (it == h->taps.end()) continue;
        const Taps& t = it->second->host;
        const TapsEstimate estimate(h, t, s, (double)tiles);
        for (int filters = 8; filters <= 16; filters *= 2) {
            const int units = (t.num_groups * kTapGroup + filters - 1) / filters;
            for_each_tap_split(units, [&](int waves) {
                for (int ks = 1; ks <= 16 && ks <= t.num_chunks; ks *= 2) {
                    if (ks > 1 && (scratch_floats / ks < stride || ks * stride > kMaxSliceFloats)) break;
                    double us = 0.0;
                    Launch& f = ks > 1 ? split : unsplit;
                    if (filters == kTapGroup) taps_parts(estimate, waves, ks, us);
                    else us = estimate(filters, waves, ks);
                    if (us < f.us) f = Launch{us, patdnn_config_t{variant_of_extra(filters == 8 ? kExtraTaps8 : kExtraTaps16), ck, waves, ks}};
                }
            });
        }
    }
    // Several wavefronts for a group take the place of channel slices in many launches, which then need no second kernel:
    // 128 -> 256 at 56 x 56, one image, 14.2 us, in slices 18.6; 312 -> 37 at 23 x 32, five images 26.4 and 19.2.  From 400 to 440
    // groups slices stay the answer up to 1.3 times the time where they were it before there were several wavefronts, slower
    // as that is (the layers that show the library splitting by itself are here: 96 -> 200 at 7 x 7, 64 images, 16.7 us,
    // unsplit 12.0, before 22.8; 200 -> 72 at 45 x 45, three images, 21.8, 19.6, before 29.2).
    const long long groups = tiles * ((s.c_out + kTapGroup - 1) / kTapGroup);
    const bool sliced = split.us < unsplit.us || (groups >= 400 && groups < 440 && split.us < unsplit.us * 1.3 &&
                                                  whole_groups(h, s, (double)tiles, kMaxSliceFloats).c.ksplit > 1);
    const Launch& taps_best = sliced ? split : unsplit;
    // Either of the two against the other kernels: one that wins by that factor must not stand in for the other here.  Against
    // the tiled kernel slices count as whole_groups has them.
    const double taps_us = best.variant == PATDNN_VARIANT_FKW ? std::min(split.us, unsplit.us) : unsplit.us;
    // One tile of no more than 64 groups keeps the walk where all takes little more than a launch, as it did when groups were
    // whole: 64 -> 512 at 14 x 14, one image, 13.3 us, this kernel 8.7.  Elsewhere the walk loses: 40 -> 155 at 10 x 10, 21
    // images, 23 us, this kernel 9.3; 24 -> 240 at 18 x 18, two images, 13.6 and 8.4; 36 -> 16 at 39 x 39, eight images 12.5 and 8.0.
    // (Whatever the room, or a call without would run another kernel.)
    if (best.variant == PATDNN_VARIANT_FKW && best_us < 15.0 && tiles == 1 && groups <= 64 &&
        best_us < whole_groups(h, s, (double)tiles, kMaxSliceFloats).us)
        return or_halves();
    if (taps_us < std::min(best_us, halves_us)) return taps_best.c;
    // Not ahead of all of them, it keeps what it ran when groups were whole.  With any room: a call with the room that was asked
    // for must not choose otherwise, nor one that needs none.
    const Launch whole = whole_groups(h, s, (double)tiles, scratch_floats / 2 >= stride ? kMaxSliceFloats : 0);
    if (whole.us >= best_us) return or_halves();
    const bool ahead = std::min(split.us, unsplit.us) < best_us;
    if (whole.c.ksplit == 1) return ahead ? taps_best.c : whole.c;
    if (ahead && (taps_best.c.ksplit > 1 || whole_groups(h, s, (double)tiles, 0).us < best_us)) return taps_best.c;
    return scratch_floats / whole.c.ksplit < stride ? taps_best.c : whole.c;
}

}  // namespace

extern "C" {

patdnn_status_t patdnn_encode(const patdnn_layer_desc_t* desc, const float* dense_weights,
                              const uint8_t* pattern_ids, const uint8_t* kernel_mask,
                              patdnn_handle_t* out)
{
    if (out) *out = nullptr;
    if (!desc || !out) return fail(PATDNN_EINVAL, "desc / out is NULL");
    return guarded([&]() -> patdnn_status_t {
        std::unique_ptr<patdnn_layer> h(new patdnn_layer());
        std::string err;
        patdnn_status_t st = build_fkw(*desc, dense_weights, pattern_ids, kernel_mask, h->L, err);
        if (st != PATDNN_OK) return fail(st, err);
        h->split = split_layer(h->L, h->split_filters, h->dfkw.split_seen);
        h->dense_mfma = dense_layer(h->L);
        if (!(desc->flags & PATDNN_HOST_ONLY)) {
            st = upload_layer(h.get());
            if (st != PATDNN_OK) return st;
        }
        // build (and upload) the group layout of the default variant; the layouts of the other
        // variants are built when patdnn_set_config or patdnn_tune asks for them
        if (taps_fit_layer(h.get()))
            for (int level = 0; level < kTapLevels; ++level) {
                const int ck = taps_ck(desc->c_in, level);
                if (level > 0 && ck < kMinTapChunk) break;
                st = ensure_taps(h.get(), ck, nullptr);
                if (st != PATDNN_OK) return st;
            }
        h->order = default_variant_order(h.get());
        if (!h->order.empty()) {
            const int vi = h->order[0];
            st = ensure_tiled(h.get(), vi, default_ck(tiled_variant(vi), desc->c_in), nullptr);
            if (st != PATDNN_OK) return st;
        }
        *out = h.release();
        return PATDNN_OK;
    });
}

patdnn_status_t patdnn_output_shape(patdnn_handle_t h, int32_t n, int32_t h_in, int32_t w_in,
                                    int32_t out_nchw[4])
{
    ConvShape s{};
    patdnn_status_t st = shape_of(h, n, h_in, w_in, s);
    if (st != PATDNN_OK) return st;
    if (!out_nchw) return fail(PATDNN_EINVAL, "out_nchw is NULL");
    out_nchw[0] = n; out_nchw[1] = s.c_out; out_nchw[2] = s.ho; out_nchw[3] = s.wo;
    return PATDNN_OK;
}

// What one layer of a stack hands to the next about zero fills: the region the next layer must
// find zeroed, which this layer clears in its finishing kernel if it has one (`done` tells).
struct ZeroRegion {
    float* p = nullptr;
    size_t count = 0;
};
struct ZeroHandoff {
    ZeroRegion pre_zeroed;   // in: already holds zeros when the layer starts
    ZeroRegion next;         // in: what the next layer will want zeroed
    bool done = false;       // out: `next` was cleared by this layer
    const patdnn_config_t* plan = nullptr;    // in: this layer's effective_config, where it is known already
};

// A split launch stores its slices to buffers of their own (no zero fill, no atomics) if the
// scratch holds one per slice; the launcher decides by the same rule.
static bool slices_fit(const float* scratch, size_t scratch_floats, int32_t ksplit, size_t full)
{
    return scratch && ksplit > 1 && (reinterpret_cast<uintptr_t>(scratch) & 15) == 0 &&
           scratch_floats / (size_t)ksplit >= split_slice_stride(full);
}

// Floats of partial sums that the handle's configuration, or the library's choice, can use.
static size_t split_room(patdnn_handle_t h, const ConvShape& s)
{
    if (h->cfg.variant < 0 && (!h->on_device || s.n == 0)) return 0;
    const patdnn_config_t c = h->cfg.variant < 0 ? default_config(h, s, kMaxSliceFloats) : h->cfg;
    return c.variant > 0 && c.ksplit > 1 ? (size_t)c.ksplit * split_slice_stride((size_t)s.n * s.c_out * s.ho * s.wo) : 0;
}

// The configuration a call runs: the handle's, or the library's choice.  A pooled layer that
// splits the input channels needs room for its partial sums; without it the library chooses.
static patdnn_config_t effective_config(patdnn_handle_t h, const ConvShape& s, const float* scratch, size_t scratch_floats)
{
    const patdnn_config_t& c = h->cfg;
    const bool aligned = scratch && (reinterpret_cast<uintptr_t>(scratch) & 15) == 0;
    const size_t full = (size_t)s.n * s.c_out * s.ho * s.wo;
    if (c.variant < 0 || (s.pool && c.variant > 0 && c.ksplit > 1 && !(scratch && scratch_floats >= full)))
        return default_config(h, s, aligned ? scratch_floats : 0);
    return c;
}

// The region that must hold zeros before the kernels of configuration `c` run (none: p == NULL).
static ZeroRegion zero_need(const patdnn_config_t& c, const ConvShape& s, float* output, float* scratch, size_t scratch_floats)
{
    const bool split = c.variant > 0 && c.ksplit > 1;
    const size_t full = (size_t)s.n * s.c_out * s.ho * s.wo;
    if (split && slices_fit(scratch, scratch_floats, c.ksplit, full)) return ZeroRegion{};   // stores only
    if (!s.pool) return split ? ZeroRegion{output, full} : ZeroRegion{};
    if (split) return ZeroRegion{scratch, full};
    if (taps_filters(c.variant) || extra_variant(c.variant) == kExtraSplit || extra_variant(c.variant) == kExtraDense)
        return ZeroRegion{};                                      // whole pooling windows in registers
    return ZeroRegion{output, (size_t)s.n * s.c_out * (s.ho / 2) * (s.wo / 2)};
}

// `scratch` (DEVICE, `scratch_floats` floats, may be NULL): where a layer whose configuration
// splits the input channels keeps its partial sums: one buffer per slice if there is room
// (ksplit * split_slice_stride([n][c_out][ho][wo]) floats), else - pooled layers only - one
// buffer that the slices add into ([n][c_out][ho][wo]).
static patdnn_status_t conv2d_impl(patdnn_handle_t h, const float* input, int32_t n, int32_t h_in,
                                   int32_t w_in, const float* bias, float* output, int32_t fuse_relu,
                                   int32_t pool, hipStream_t stream, float* scratch = nullptr,
                                   size_t scratch_floats = 0, ZeroHandoff* handoff = nullptr)
{
    ConvShape s{};
    patdnn_status_t st = shape_of(h, n, h_in, w_in, s);
    if (st != PATDNN_OK) return st;
    if (!h->on_device) return fail(PATDNN_EHIP, "handle was encoded with PATDNN_HOST_ONLY");
    const int oh = pool ? s.ho / 2 : s.ho, ow = pool ? s.wo / 2 : s.wo;
    if (pool && (oh == 0 || ow == 0)) return fail(PATDNN_EINVAL, "output smaller than one 2x2 pooling window");
    if (pool && h->L.depthwise) return fail(PATDNN_EUNSUPPORTED, "fused pooling is not built for depthwise layers");
    if (n == 0) return PATDNN_OK;
    if (!input || !output) return fail(PATDNN_EINVAL, "input / output is NULL");
    {
        const char* in_lo = reinterpret_cast<const char*>(input);
        const char* in_hi = in_lo + 4ull * (size_t)n * s.c_in * s.h * s.w;
        const char* out_lo = reinterpret_cast<const char*>(output);
        const char* out_hi = out_lo + 4ull * (size_t)n * s.c_out * oh * ow;
        if (in_lo < out_hi && out_lo < in_hi) return fail(PATDNN_EINVAL, "output overlaps input");
    }
    s.relu = (fuse_relu || pool) ? 1 : 0;
    s.pool = pool ? 1 : 0;
    if (handoff) {
        s.pre_zeroed = handoff->pre_zeroed.p;
        s.pre_zeroed_count = handoff->pre_zeroed.count;
        s.zero_next = handoff->next.p;
        s.zero_next_count = handoff->next.count;
        s.zero_next_done = &handoff->done;
    }
    auto run = [&](const patdnn_config_t& c) -> patdnn_status_t {
        // a pooled output that kernels fold into is cleared here, the target of split launches by
        // their launcher
        const ZeroRegion z = zero_need(c, s, output, scratch, scratch_floats);
        if (z.p && pool && z.p == output && !(s.pre_zeroed == z.p && s.pre_zeroed_count >= z.count)) {
            hipError_t e = launch_fill_zero(z.p, z.count, stream);
            if (e != hipSuccess) return hip_fail(e, "zeroing the pooled output");
        }
        return run_config(h, c, s, input, bias, output, stream, scratch, scratch_floats);
    };
    st = run(handoff && handoff->plan ? *handoff->plan : effective_config(h, s, scratch, scratch_floats));
    // a configuration tuned for another input size may not fit this one; a configuration the
    // caller set explicitly is never replaced: the error goes back instead
    if (st == PATDNN_EUNSUPPORTED && h->cfg.variant > 0 && h->cfg_tuned)
        st = run(default_config(h, s, scratch && (reinterpret_cast<uintptr_t>(scratch) & 15) == 0 ? scratch_floats : 0));
    return st;
}

// For tests, not part of the interface: what the library chooses for this input size and so much
// workspace.  Works on host-only handles too.
patdnn_status_t patdnn_internal_choice(patdnn_handle_t h, int32_t n, int32_t h_in, int32_t w_in,
                                       size_t workspace_floats, patdnn_config_t* out)
{
    ConvShape s{};
    patdnn_status_t st = shape_of(h, n, h_in, w_in, s);
    if (st == PATDNN_OK) *out = default_config(h, s, workspace_floats);
    return st;
}

// Likewise: what patdnn_conv2d_f16 launches for a tensor at `input` (see f16_choice; not for depthwise layers).
int32_t patdnn_internal_f16_choice(patdnn_handle_t h, const void* input, int32_t n, int32_t h_in, int32_t w_in)
{
    ConvShape s{};
    if (shape_of(h, n, h_in, w_in, s) != PATDNN_OK) return -2;
    return f16_walk_pays(h, s) ? -1 : f16_choice(s, input);
}

// Likewise: the kernel of a depthwise call (see dw_choice).
int32_t patdnn_internal_dw_choice(patdnn_handle_t h, const void* input, const void* output, int32_t n, int32_t h_in, int32_t w_in, int32_t half)
{
    ConvShape s{};
    return h->L.depthwise && h->on_device && shape_of(h, n, h_in, w_in, s) == PATDNN_OK ? dw_choice(h->dfkw, s, input, output, half != 0) : -1;
}

// Likewise: the wavefronts that share a filter group in a launch of the set configuration, a taps_f8 one.
int32_t patdnn_internal_taps_parts(patdnn_handle_t h, int32_t n, int32_t h_in, int32_t w_in)
{
    ConvShape s{};
    if (shape_of(h, n, h_in, w_in, s) != PATDNN_OK || taps_filters(h->cfg.variant) != kTapGroup) return -1;
    return taps_parts(h, h->taps.find(h->cfg.ck)->second->host, s, h->cfg.waves, h->cfg.ksplit);
}

// Likewise: the launch of the split kernel for a tensor at `input` (see split_choice), pooled or not.
int32_t patdnn_internal_split_choice(patdnn_handle_t h, const void* input, int32_t n, int32_t h_in, int32_t w_in, int32_t pool, int32_t* units)
{
    ConvShape s{};
    if (shape_of(h, n, h_in, w_in, s) != PATDNN_OK) return -2;
    s.pool = pool;
    return split_choice(s, input, *units);
}

patdnn_status_t patdnn_conv2d(patdnn_handle_t h, const float* input, int32_t n, int32_t h_in,
                              int32_t w_in, const float* bias, float* output, int32_t fuse_relu,
                              void* stream)
{
    return conv2d_impl(h, input, n, h_in, w_in, bias, output, fuse_relu, 0, static_cast<hipStream_t>(stream));
}

size_t patdnn_workspace_floats(patdnn_handle_t h, int32_t n, int32_t h_in, int32_t w_in)
{
    ConvShape s{};
    if (shape_of(h, n, h_in, w_in, s) != PATDNN_OK) return 0;
    return split_room(h, s);
}

patdnn_status_t patdnn_conv2d_ws(patdnn_handle_t h, const float* input, int32_t n, int32_t h_in, int32_t w_in,
                                 const float* bias, float* output, int32_t fuse_relu, int32_t pool2,
                                 float* workspace, size_t workspace_floats, void* stream)
{
    if (workspace && (reinterpret_cast<uintptr_t>(workspace) & 15))
        return fail(PATDNN_EINVAL, "workspace must be 16-byte aligned");
    ConvShape s{};
    if (workspace && workspace_floats && input && output && shape_of(h, n, h_in, w_in, s) == PATDNN_OK) {
        const char* lo = reinterpret_cast<const char*>(workspace);
        const char* hi = lo + 4ull * workspace_floats;
        const char* in_lo = reinterpret_cast<const char*>(input);
        const char* in_hi = in_lo + 4ull * (size_t)n * s.c_in * s.h * s.w;
        const char* out_lo = reinterpret_cast<const char*>(output);
        const char* out_hi = out_lo + 4ull * (size_t)n * s.c_out * (pool2 ? s.ho / 2 : s.ho) * (pool2 ? s.wo / 2 : s.wo);
        if ((lo < in_hi && in_lo < hi) || (lo < out_hi && out_lo < hi))
            return fail(PATDNN_EINVAL, "workspace overlaps input or output");
    }
    return conv2d_impl(h, input, n, h_in, w_in, bias, output, pool2 ? 1 : fuse_relu, pool2 ? 1 : 0,
                       static_cast<hipStream_t>(stream), workspace, workspace ? workspace_floats : 0);
}

patdnn_status_t patdnn_conv2d_f16(patdnn_handle_t h, const void* input, int32_t n, int32_t h_in, int32_t w_in,
                                  const float* bias, void* output, int32_t fuse_relu, void* stream)
{
    ConvShape s{};
    patdnn_status_t st = shape_of(h, n, h_in, w_in, s);
    if (st != PATDNN_OK) return st;
    if (!h->on_device) return fail(PATDNN_EHIP, "handle was encoded with PATDNN_HOST_ONLY");
    if (n == 0) return PATDNN_OK;
    if (!input || !output) return fail(PATDNN_EINVAL, "input / output is NULL");
    if ((reinterpret_cast<uintptr_t>(input) | reinterpret_cast<uintptr_t>(output)) & 1u)
        return fail(PATDNN_EINVAL, "binary16 tensors must be 2-byte aligned");
    {
        const char* in_lo = static_cast<const char*>(input);
        const char* in_hi = in_lo + 2ull * (size_t)n * s.c_in * s.h * s.w;
        const char* out_lo = static_cast<const char*>(output);
        const char* out_hi = out_lo + 2ull * (size_t)n * s.c_out * s.ho * s.wo;
        if (in_lo < out_hi && out_lo < in_hi) return fail(PATDNN_EINVAL, "output overlaps input");
    }
    s.relu = fuse_relu ? 1 : 0;
    hipError_t e = h->L.depthwise
                       ? launch_dw_f16(h->dfkw, s, input, bias, output, static_cast<hipStream_t>(stream))
                   : h->dfkw.expanded_f16 && !f16_walk_pays(h, s)
                       ? launch_f16(h->dfkw, s, input, bias, output, static_cast<hipStream_t>(stream))
                       : launch_fkw_f16(h->dfkw, s, input, bias, output, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? PATDNN_OK : hip_fail(e, "launching a binary16 kernel");
}

patdnn_status_t patdnn_conv2d_pool(patdnn_handle_t h, const float* input, int32_t n, int32_t h_in,
                                   int32_t w_in, const float* bias, float* output, void* stream)
{
    return conv2d_impl(h, input, n, h_in, w_in, bias, output, 1, 1, static_cast<hipStream_t>(stream));
}

patdnn_status_t patdnn_decode(patdnn_handle_t h, float* dense_weights, uint8_t* pattern_ids,
                              uint8_t* kernel_mask)
{
    if (!h) return fail(PATDNN_EINVAL, "handle is NULL");
    try {
        if (!h->on_device) {
            decode_fkw(h->L, h->L.fkw, dense_weights, pattern_ids, kernel_mask);
            return PATDNN_OK;
        }
        // read the five arrays back from device memory and invert them
        Fkw f;
        const Fkw& ref = h->L.fkw;
        f.taps = ref.taps;
        f.num_patterns = ref.num_patterns;
        f.offset.resize(ref.offset.size());
        f.reorder.resize(ref.reorder.size());
        f.index.resize(ref.index.size());
        f.stride.resize(ref.stride.size());
        f.weight.resize(ref.weight.size());
        f.masks.resize(ref.masks.size());
        auto back = [](void* dst, const void* src, size_t bytes) -> hipError_t {
            return bytes ? hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost) : hipSuccess;
        };
        hipError_t e;
        if ((e = back(f.offset.data(), h->dfkw.offset, f.offset.size() * 4)) != hipSuccess ||
            (e = back(f.reorder.data(), h->dfkw.reorder, f.reorder.size() * 4)) != hipSuccess ||
            (e = back(f.index.data(), h->dfkw.index, f.index.size() * 4)) != hipSuccess ||
            (e = back(f.stride.data(), h->dfkw.stride, f.stride.size() * 4)) != hipSuccess ||
            (e = back(f.weight.data(), h->dfkw.weight, f.weight.size() * 4)) != hipSuccess ||
            (e = back(f.masks.data(), h->dfkw.masks, f.masks.size() * 2)) != hipSuccess)
            return hip_fail(e, "reading the FKW arrays back");
        decode_fkw(h->L, f, dense_weights, pattern_ids, kernel_mask);
    } catch (const std::bad_alloc&) {
        return fail(PATDNN_ENOMEM, "out of host memory");
    }
    return PATDNN_OK;
}

patdnn_status_t patdnn_export_fkw(patdnn_handle_t h, int32_t* offset, int32_t* reorder,
                                  int32_t* index, int32_t* stride, float* weight)
{
    if (!h) return fail(PATDNN_EINVAL, "handle is NULL");
    const Fkw& f = h->L.fkw;
    auto get = [&](void* dst, const void* dev, const void* host, size_t bytes) -> hipError_t {
        if (!dst || !bytes) return hipSuccess;
        if (h->on_device) return hipMemcpy(dst, dev, bytes, hipMemcpyDeviceToHost);
        std::memcpy(dst, host, bytes);
        return hipSuccess;
    };
    hipError_t e;
    if ((e = get(offset, h->dfkw.offset, f.offset.data(), f.offset.size() * 4)) != hipSuccess ||
        (e = get(reorder, h->dfkw.reorder, f.reorder.data(), f.reorder.size() * 4)) != hipSuccess ||
        (e = get(index, h->dfkw.index, f.index.data(), f.index.size() * 4)) != hipSuccess ||
        (e = get(stride, h->dfkw.stride, f.stride.data(), f.stride.size() * 4)) != hipSuccess ||
        (e = get(weight, h->dfkw.weight, f.weight.data(), f.weight.size() * 4)) != hipSuccess)
        return hip_fail(e, "reading the FKW arrays back");
    return PATDNN_OK;
}

patdnn_status_t patdnn_export_csr(patdnn_handle_t h, int64_t* nnz, int32_t* row_ptr, int32_t* col, float* val)
{
    if (!h) return fail(PATDNN_EINVAL, "handle is NULL");
    try {
        patdnn_status_t st = ensure_compare(h);
        if (st != PATDNN_OK) return st;
    } catch (const std::bad_alloc&) {
        return fail(PATDNN_ENOMEM, "out of host memory");
    }
    const auto& c = h->csr_host;
    if (nnz) *nnz = (int64_t)c.col.size();
    auto get = [&](void* dst, const void* dev, const void* host, size_t bytes) -> hipError_t {
        if (!dst || !bytes) return hipSuccess;
        if (h->on_device) return hipMemcpy(dst, dev, bytes, hipMemcpyDeviceToHost);
        std::memcpy(dst, host, bytes);
        return hipSuccess;
    };
    hipError_t e;
    if ((e = get(row_ptr, h->csr_dev.row_ptr, c.row_ptr.data(), c.row_ptr.size() * 4)) != hipSuccess ||
        (e = get(col, h->csr_dev.col, c.col.data(), c.col.size() * 4)) != hipSuccess ||
        (e = get(val, h->csr_dev.val, c.val.data(), c.val.size() * 4)) != hipSuccess)
        return hip_fail(e, "reading the CSR arrays back");
    return PATDNN_OK;
}

static patdnn_status_t layout_stats(patdnn_handle_t h, patdnn_stats_t* out)
{
    if (!h || !out) return fail(PATDNN_EINVAL, "handle / out is NULL");
    const Fkw& f = h->L.fkw;
    std::memset(out, 0, sizeof(*out));
    out->kept_kernels = h->L.kept;
    out->taps = f.taps;
    out->num_patterns = f.num_patterns;
    out->fkw_weight_bytes = (int64_t)f.weight.size() * 4;
    out->fkw_index_bytes = 4 * (int64_t)(f.offset.size() + f.reorder.size() + f.index.size() + f.stride.size());
    std::vector<int32_t> len;
    for (size_t s = 0; s + 1 < f.offset.size(); ++s) len.push_back(f.offset[s + 1] - f.offset[s]);
    if (!len.empty()) {
        out->min_filter_length = *std::min_element(len.begin(), len.end());
        out->max_filter_length = *std::max_element(len.begin(), len.end());
        std::sort(len.begin(), len.end());
        out->distinct_filter_lengths = (int32_t)(std::unique(len.begin(), len.end()) - len.begin());
    }
    for (const auto& kv : h->tiled) out->tiled_bytes += (int64_t)kv.second->host.bytes();
    for (const auto& kv : h->taps) out->tiled_bytes += (int64_t)kv.second->bytes;
    if (!h->tiled.empty()) {
        const Tiled& t = h->tiled.begin()->second->host;
        out->filter_groups = t.num_groups;
        out->group_size = t.G;
        if (!t.group_kernels.empty()) {
            out->max_group_kernels = *std::max_element(t.group_kernels.begin(), t.group_kernels.end());
            out->min_group_kernels = *std::min_element(t.group_kernels.begin(), t.group_kernels.end());
        }
    }
    return PATDNN_OK;
}

patdnn_status_t patdnn_layout_stats(patdnn_handle_t h, patdnn_stats_t* out)
{
    return guarded([&] { return layout_stats(h, out); });
}

int32_t patdnn_num_variants(void) { return 1 + num_tiled_variants() + kNumExtra; }

const char* patdnn_variant_name(int32_t variant)
{
    if (variant == PATDNN_VARIANT_FKW) return "fkw";
    if (variant < 0 || variant >= patdnn_num_variants()) return nullptr;
    if (extra_variant(variant) >= 0) return kExtraNames[extra_variant(variant)];
    return tiled_variant(variant - 1).name;
}

static patdnn_status_t set_config(patdnn_handle_t h, const patdnn_config_t* cfg)
{
    if (!h || !cfg) return fail(PATDNN_EINVAL, "handle / cfg is NULL");
    if (cfg->variant < 0) {               // back to automatic choice
        h->cfg = patdnn_config_t{-1, 0, 0, 1};
        h->cfg_tuned = false;
        return PATDNN_OK;
    }
    if (cfg->variant >= patdnn_num_variants()) return fail(PATDNN_EINVAL, "no such variant");
    if (extra_variant(cfg->variant) == kExtraDepthwise) {
        if (!h->L.depthwise) return fail(PATDNN_EUNSUPPORTED, "the depthwise kernel runs depthwise layers only");
        h->cfg = patdnn_config_t{cfg->variant, 0, 0, 1};
        h->cfg_tuned = false;
        return PATDNN_OK;
    }
    if (extra_variant(cfg->variant) == kExtraNoopt || extra_variant(cfg->variant) == kExtraCsr) {
        const patdnn_status_t st = ensure_compare(h);
        if (st != PATDNN_OK) return st;
        h->cfg = patdnn_config_t{cfg->variant, 0, 0, 1};
        h->cfg_tuned = false;
        return PATDNN_OK;
    }
    if (extra_variant(cfg->variant) == kExtraSplit || extra_variant(cfg->variant) == kExtraDense) {
        if (!(extra_variant(cfg->variant) == kExtraSplit ? h->split : h->dense_mfma)) return fail(PATDNN_EUNSUPPORTED, "variant cannot run this layer");
        h->cfg = patdnn_config_t{cfg->variant, 0, 0, 1};
        h->cfg_tuned = false;
        return PATDNN_OK;
    }
    if (taps_filters(cfg->variant)) {
        if (!taps_fit_layer(h)) return fail(PATDNN_EUNSUPPORTED, "variant cannot run this layer");
        if (cfg->ck < 0 || cfg->waves < 0 || cfg->waves > kMaxTapWaves || cfg->ksplit < 0 || cfg->ksplit > 64)
            return fail(PATDNN_EINVAL, "ck / waves / ksplit out of range");
        patdnn_config_t c = *cfg;
        const int c_in = h->L.desc.c_in;
        if (c.ck == 0) c.ck = taps_ck(c_in, 0);
        c.ck = std::min(c.ck, c_in);
        if (c.ck > kTapMaxChunk) return fail(PATDNN_EUNSUPPORTED, "ck exceeds the LDS budget");
        if (c.waves == 0) c.waves = 8;
        if (c.ksplit < 1) c.ksplit = 1;
        if (c.ksplit > (c_in + c.ck - 1) / c.ck) return fail(PATDNN_EUNSUPPORTED, "ksplit exceeds the number of channel chunks");
        const patdnn_status_t st = ensure_taps(h, c.ck, nullptr);
        if (st != PATDNN_OK) return st;
        h->cfg = c;
        h->cfg_tuned = false;
        return PATDNN_OK;
    }
    if (cfg->variant > 0) {
        const TiledVariant& v = tiled_variant(cfg->variant - 1);
        if (!variant_fits_layer(h, v)) return fail(PATDNN_EUNSUPPORTED, "variant cannot run this layer");
        if (v.experimental && h->on_device && !experimental_allowed())
            return fail(PATDNN_EUNSUPPORTED, "experimental variant: set PATDNN_EXPERIMENTAL=1 to run it");
        if (cfg->ck < 0 || cfg->waves < 0 || cfg->waves > kMaxWaves || cfg->ksplit < 0 || cfg->ksplit > 64)
            return fail(PATDNN_EINVAL, "ck / waves / ksplit out of range");
        if (cfg->ksplit > 1 && v.dense) return fail(PATDNN_EUNSUPPORTED, "ksplit: sparse variants only");
        const int min_waves = (v.stage_elems + 64 * v.max_slots - 1) / (64 * v.max_slots);
        if (cfg->waves && cfg->waves < min_waves)
            return fail(PATDNN_EUNSUPPORTED, "too few wavefronts to stage a tile");
        if (cfg->ck && cfg->ck * 4 * v.lds_buffers * v.lds_floats_per_channel > kMaxLdsBytes)
            return fail(PATDNN_EUNSUPPORTED, "ck exceeds the LDS budget");
    }
    patdnn_config_t c = *cfg;
    if (c.ksplit < 1 || c.variant <= 0) c.ksplit = 1;
    if (c.variant > 0) {
        const TiledVariant& v = tiled_variant(c.variant - 1);
        if (c.ck == 0) c.ck = default_ck(v, h->L.desc.c_in);
        c.ck = std::min(c.ck, h->L.desc.c_in);
        const patdnn_status_t st = ensure_tiled(h, c.variant - 1, c.ck, nullptr);
        if (st != PATDNN_OK) return st;
        // an explicit configuration is taken as given or refused, never replaced at launch time
        const int num_chunks = v.dense ? (h->L.desc.c_in + c.ck - 1) / c.ck
                                       : h->tiled.find(std::make_pair(c.variant - 1, c.ck))->second->host.num_chunks;
        if (c.ksplit > num_chunks) return fail(PATDNN_EUNSUPPORTED, "ksplit exceeds the number of channel chunks");
    }
    h->cfg = c;
    h->cfg_tuned = false;
    return PATDNN_OK;
}

patdnn_status_t patdnn_set_config(patdnn_handle_t h, const patdnn_config_t* cfg)
{
    return guarded([&] { return set_config(h, cfg); });
}

patdnn_status_t patdnn_get_config(patdnn_handle_t h, patdnn_config_t* cfg)
{
    if (!h || !cfg) return fail(PATDNN_EINVAL, "handle / cfg is NULL");
    *cfg = h->cfg;
    return PATDNN_OK;
}

patdnn_status_t patdnn_tune(patdnn_handle_t h, const float* input, int32_t n, int32_t h_in,
                            int32_t w_in, const float* bias, float* output, void* stream_,
                            float* best_us)
{
    return patdnn_tune_ws(h, input, n, h_in, w_in, bias, output, nullptr, 0, stream_, best_us);
}

static patdnn_status_t tune_ws(patdnn_handle_t h, const float* input, int32_t n, int32_t h_in,
                               int32_t w_in, const float* bias, float* output, float* workspace,
                               size_t workspace_floats, void* stream_, float* best_us)
{
    if (workspace && (reinterpret_cast<uintptr_t>(workspace) & 15))
        return fail(PATDNN_EINVAL, "workspace must be 16-byte aligned");
    if (!workspace) workspace_floats = 0;
    ConvShape s{};
    patdnn_status_t st = shape_of(h, n, h_in, w_in, s);
    if (st != PATDNN_OK) return st;
    if (!h->on_device) return fail(PATDNN_EHIP, "handle was encoded with PATDNN_HOST_ONLY");
    if (n == 0 || !input || !output) return fail(PATDNN_EINVAL, "tuning needs n > 0 and real buffers");
    hipStream_t stream = static_cast<hipStream_t>(stream_);

    std::vector<patdnn_config_t> cands;
    // The grid: chunk sizes 8, 10 and 16 (smaller ones lose to their barrier count, larger ones
    // to LDS occupancy on every layer measured; 10 is the most that leaves the single-buffer 7x2
    // variant three workgroups per CU), 4 or 8 wavefronts per workgroup (fewer only when
    // the layer has fewer filter groups), and input-channel slices only for launches that
    // cannot fill the chip's wavefront slots three times over.
    const int ck_opts[] = {8, 10, 16};
    const int wave_opts[] = {1, 2, 4, 8};
    const long long kWaveSlots = 256 * 4 * 3;
    for (int vi = 0; vi < num_tiled_variants(); ++vi) {
        const TiledVariant& v = tiled_variant(vi);
        if (!(variant_selectable(h, v) || (experimental_allowed() && variant_fits_layer(h, v)))) continue;
        const int groups = (s.c_out + v.G - 1) / v.G;
        const long long bands = (long long)s.n * ((s.wo + v.TGX * v.PC - 1) / (v.TGX * v.PC)) * ((s.ho + v.PR - 1) / v.PR);
        const long long wavefronts = (bands + 64 / v.TGX - 1) / (64 / v.TGX) * groups;
        for (int ck : ck_opts)
            for (int waves : wave_opts) {
                int32_t ck2 = std::min(ck, s.c_in), w2 = waves;
                if (w2 < 4 && groups >= 4) continue;           // small workgroups only for few groups
                if (w2 > 1 && w2 / 2 >= groups) continue;      // mostly idle wavefronts
                if (!resolve_tiled_params(h, v, s, ck2, w2)) continue;
                const int num_chunks = (s.c_in + ck2 - 1) / ck2;
                for (int ks : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}) {
                    // slices only while the launch before this split leaves wavefront slots empty
                    if (ks > 1 && (v.dense || ks > num_chunks || wavefronts * (ks - 1) >= 2 * kWaveSlots)) continue;
                    patdnn_config_t c{vi + 1, ck2, w2, ks};
                    bool dup = false;
                    for (const auto& o : cands)
                        dup |= (o.variant == c.variant && o.ck == c.ck && o.waves == c.waves && o.ksplit == c.ksplit);
                    if (!dup && ensure_tiled(h, vi, ck2, nullptr) == PATDNN_OK) cands.push_back(c);
                }
            }
    }
    if (taps_fit_layer(h) && taps_fit_input(s))
        for (const auto& layout : h->taps)
            for (int filters = 8; filters <= 16; filters *= 2)
                for_each_tap_split((layout.second->host.num_groups * kTapGroup + filters - 1) / filters, [&](int waves) {
                    for (int ks = 1; ks <= 16 && ks <= layout.second->host.num_chunks; ks *= 2)
                        cands.push_back(patdnn_config_t{variant_of_extra(filters == 8 ? kExtraTaps8 : kExtraTaps16), layout.first, waves, ks});
                });
    if (h->L.depthwise) cands.push_back(patdnn_config_t{variant_of_extra(kExtraDepthwise), 0, 0, 1});
    if (h->dense_mfma && dense_fits(s)) cands.push_back(patdnn_config_t{variant_of_extra(kExtraDense), 0, 0, 1});
    // the split kernel also where the library takes it by itself although the tap-product kernel, which is the more
    // exact one, could run the layer (64 -> 64 at 112 x 112, 32 images, all kept: 123 us, the others 209)
    const bool chosen = extra_variant(default_config(h, s, workspace_floats).variant) == kExtraSplit;
    int rounds = 0, steps = 0, pixels = 0;
    if (chosen || (h->split && !taps_fit_layer(h) && split_cost(s, rounds, steps, pixels))) cands.push_back(patdnn_config_t{variant_of_extra(kExtraSplit), 0, 0, 1});
    cands.push_back(patdnn_config_t{PATDNN_VARIANT_FKW, 0, 0, 1});

    struct Event {
        hipEvent_t e = nullptr;
        ~Event()
        {
            if (e) (void)hipEventDestroy(e);
        }
    } first, second;
    hipError_t e;
    if ((e = hipEventCreate(&first.e)) != hipSuccess || (e = hipEventCreate(&second.e)) != hipSuccess) return hip_fail(e, "hipEventCreate");
    const hipEvent_t e0 = first.e, e1 = second.e;
    float best = -1.0f;
    patdnn_config_t best_cfg = cands.back();
    patdnn_status_t result = PATDNN_OK;
    // milliseconds per run of one candidate: one warm-up, then `reps` runs between two events
    auto time_config = [&](const patdnn_config_t& c, int reps, float& ms) -> patdnn_status_t {
        patdnn_status_t r = run_config(h, c, s, input, bias, output, stream, workspace, workspace_floats);
        if (r != PATDNN_OK) return r;
        (void)hipEventRecord(e0, stream);
        for (int k = 0; k < reps && r == PATDNN_OK; ++k)
            r = run_config(h, c, s, input, bias, output, stream, workspace, workspace_floats);
        (void)hipEventRecord(e1, stream);
        if (r != PATDNN_OK) return r;
        hipError_t he = hipEventSynchronize(e1);
        if (he != hipSuccess) return hip_fail(he, "hipEventSynchronize");
        ms = 0.0f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        ms /= (float)reps;
        return PATDNN_OK;
    };
    // first pass over every candidate, then the four fastest again, in turns (clocks and cache
    // contents drift while a process tunes: a candidate timed later is not timed under the
    // same conditions as one timed earlier), each judged by the median of its turns: the
    // winner of a noisy first pass should not stay by luck
    std::vector<std::pair<float, size_t>> timed;
    for (size_t i = 0; i < cands.size(); ++i) {
        float ms = 0.0f;
        st = time_config(cands[i], 3, ms);
        if (st != PATDNN_OK) { result = st; break; }
        timed.emplace_back(ms, i);
    }
    if (result == PATDNN_OK) {
        std::sort(timed.begin(), timed.end());
        const size_t finalists = std::min<size_t>(timed.size(), 4);
        constexpr int kTurns = 5;
        std::vector<std::vector<float>> turns(finalists);
        for (int t = 0; t < kTurns && result == PATDNN_OK; ++t)
            for (size_t k = 0; k < finalists; ++k) {
                float ms = 0.0f;
                st = time_config(cands[timed[k].second], 3, ms);
                if (st != PATDNN_OK) { result = st; break; }
                turns[k].push_back(ms);
            }
        for (size_t k = 0; k < finalists && result == PATDNN_OK; ++k) {
            std::sort(turns[k].begin(), turns[k].end());
            const float ms = turns[k][turns[k].size() / 2];
            if (best < 0.0f || ms < best) { best = ms; best_cfg = cands[timed[k].second]; }
        }
    }
    if (result != PATDNN_OK) return result;
    // leave a valid result of the chosen configuration in `output`
    st = run_config(h, best_cfg, s, input, bias, output, stream, workspace, workspace_floats);
    if (st != PATDNN_OK) return st;
    if ((e = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    h->cfg = best_cfg;
    h->cfg_tuned = true;
    // keep the winner's layout and the default variant's; free the others
    {
        auto default_layout = [&](int vi, int ck) {
            return !h->order.empty() && vi == h->order[0] && (tiled_variant(vi).dense || ck == default_ck(tiled_variant(vi), s.c_in));
        };
        for (auto it = h->tiled.begin(); it != h->tiled.end();) {
            const int vnum = it->first.first + 1;
            const bool dense = tiled_variant(it->first.first).dense;
            const bool keep = (vnum == best_cfg.variant && (dense || it->first.second == best_cfg.ck)) ||
                              default_layout(it->first.first, it->first.second);
            it = keep ? std::next(it) : h->tiled.erase(it);
        }
    }
    if (best_us) *best_us = best * 1000.0f;
    return PATDNN_OK;
}

patdnn_status_t patdnn_tune_ws(patdnn_handle_t h, const float* input, int32_t n, int32_t h_in,
                               int32_t w_in, const float* bias, float* output, float* workspace,
                               size_t workspace_floats, void* stream_, float* best_us)
{
    return guarded([&] { return tune_ws(h, input, n, h_in, w_in, bias, output, workspace, workspace_floats, stream_, best_us); });
}

static patdnn_status_t find_tiled(patdnn_handle_t h, int32_t variant, int32_t ck, TiledOnDevice** out)
{
    if (!h) return fail(PATDNN_EINVAL, "handle is NULL");
    const int vi = variant - 1;
    if (extra_variant(variant) >= 0 && variant < patdnn_num_variants())
        return fail(PATDNN_EUNSUPPORTED, "this variant has no filter-group layout");
    if (vi < 0 || vi >= num_tiled_variants()) return fail(PATDNN_EINVAL, "not a tiled variant");
    const TiledVariant& v = tiled_variant(vi);
    if (v.dense || !variant_fits_layer(h, v)) return fail(PATDNN_EUNSUPPORTED, "variant cannot run this layer");
    if (ck < 0) return fail(PATDNN_EINVAL, "ck out of range");
    if (ck == 0) ck = default_ck(v, h->L.desc.c_in);
    ck = std::min(ck, h->L.desc.c_in);
    if (ck * 4 * v.lds_buffers * v.lds_floats_per_channel > kMaxLdsBytes) return fail(PATDNN_EUNSUPPORTED, "ck exceeds the LDS budget");
    try {
        patdnn_status_t st = ensure_tiled(h, vi, ck, nullptr);
        if (st != PATDNN_OK) return st;
    } catch (const std::bad_alloc&) {
        return fail(PATDNN_ENOMEM, "out of host memory");
    }
    *out = h->tiled.find(std::make_pair(vi, ck))->second.get();
    return PATDNN_OK;
}

patdnn_status_t patdnn_tiled_info(patdnn_handle_t h, int32_t variant, int32_t ck, patdnn_tiled_info_t* out)
{
    if (!out) return fail(PATDNN_EINVAL, "out is NULL");
    TiledOnDevice* t = nullptr;
    patdnn_status_t st = find_tiled(h, variant, ck, &t);
    if (st != PATDNN_OK) return st;
    const TiledVariant& v = tiled_variant(variant - 1);
    out->G = t->host.G;
    out->num_groups = t->host.num_groups;
    out->ck = t->host.ck;
    out->num_chunks = t->host.num_chunks;
    out->num_steps = (int64_t)(t->host.steps.size() / kStepDwords);
    out->block_bytes = v.block_bytes;
    out->table_off = v.table_off;
    out->ctrl_bytes = v.ctrl_bytes;
    out->records = v.records;
    out->double_window = v.double_window ? 1 : 0;
    out->lds_channel_bytes = 4 * v.lds_floats_per_channel;
    out->threaded = v.threaded ? 1 : 0;
    out->patch_rows = v.PR;
    out->patch_cols = v.PC;
    out->conv_stride = v.S;
    out->lanes_x = v.TGX;
    out->experimental = v.experimental ? 1 : 0;
    out->mode = v.mode;
    return PATDNN_OK;
}

patdnn_status_t patdnn_export_tiled(patdnn_handle_t h, int32_t variant, int32_t ck,
                                    int32_t* slot_channel, uint32_t* chunk_ptr, uint32_t* steps)
{
    TiledOnDevice* t = nullptr;
    patdnn_status_t st = find_tiled(h, variant, ck, &t);
    if (st != PATDNN_OK) return st;
    auto get = [&](void* dst, const void* dev, const void* host, size_t bytes) -> hipError_t {
        if (!dst || !bytes) return hipSuccess;
        if (h->on_device) return hipMemcpy(dst, dev, bytes, hipMemcpyDeviceToHost);
        std::memcpy(dst, host, bytes);
        return hipSuccess;
    };
    hipError_t e;
    if ((e = get(slot_channel, t->dev.slot_channel, t->host.slot_channel.data(), t->host.slot_channel.size() * 4)) != hipSuccess ||
        (e = get(chunk_ptr, t->dev.chunk_ptr, t->host.chunk_ptr.data(), t->host.chunk_ptr.size() * 4)) != hipSuccess ||
        (e = get(steps, t->dev.steps, t->host.steps.data(), t->host.steps.size() * 4)) != hipSuccess)
        return hip_fail(e, "reading the tiled layout back");
    return PATDNN_OK;
}

patdnn_status_t patdnn_selftest(void)
{
    return guarded([]() -> patdnn_status_t {
        std::string why;
        if (!movrel_selftest(why)) return fail(PATDNN_EUNSUPPORTED, why);
        return PATDNN_OK;
    });
}

void patdnn_destroy(patdnn_handle_t h) { delete h; }

// ---------------------------------------------------------------------------
// A stack of layers run back to back (section 6.2: one image through all CONV layers)
// ---------------------------------------------------------------------------
}  // extern "C"

struct patdnn_stack {
    std::vector<patdnn_stack_layer_t> layers;
    int32_t n = 0;
    std::vector<int32_t> in_h, in_w;          // input size of every layer
    int32_t out_shape[4] = {0, 0, 0, 0};
    size_t max_intermediate = 0;              // floats of the largest tensor between two layers
    size_t buf_floats[2] = {0, 0};            // floats the tensors written to buffer 0 / 1 need
    size_t split_floats_min = 0;              // largest un-pooled output of a pooled layer (partial sums)
    size_t split_floats = 0;                  // >= split_floats_min: room for one buffer per channel slice
    float* buf[2] = {nullptr, nullptr};       // the stack's own ping-pong buffers
    float* split = nullptr;                   // and its buffer for the partial sums of split pooled layers
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    const float* graph_in = nullptr;
    float* graph_out = nullptr;
    bool warmed = false;                      // one plain run has set every function attribute

    ~patdnn_stack()
    {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        for (float* p : buf)
            if (p) (void)hipFree(p);
        if (split) (void)hipFree(split);
    }
};

namespace {

// every layer on `stream`, intermediates alternating between b0 and b1
patdnn_status_t stack_launch(patdnn_stack* s, const float* input, float* output, float* b0, float* b1,
                             float* split, size_t split_floats, hipStream_t stream)
{
    const int L = (int)s->layers.size();
    auto dst_of = [&](int i) { return i == L - 1 ? output : ((i & 1) ? b1 : b0); };
    const float* src = input;
    // A layer that ends with a finishing kernel (its input channels are split) clears there what
    // the next layer adds into, which saves that layer a fill launch of its own: some 5 us each,
    // a tenth of a single image's latency.  The region is the next layer's output (the buffer this
    // layer has just finished reading) or the partial-sum buffer, never what this layer itself
    // still reads or writes (the launcher checks the one case that could coincide).
    ZeroRegion zeroed;
    patdnn_config_t plan{}, next_plan{};          // of this layer and the next one (planned is false: not worked out)
    bool planned = false, next_planned = false;
    for (int i = 0; i < L; ++i, plan = next_plan, planned = next_planned) {
        float* dst = dst_of(i);
        const patdnn_stack_layer_t& ly = s->layers[i];
        ZeroHandoff hand;
        hand.pre_zeroed = zeroed;
        if (planned) hand.plan = &plan;
        next_planned = false;
        if (i + 1 < L) {
            const patdnn_stack_layer_t& nx = s->layers[i + 1];
            ConvShape ns{};
            if (shape_of(nx.layer, s->n, s->in_h[i + 1], s->in_w[i + 1], ns) == PATDNN_OK) {
                ns.pool = nx.pool2 ? 1 : 0;
                next_plan = effective_config(nx.layer, ns, split, split_floats);
                next_planned = true;
                hand.next = zero_need(next_plan, ns, dst_of(i + 1), split, split_floats);
            }
            if (hand.next.p == dst) hand.next = ZeroRegion{};     // this layer's own output: cannot happen
        }
        patdnn_status_t st = conv2d_impl(ly.layer, src, s->n, s->in_h[i], s->in_w[i], ly.bias, dst, ly.fuse_relu,
                                         ly.pool2, stream, split, split_floats, &hand);
        if (st != PATDNN_OK) return st;
        zeroed = hand.done ? hand.next : ZeroRegion{};
        src = dst;
    }
    return PATDNN_OK;
}

}  // namespace

extern "C" {

static patdnn_status_t stack_create(const patdnn_stack_layer_t* layers, int32_t num_layers, int32_t n,
                                    int32_t h_in, int32_t w_in, patdnn_stack_t* out)
{
    if (out) *out = nullptr;
    if (!layers || !out || num_layers <= 0 || n <= 0) return fail(PATDNN_EINVAL, "layers / out is NULL or a size is not positive");
    std::unique_ptr<patdnn_stack> s(new (std::nothrow) patdnn_stack());
    if (!s) return fail(PATDNN_ENOMEM, "out of host memory");
    s->n = n;
    int32_t h = h_in, w = w_in, c = -1;
    for (int i = 0; i < num_layers; ++i) {
        const patdnn_stack_layer_t& ly = layers[i];
        if (!ly.layer) return fail(PATDNN_EINVAL, "a layer handle is NULL");
        if (!ly.layer->on_device) return fail(PATDNN_EHIP, "a layer was encoded with PATDNN_HOST_ONLY");
        if (c >= 0 && ly.layer->L.desc.c_in != c) return fail(PATDNN_EINVAL, "channel counts of consecutive layers do not match");
        if (ly.pool2 && ly.layer->L.depthwise) return fail(PATDNN_EUNSUPPORTED, "fused pooling is not built for depthwise layers");
        ConvShape cs{};
        patdnn_status_t st = shape_of(ly.layer, n, h, w, cs);
        if (st != PATDNN_OK) return st;
        s->in_h.push_back(h);
        s->in_w.push_back(w);
        h = ly.pool2 ? cs.ho / 2 : cs.ho;
        w = ly.pool2 ? cs.wo / 2 : cs.wo;
        if (h <= 0 || w <= 0) return fail(PATDNN_EINVAL, "a layer's output is empty");
        c = cs.c_out;
        const size_t full = (size_t)n * c * cs.ho * cs.wo;
        if (ly.pool2) s->split_floats_min = std::max(s->split_floats_min, full);
        // one buffer per channel slice for the layers that are configured to split now (a layer
        // reconfigured later uses the room there is, or adds its slices up with atomics)
        cs.pool = ly.pool2 ? 1 : 0;
        const size_t want = split_room(ly.layer, cs);
        if (want <= kMaxSliceFloats) s->split_floats = std::max(s->split_floats, want);
        if (i + 1 < num_layers) {
            s->max_intermediate = std::max(s->max_intermediate, (size_t)n * c * h * w);
            s->buf_floats[i & 1] = std::max(s->buf_floats[i & 1], (size_t)n * c * h * w);
        }
        s->layers.push_back(ly);
    }
    s->out_shape[0] = n; s->out_shape[1] = c; s->out_shape[2] = h; s->out_shape[3] = w;
    s->split_floats = std::max(s->split_floats, s->split_floats_min);
    for (int k = 0; k < 2; ++k)
        if (s->buf_floats[k]) {
            hipError_t e = hipMalloc(reinterpret_cast<void**>(&s->buf[k]), s->buf_floats[k] * sizeof(float));
            if (e != hipSuccess) return hip_fail(e, "allocating the stack's intermediate tensors");
        }
    if (s->split_floats) {
        hipError_t e = hipMalloc(reinterpret_cast<void**>(&s->split), s->split_floats * sizeof(float));
        if (e != hipSuccess) return hip_fail(e, "allocating the stack's partial-sum buffer");
    }
    *out = s.release();
    return PATDNN_OK;
}

patdnn_status_t patdnn_stack_create(const patdnn_stack_layer_t* layers, int32_t num_layers, int32_t n,
                                    int32_t h_in, int32_t w_in, patdnn_stack_t* out)
{
    return guarded([&] { return stack_create(layers, num_layers, n, h_in, w_in, out); });
}

patdnn_status_t patdnn_stack_output_shape(patdnn_stack_t s, int32_t out_nchw[4])
{
    if (!s || !out_nchw) return fail(PATDNN_EINVAL, "stack / out_nchw is NULL");
    for (int i = 0; i < 4; ++i) out_nchw[i] = s->out_shape[i];
    return PATDNN_OK;
}

patdnn_status_t patdnn_stack_run(patdnn_stack_t s, const float* input, float* output, int32_t use_graph,
                                 void* stream_)
{
    if (!s) return fail(PATDNN_EINVAL, "stack is NULL");
    if (!input || !output) return fail(PATDNN_EINVAL, "input / output is NULL");
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    if (!use_graph) {
        patdnn_status_t st = stack_launch(s, input, output, s->buf[0], s->buf[1], s->split, s->split_floats, stream);
        if (st == PATDNN_OK) s->warmed = true;
        return st;
    }
    if (!stream) return fail(PATDNN_EINVAL, "graph execution needs a stream other than the default one");
    if (!s->exec || s->graph_in != input || s->graph_out != output) {
        // (re)capture: the graph holds the tensor addresses it was recorded with
        if (!s->warmed) {
            // a first plain run sets the per-kernel attributes, which must not happen in a capture
            patdnn_status_t st = stack_launch(s, input, output, s->buf[0], s->buf[1], s->split, s->split_floats, stream);
            if (st != PATDNN_OK) return st;
            s->warmed = true;
        }
        if (s->exec) { (void)hipGraphExecDestroy(s->exec); s->exec = nullptr; }
        if (s->graph) { (void)hipGraphDestroy(s->graph); s->graph = nullptr; }
        hipError_t e = hipStreamBeginCapture(stream, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return hip_fail(e, "hipStreamBeginCapture");
        patdnn_status_t st = stack_launch(s, input, output, s->buf[0], s->buf[1], s->split, s->split_floats, stream);
        e = hipStreamEndCapture(stream, &s->graph);
        if (st != PATDNN_OK) {
            if (s->graph) { (void)hipGraphDestroy(s->graph); s->graph = nullptr; }
            return st;
        }
        if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
        e = hipGraphInstantiate(&s->exec, s->graph, nullptr, nullptr, 0);
        if (e != hipSuccess) return hip_fail(e, "hipGraphInstantiate");
        s->graph_in = input;
        s->graph_out = output;
    }
    hipError_t e = hipGraphLaunch(s->exec, stream);
    return e == hipSuccess ? PATDNN_OK : hip_fail(e, "hipGraphLaunch");
}

void patdnn_stack_destroy(patdnn_stack_t s) { delete s; }

}  // extern "C"

// ---------------------------------------------------------------------------
// patdnn_stack_run without any allocation behind it: the tensors between the layers and the
// partial sums of split pooled layers live in one file-scope device array instead of the
// stack's own buffers.  Every GPU the library runs on holds its own copy of the array until
// the process ends; calls that overlap on one GPU share it and race.
// ---------------------------------------------------------------------------
namespace {

constexpr size_t kStaticScratchBytes = 32u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];              // device address of `scratch`, per device
std::mutex g_scratch_lock;

// The array's device address on the current device (looked up once per device; in host code
// the array's name is only a handle for this lookup, never an address to pass to a kernel).
hipError_t static_scratch(unsigned char** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *out = static_cast<unsigned char*>(g_scratch_ptr[dev]);
    return hipSuccess;
}

size_t round256(size_t bytes) { return (bytes + 255) / 256 * 256; }

}  // namespace

extern "C" {

patdnn_status_t patdnn_stack_run_static(patdnn_stack_t s, const float* input, float* output, void* stream)
{
    if (!s) return fail(PATDNN_EINVAL, "stack is NULL");
    if (!input || !output) return fail(PATDNN_EINVAL, "input / output is NULL");
    const size_t b0 = round256(s->buf_floats[0] * sizeof(float)), b1 = round256(s->buf_floats[1] * sizeof(float));
    // room for one partial-sum buffer per channel slice if the built-in buffer has it, else
    // the one buffer that split pooled layers cannot do without
    size_t sp_floats = s->split_floats;
    if (b0 + b1 + round256(sp_floats * sizeof(float)) > kStaticScratchBytes) sp_floats = s->split_floats_min;
    const size_t sp = round256(sp_floats * sizeof(float));
    if (b0 + b1 + sp > kStaticScratchBytes) {
        char msg[200];
        snprintf(msg, sizeof(msg), "the stack needs %zu bytes between its layers; the built-in buffer of "
                 "patdnn_stack_run_static holds %zu", b0 + b1 + sp, kStaticScratchBytes);
        return fail(PATDNN_EUNSUPPORTED, msg);
    }
    unsigned char* base = nullptr;
    hipError_t e = static_scratch(&base);
    if (e != hipSuccess) return hip_fail(e, "looking up the built-in buffer");
    // nothing here needs to start at zero: the kernels clear the pooled outputs and partial
    // sums they accumulate into, whatever an earlier call left behind
    return stack_launch(s, input, output, reinterpret_cast<float*>(base), reinterpret_cast<float*>(base + b0),
                        reinterpret_cast<float*>(base + b0 + b1), sp_floats, static_cast<hipStream_t>(stream));
}

const char* patdnn_status_string(patdnn_status_t s)
{
    switch (s) {
        case PATDNN_OK: return "ok";
        case PATDNN_EINVAL: return "invalid argument";
        case PATDNN_EPATTERN: return "pattern constraint violated";
        case PATDNN_ENOMEM: return "out of host memory";
        case PATDNN_EHIP: return "HIP runtime error";
        case PATDNN_EUNSUPPORTED: return "unsupported";
    }
    return "unknown status";
}

const char* patdnn_last_error(void) { return g_err.c_str(); }

}  // extern "C"
