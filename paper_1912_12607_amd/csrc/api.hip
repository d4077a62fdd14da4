// C ABI of the library (see include/int8t.h): argument validation, scratch carving, dispatch.
// No device memory is allocated here and nothing synchronises with the host.
#include <math.h>

#include <algorithm>
#include <array>
#include <map>
#include <mutex>

#include "../../include/int8t.h"
#include "kernels.h"
#include "device_common.h"

using namespace int8t;

// Scratch of int8t_dsgc_clip_static: the clip search's absmax partials, its 64-bit accumulator sets
// with the ticket word, and the sum-of-squares partials -- the same three areas int8t_dsgc_clip carves
// out of the caller's scratch.  One copy per GPU, held until the process ends.
#define INT8T_STATIC_A256(v) (((v) + 255) & ~(size_t)255)
constexpr size_t kStaticDsgcBytes = INT8T_STATIC_A256(kMaxPartials * sizeof(float)) +
                                    INT8T_STATIC_A256((kDsgcAccWords + 1) * sizeof(unsigned long long)) +
                                    INT8T_STATIC_A256(kMaxPartials * sizeof(double));
static __device__ __align__(256) unsigned char scratch[kStaticDsgcBytes];

namespace {

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
inline int pad16(int v) { return (v + 15) & ~15; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
inline bool aligned8(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 7) == 0; }
inline bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3) == 0; }

// whether two ranges of bytes share one
inline bool overlap(const void* p, size_t np, const void* q, size_t nq) {
    return (uintptr_t)p < (uintptr_t)q + nq && (uintptr_t)q < (uintptr_t)p + np;
}

constexpr size_t kMaxElems = 0x7FFFFFFFull;   // 32-bit indices inside the kernels

bool dims_ok(const int d[4], size_t* n) {
    if (!d) return false;
    size_t t = 1;
    for (int i = 0; i < 4; ++i) {
        if (d[i] <= 0) return false;
        t *= (size_t)d[i];
        if (t > kMaxElems) return false;
    }
    *n = t;
    return true;
}

struct Geo {
    int P, Q;
    bool depthwise;
};

int8t_status desc_ok(const int8t_conv_desc* d, Geo* g) {
    if (!d) return INT8T_ERR_NULL;
    if (d->N <= 0 || d->C <= 0 || d->H <= 0 || d->W <= 0 || d->K <= 0 || d->R <= 0 || d->S <= 0 ||
        d->stride_h <= 0 || d->stride_w <= 0 || d->pad_h < 0 || d->pad_w < 0 || d->groups <= 0)
        return INT8T_ERR_SHAPE;
    if (d->H + 2 * d->pad_h < d->R || d->W + 2 * d->pad_w < d->S) return INT8T_ERR_SHAPE;
    g->P = (d->H + 2 * d->pad_h - d->R) / d->stride_h + 1;
    g->Q = (d->W + 2 * d->pad_w - d->S) / d->stride_w + 1;
    if (d->groups == 1) g->depthwise = false;
    else if (d->groups == d->C && d->K == d->C) g->depthwise = true;
    else return INT8T_ERR_SHAPE;
    // element counts must fit the kernels' 32-bit indices (padded channel pitch included)
    const size_t nx = (size_t)d->N * pad16(d->C) * d->H * d->W;
    const size_t ny = (size_t)d->N * pad16(d->K) * g->P * g->Q;
    const size_t nw = (size_t)pad16(d->K) * pad16(d->C / d->groups) * d->R * d->S;
    if (nx > kMaxElems || ny > kMaxElems || nw > kMaxElems) return INT8T_ERR_SHAPE;
    if ((size_t)g->P * g->Q > (1u << 22) || (size_t)d->H * d->W > (1u << 22)) return INT8T_ERR_SHAPE;
    if (g->depthwise) {
        if (d->R * d->S > 64) return INT8T_ERR_SHAPE;
        if ((size_t)d->H * d->W + (size_t)g->P * g->Q > 48000) return INT8T_ERR_SHAPE;   // LDS planes
    }
    return INT8T_OK;
}

// scratch of int8t_quantize: [absmax partials][deviation partials]
size_t quant_ws_bytes(int blocks) { return align256(kMaxPartials * sizeof(float)) + align256((size_t)blocks * sizeof(DevPartial)); }

// The pass that writes a tensor's codes.  Channels-last codes of a 1 x 1 image whose channel count
// needs no padding (the input of a fully connected layer) are the tensor's own element order: the
// element-wise pass writes them, instead of the transposing one at one pixel per block.
int8t_kind pass_kind(const int d[4], int8t_kind kind) {
    if (kind == INT8T_ACT && d[2] * d[3] == 1 && (d[1] & 15) == 0) return INT8T_ACT_PLANAR;
    return kind;
}

int quant_blocks(const int d[4], int8t_kind kind) {
    switch (pass_kind(d, kind)) {
        case INT8T_ACT: return quant_blocks_act(d[0], pad16(d[1]), d[2] * d[3]);
        case INT8T_WGT: return quant_blocks_wgt(d[0], d[1], d[2], d[3]);
        default: return quant_blocks_planar((size_t)d[0] * d[1] * d[2] * d[3]);
    }
}

size_t dsgc_ws_bytes(size_t n) {
    (void)n;
    return align256(kMaxPartials * sizeof(float)) + align256((dsgc_acc_words() + 1) * sizeof(unsigned long long)) +
           align256(kMaxPartials * sizeof(double));
}

void fill_wgrad_geometry(WgradArgs* a, const int8t_conv_desc* d, const Geo& g) {
    a->N = d->N; a->C = d->C; a->Cp = pad16(d->C); a->H = d->H; a->W = d->W;
    a->K = d->K; a->Kp = pad16(d->K); a->P = g.P; a->Q = g.Q; a->R = d->R; a->S = d->S;
    a->stride_h = d->stride_h; a->stride_w = d->stride_w; a->pad_h = d->pad_h; a->pad_w = d->pad_w;
}

// geometry of the depthwise passes (pointers are set by the entry points)
DwArgs dw_args(const int8t_conv_desc* d, const Geo& g, bool dgrad) {
    DwArgs a{};
    a.N = d->N; a.C = d->C; a.R = d->R; a.S = d->S;
    a.IH = dgrad ? g.P : d->H; a.IW = dgrad ? g.Q : d->W;
    a.OH = dgrad ? d->H : g.P; a.OW = dgrad ? d->W : g.Q;
    a.stride_h = d->stride_h; a.stride_w = d->stride_w; a.pad_h = d->pad_h; a.pad_w = d->pad_w;
    a.dgrad = dgrad;
    return a;
}
DwArgs dw_wgrad_args(const int8t_conv_desc* d, const Geo& g) {
    DwArgs a = dw_args(d, g, false);
    dw_wgrad_shape(d->N, d->C, d->H, d->W, g.P, g.Q, d->R, d->S, d->stride_h, d->stride_w, &a.threads, &a.chunks, &a.cg);
    return a;
}

// geometry of the implicit GEMMs (pointers are set by the entry points)
void fill_igemm_fwd(IgemmArgs* a, const int8t_conv_desc* d, const Geo& g) {
    a->N = d->N; a->rows = d->K; a->Ca = pad16(d->C);
    a->IH = d->H; a->IW = d->W; a->OH = g.P; a->OW = g.Q; a->R = d->R; a->S = d->S;
    a->stride_h = d->stride_h; a->stride_w = d->stride_w; a->pad_h = d->pad_h; a->pad_w = d->pad_w;
    a->dgrad = 0;
    a->C = d->C;
}
void fill_igemm_bwd_data(IgemmArgs* a, const int8t_conv_desc* d, const Geo& g) {
    a->N = d->N; a->rows = d->C; a->Ca = pad16(d->K);
    a->IH = g.P; a->IW = g.Q; a->OH = d->H; a->OW = d->W; a->R = d->R; a->S = d->S;
    a->stride_h = d->stride_h; a->stride_w = d->stride_w; a->pad_h = d->pad_h; a->pad_w = d->pad_w;
    a->dgrad = 1;
}

// Kernel variants selected per (pass, layer) by int8t_conv_select_variant; everything else runs the
// library's own choice.  Process-wide, guarded by a mutex (a lookup per convolution call).
std::mutex g_variant_mutex;
std::map<std::array<int, 13>, int> g_variant_table;

// What the forward pass of a layer that runs in space-to-depth form puts at the front of its scratch, 0: another layer
size_t fwd_s2d_bytes(const int8t_conv_desc* d, const Geo& g) {
    if (g.depthwise) return 0;
    IgemmArgs a{};
    fill_igemm_fwd(&a, d, g);
    return igemm_s2d(&a);
}

std::array<int, 13> variant_key(int8t_op op, const int8t_conv_desc* d) {
    return {(int)op, d->N, d->C, d->H, d->W, d->K, d->R, d->S, d->stride_h, d->stride_w, d->pad_h, d->pad_w, d->groups};
}
int selected_variant(int8t_op op, const int8t_conv_desc* d) {
    std::lock_guard<std::mutex> lock(g_variant_mutex);
    if (g_variant_table.empty()) return VAR_AUTO;
    const auto it = g_variant_table.find(variant_key(op, d));
    return it == g_variant_table.end() ? VAR_AUTO : it->second;
}

// whether `variant` can run pass `op` of the layer
bool variant_ok(int8t_op op, const int8t_conv_desc* d, const Geo& g, int variant) {
    if (variant == VAR_AUTO) return true;
    if (g.depthwise) return false;
    if (op == INT8T_OP_CONV_BWD_WEIGHT) {
        if (variant == VAR_WGRAD_FEWER || variant == VAR_WGRAD_MORE || variant == VAR_WGRAD_IMAGES) return true;
        if (variant != VAR_WGRAD_LINES) return false;
        WgradArgs a{};
        fill_wgrad_geometry(&a, d, g);
        (void)wgrad_s2d(&a);
        return wgrad_lines_applies(a);
    }
    if (op != INT8T_OP_CONV_FWD && op != INT8T_OP_CONV_BWD_DATA) return false;
    IgemmArgs a{};
    if (op == INT8T_OP_CONV_FWD) fill_igemm_fwd(&a, d, g);
    else fill_igemm_bwd_data(&a, d, g);
    (void)igemm_s2d(&a);      // a layer that runs on its space-to-depth form is judged in that form
    return igemm_variant_ok(a, variant);
}

}  // namespace

extern "C" {

int int8t_conv_variant_ok(int8t_op op, const int8t_conv_desc* desc, int8t_variant variant) {
    Geo g;
    if (desc_ok(desc, &g) != INT8T_OK) return 0;
    if ((int)variant < 0 || (int)variant >= VAR_COUNT) return 0;
    return variant_ok(op, desc, g, (int)variant) ? 1 : 0;
}

int8t_status int8t_conv_select_variant(int8t_op op, const int8t_conv_desc* desc, int8t_variant variant) {
    Geo g;
    const int8t_status s = desc_ok(desc, &g);
    if (s != INT8T_OK) return s;
    if (op != INT8T_OP_CONV_FWD && op != INT8T_OP_CONV_BWD_DATA && op != INT8T_OP_CONV_BWD_WEIGHT) return INT8T_ERR_ARG;
    if ((int)variant < 0 || (int)variant >= VAR_COUNT || !variant_ok(op, desc, g, (int)variant)) return INT8T_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_variant_mutex);
    if (variant == INT8T_VARIANT_AUTO) g_variant_table.erase(variant_key(op, desc));
    else g_variant_table[variant_key(op, desc)] = (int)variant;
    return INT8T_OK;
}

int8t_variant int8t_conv_selected_variant(int8t_op op, const int8t_conv_desc* desc) {
    Geo g;
    if (desc_ok(desc, &g) != INT8T_OK) return INT8T_VARIANT_AUTO;
    return (int8t_variant)selected_variant(op, desc);
}

const char* int8t_status_string(int8t_status s) {
    switch (s) {
        case INT8T_OK: return "ok";
        case INT8T_ERR_NULL: return "required pointer is NULL";
        case INT8T_ERR_SHAPE: return "bad or unsupported shape";
        case INT8T_ERR_ARG: return "bad argument (enum value, alignment, candidate count)";
        case INT8T_ERR_WORKSPACE: return "workspace too small";
        case INT8T_ERR_RUNTIME: return "HIP launch failed";
        case INT8T_ERR_LIMIT: return "size beyond the limit of the allocation-free variant";
        default: break;
    }
    return "unknown status";
}

size_t int8t_code_bytes(const int dims[4], int8t_kind kind) {
    size_t n;
    if (!dims_ok(dims, &n)) return 0;
    switch (kind) {
        case INT8T_ACT: return (size_t)dims[0] * dims[2] * dims[3] * pad16(dims[1]);
        case INT8T_WGT:
            return align256((size_t)dims[0] * dims[2] * dims[3] * pad16(dims[1])) +
                   (size_t)dims[1] * dims[2] * dims[3] * pad16(dims[0]);
        case INT8T_ACT_PLANAR:
        case INT8T_WGT_PLANAR: return n;
        default: break;
    }
    return 0;
}

int8t_status int8t_unpack_codes(const int8_t* codes_host, const int dims[4], int8t_kind kind, int copy,
                                int8_t* out_host, size_t* pad_nonzero) {
    if (!codes_host || !dims || !out_host) return INT8T_ERR_NULL;
    size_t n;
    if (!dims_ok(dims, &n)) return INT8T_ERR_SHAPE;
    if (kind != INT8T_ACT && kind != INT8T_WGT && kind != INT8T_ACT_PLANAR && kind != INT8T_WGT_PLANAR) return INT8T_ERR_ARG;
    if (copy != 0 && !(kind == INT8T_WGT && copy == 1)) return INT8T_ERR_ARG;
    size_t bad = 0;
    if (kind == INT8T_ACT_PLANAR || kind == INT8T_WGT_PLANAR) {
        for (size_t i = 0; i < n; ++i) out_host[i] = codes_host[i];
    } else {
        // both dense layouts are [outer][plane position][inner padded to 16]: activations outer = N,
        // inner = C; weights, forward copy outer = K, inner = Cg; backward-data copy outer = Cg, inner = K
        const int plane = dims[2] * dims[3];
        const bool second = kind == INT8T_WGT && copy == 1;
        const int outer = second ? dims[1] : dims[0], inner = second ? dims[0] : dims[1];
        const int ip = pad16(inner);
        const int8_t* src = codes_host;
        if (second) src += align256((size_t)dims[0] * plane * pad16(dims[1]));
        for (int o = 0; o < outer; ++o)
            for (int p = 0; p < plane; ++p) {
                const int8_t* g = src + ((size_t)o * plane + p) * ip;
                for (int i = 0; i < inner; ++i) {
                    // logical index: [dims0][dims1][plane]
                    const size_t d0 = second ? (size_t)i : (size_t)o, d1 = second ? (size_t)o : (size_t)i;
                    out_host[(d0 * dims[1] + d1) * plane + p] = g[i];
                }
                for (int i = inner; i < ip; ++i) bad += g[i] != 0;
            }
    }
    if (pad_nonzero) *pad_nonzero = bad;
    return INT8T_OK;
}

size_t int8t_workspace_bytes(int8t_op op, const int8t_conv_desc* desc, size_t n, int n_cand) {
    (void)n_cand;
    switch (op) {
        case INT8T_OP_QUANTIZE: return 0;
        case INT8T_OP_DSGC: return dsgc_ws_bytes(n);
        case INT8T_OP_CONV_FWD:
        case INT8T_OP_CONV_BWD_DATA: {
            // optional: partial sums of a split reduction (layers with few output tiles)
            Geo g;
            if (desc_ok(desc, &g) != INT8T_OK || g.depthwise) return 0;
            // ... and, in the forward pass of a stride-2 layer with at most 4 channels, its rewritten codes
            IgemmArgs a{};
            if (op == INT8T_OP_CONV_FWD) fill_igemm_fwd(&a, desc, g);
            else fill_igemm_bwd_data(&a, desc, g);
            const size_t s2d_bytes = igemm_s2d(&a);   // (sized for the split variant whichever is selected)
            const int ks = igemm_ksplit(a);
            return s2d_bytes + (ks > 1 ? align256((size_t)ks * a.N * a.rows * a.OH * a.OW * 4) : 0);
        }
        case INT8T_OP_CONV_BWD_WEIGHT: {
            Geo g;
            if (desc_ok(desc, &g) != INT8T_OK) return 0;
            if (g.depthwise) {
                int threads, chunks, cg;
                dw_wgrad_shape(desc->N, desc->C, desc->H, desc->W, g.P, g.Q, desc->R, desc->S, desc->stride_h, desc->stride_w, &threads, &chunks, &cg);
                return align256((size_t)chunks * desc->C * desc->R * desc->S * 4);
            }
            WgradArgs a{};
            fill_wgrad_geometry(&a, desc, g);
            const size_t s2d_bytes = wgrad_s2d(&a);
            a.variant = selected_variant(INT8T_OP_CONV_BWD_WEIGHT, desc);
            wgrad_plan(&a);
            return wgrad_partial_bytes(a) + align256(s2d_bytes);
        }
        default: break;
    }
    return 0;
}

size_t int8t_quantize_workspace_bytes(const int dims[4], int8t_kind kind) {
    size_t n;
    if (!dims_ok(dims, &n)) return 0;
    if (kind != INT8T_ACT && kind != INT8T_WGT && kind != INT8T_ACT_PLANAR && kind != INT8T_WGT_PLANAR) return 0;
    return quant_ws_bytes(quant_blocks(dims, kind));
}

int8t_status int8t_quantize(const float* x_dev, const int dims[4], int8t_kind kind,
                            const float* clip_dev, int8t_round mode, uint64_t seed, int8_t* q_dev,
                            float* scale_dev, double* deviation_dev, void* ws_dev, size_t ws_bytes,
                            void* stream) {
    if (!x_dev || !dims || !q_dev || !scale_dev) return INT8T_ERR_NULL;
    size_t n;
    if (!dims_ok(dims, &n)) return INT8T_ERR_SHAPE;
    if (kind != INT8T_ACT && kind != INT8T_WGT && kind != INT8T_ACT_PLANAR && kind != INT8T_WGT_PLANAR)
        return INT8T_ERR_ARG;
    if (mode != INT8T_ROUND_NEAREST_EVEN && mode != INT8T_ROUND_STOCHASTIC) return INT8T_ERR_ARG;
    if (!aligned16(x_dev) || !aligned16(q_dev) || !aligned4(scale_dev)) return INT8T_ERR_ARG;
    if (kind == INT8T_ACT && (size_t)dims[0] * pad16(dims[1]) * dims[2] * dims[3] > kMaxElems) return INT8T_ERR_SHAPE;
    if (kind == INT8T_ACT && dims[0] > 65535) return INT8T_ERR_SHAPE;   // grid.z
    const bool need_absmax = (clip_dev == nullptr);
    const bool need_dev = (deviation_dev != nullptr);
    const int blocks = quant_blocks(dims, kind);
    if (need_absmax || need_dev) {
        if (!ws_dev) return INT8T_ERR_NULL;
        if (ws_bytes < quant_ws_bytes(need_dev ? blocks : 0)) return INT8T_ERR_WORKSPACE;
        if (!aligned16(ws_dev)) return INT8T_ERR_ARG;
    }
    hipStream_t st = (hipStream_t)stream;
    char* ws = (char*)ws_dev;
    float* absmax_part = (float*)ws;
    DevPartial* devpart = need_dev ? (DevPartial*)(ws + align256(kMaxPartials * sizeof(float))) : nullptr;

    int nparts = 0;
    if (need_absmax && launch_absmax(x_dev, n, absmax_part, &nparts, st) != hipSuccess) return INT8T_ERR_RUNTIME;
    QuantArgs a;
    a.x = x_dev;
    a.d0 = dims[0]; a.d1 = dims[1]; a.d2 = dims[2]; a.d3 = dims[3];
    a.clip = clip_dev;
    a.absmax_part = absmax_part;
    a.nparts = nparts;
    a.stochastic = (mode == INT8T_ROUND_STOCHASTIC);
    a.seed = seed;
    a.q = q_dev;
    a.scale = scale_dev;
    a.devpart = devpart;
    hipError_t e;
    const int8t_kind pk = pass_kind(dims, kind);
    if (pk == INT8T_ACT) e = launch_quantize_act(a, st);
    else if (pk == INT8T_WGT) e = launch_quantize_wgt(a, st);
    else e = launch_quantize_planar(a, st);
    if (e != hipSuccess) return INT8T_ERR_RUNTIME;
    if (need_dev && launch_deviation_finish(devpart, blocks, deviation_dev, st) != hipSuccess) return INT8T_ERR_RUNTIME;
    return INT8T_OK;
}

size_t int8t_quantize_batch_workspace_bytes(int count, const int8t_quantize_item* items) {
    if (count < 1 || count > INT8T_MAX_BATCH || !items) return 0;
    return (size_t)count * align256(kMaxPartials * sizeof(float));
}

}  // extern "C"

namespace {
DsgcWs dsgc_ws_layout(void* ws_dev);

// Argument checks of a batch of tensors (and of the tensor of a clip search beside them); codes: their codes and scales are
// written, not only their maxima found.
int8t_status quantize_batch_check(int count, const int8t_quantize_item* items, bool codes, const void* ws_dev, size_t ws_bytes,
                                  const float* g_dev, size_t g_n, const void* dsgc_ws_dev, size_t dsgc_ws_size) {
    if (!items) return INT8T_ERR_NULL;
    if (count < 1 || count > INT8T_MAX_BATCH) return INT8T_ERR_ARG;
    if (g_dev) {
        if (!dsgc_ws_dev) return INT8T_ERR_NULL;
        if (g_n == 0 || g_n > kMaxElems) return INT8T_ERR_SHAPE;
        if (!aligned16(g_dev) || !aligned16(dsgc_ws_dev)) return INT8T_ERR_ARG;
        if (dsgc_ws_size < dsgc_ws_bytes(g_n)) return INT8T_ERR_WORKSPACE;
    }
    bool any_absmax = false;
    for (int i = 0; i < count; ++i) {
        const int8t_quantize_item& it = items[i];
        if (!it.x_dev || (codes && (!it.q_dev || !it.scale_dev))) return INT8T_ERR_NULL;
        size_t n;
        if (!dims_ok(it.dims, &n)) return INT8T_ERR_SHAPE;
        if (it.kind != INT8T_ACT && it.kind != INT8T_WGT && it.kind != INT8T_ACT_PLANAR && it.kind != INT8T_WGT_PLANAR)
            return INT8T_ERR_ARG;
        if (it.mode != INT8T_ROUND_NEAREST_EVEN && it.mode != INT8T_ROUND_STOCHASTIC) return INT8T_ERR_ARG;
        if (!aligned16(it.x_dev) || !aligned16(it.q_dev) || !aligned4(it.scale_dev) || !aligned4(it.clip_dev))
            return INT8T_ERR_ARG;
        if (it.kind == INT8T_ACT && (size_t)it.dims[0] * pad16(it.dims[1]) * it.dims[2] * it.dims[3] > kMaxElems)
            return INT8T_ERR_SHAPE;
        if (!it.clip_dev) any_absmax = true;
    }
    if (any_absmax) {
        if (!ws_dev) return INT8T_ERR_NULL;
        if (ws_bytes < int8t_quantize_batch_workspace_bytes(count, items)) return INT8T_ERR_WORKSPACE;
        if (!aligned16(ws_dev)) return INT8T_ERR_ARG;
    }
    return INT8T_OK;
}

// Block ranges are dealt smallest tensor first: the dispatcher hands out blocks in order, so the
// few blocks of a small tensor run beside the first blocks of a large one instead of after its last.
void batch_order(int count, const int8t_quantize_item* items, int order[INT8T_MAX_BATCH], size_t sizes[INT8T_MAX_BATCH]) {
    for (int i = 0; i < count; ++i) {
        order[i] = i;
        (void)dims_ok(items[i].dims, &sizes[i]);
    }
    for (int i = 1; i < count; ++i)
        for (int j = i; j > 0 && sizes[order[j]] < sizes[order[j - 1]]; --j) { const int t = order[j]; order[j] = order[j - 1]; order[j - 1] = t; }
}
float* batch_partials(void* ws_dev, int i) { return (float*)((char*)ws_dev + (size_t)i * align256(kMaxPartials * sizeof(float))); }

// First launch of a batch: the absmax partials of the items without a clip value and, with g_dev, the first phase of a
// clip search on g.  (checked arguments)
// sums: the column sums of `sums_of` (g_n elements) as a matrix of `cols` columns, in the same launch.
hipError_t batch_absmax(int count, const int8t_quantize_item* items, void* ws_dev, const float* g_dev, size_t g_n, void* dsgc_ws_dev,
                        hipStream_t st, float* sums = nullptr, const float* sums_of = nullptr, int cols = 0) {
    AbsmaxBatch ab{};
    std::fill(std::begin(ab.block0), std::end(ab.block0), 0x7fffffff);
    long long ablocks = 0;
    int order[INT8T_MAX_BATCH];
    size_t sizes[INT8T_MAX_BATCH];
    if (sums) {
        ab.block0[ab.count] = (int)ablocks;
        AbsmaxBatchItem& a = ab.it[ab.count++];
        a.x = sums_of; a.n = g_n; a.part = sums; a.cols = cols; a.nblocks = absmax_colsum_blocks(cols);
        ablocks += a.nblocks;
    }
    batch_order(count, items, order, sizes);
    for (int oi = 0; oi < count; ++oi) {
        const int i = order[oi];
        if (items[i].clip_dev) continue;
        ab.block0[ab.count] = (int)ablocks;
        AbsmaxBatchItem& a = ab.it[ab.count++];
        a.x = items[i].x_dev; a.n = sizes[i]; a.part = batch_partials(ws_dev, i); a.nblocks = absmax_blocks(sizes[i]);
        ablocks += a.nblocks;
    }
    if (g_dev) {
        const DsgcWs dws = dsgc_ws_layout(dsgc_ws_dev);
        ab.block0[ab.count] = (int)ablocks;
        AbsmaxBatchItem& a = ab.it[ab.count++];
        a.x = g_dev; a.n = g_n; a.part = dws.absmax_part; a.nblocks = absmax_blocks(g_n);
        a.sumsq = dws.partG; a.zero = dws.acc; a.nzero = (int)dsgc_acc_words() + 1;
        ablocks += a.nblocks;
    }
    return ab.count ? launch_absmax_batch(ab, (int)ablocks, st) : hipSuccess;
}

int batch_kind(const int8t_quantize_item& it) {
    const int8t_kind pk = pass_kind(it.dims, it.kind);
    return pk == INT8T_ACT ? 0 : pk == INT8T_WGT ? 1 : 2;
}

// Second launch: the codes and scales, from the clip values and the partials of the first.  (checked arguments)
// s2d (nullable): where the space-to-depth codes of the first item go, activations of at most 4 channels rounded to nearest.
int8t_status batch_codes(int count, const int8t_quantize_item* items, void* ws_dev, hipStream_t st, int8_t* s2d = nullptr) {
    QuantBatch qb{};
    qb.count = count;
    std::fill(std::begin(qb.block0), std::end(qb.block0), 0x7fffffff);
    long long qblocks = 0;
    int order[INT8T_MAX_BATCH];
    size_t sizes[INT8T_MAX_BATCH];
    batch_order(count, items, order, sizes);
    for (int oi = 0; oi < count; ++oi) {
        const int i = order[oi];
        const int8t_quantize_item& it = items[i];
        QuantBatchItem& q = qb.it[oi];
        q.x = it.x_dev; q.d0 = it.dims[0]; q.d1 = it.dims[1]; q.d2 = it.dims[2]; q.d3 = it.dims[3];
        q.clip = it.clip_dev; q.absmax_part = it.clip_dev ? nullptr : batch_partials(ws_dev, i); q.nparts = it.clip_dev ? 0 : absmax_blocks(sizes[i]);
        q.q = it.q_dev; q.scale = it.scale_dev;
        q.kind = batch_kind(it);
        q.stoch = it.mode == INT8T_ROUND_STOCHASTIC;
        q.seed_lo = seed_key_x(it.seed);
        q.seed_hi = seed_key_a(it.seed);
        quant_grid(q.kind, it.dims, &q.gx, &q.gy, &q.gz);
        if (s2d && i == 0) {
            q.kind = 3;
            q.gx = (int)(((size_t)q.d0 * ((q.d2 + 1) / 2) * ((q.d3 + 1) / 2) + 255) / 256);      // (no more blocks than of kind 0)
            q.gy = q.gz = 1;
        }
        qb.block0[oi] = (int)qblocks;
        qblocks += (long long)q.gx * q.gy * q.gz;      // (batch_blocks_ok)
    }
    return launch_quantize_batch(qb, (int)qblocks, st, s2d) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
}

// the codes' launch has one block index over all tensors of a batch
bool batch_blocks_ok(int count, const int8t_quantize_item* items) {
    long long blocks = 0;
    for (int i = 0; i < count; ++i) {
        int gx, gy, gz;
        quant_grid(batch_kind(items[i]), items[i].dims, &gx, &gy, &gz);
        blocks += (long long)gx * gy * gz;
    }
    return blocks <= 0x7FFFFFFFll;
}

// int8t_quantize_batch, and with g_dev also the first phase of a clip search on g in the same absmax launch
int8t_status quantize_batch_impl(int count, const int8t_quantize_item* items, void* ws_dev, size_t ws_bytes,
                                 const float* g_dev, size_t g_n, void* dsgc_ws_dev, size_t dsgc_ws_size, void* stream) {
    const int8t_status s = quantize_batch_check(count, items, true, ws_dev, ws_bytes, g_dev, g_n, dsgc_ws_dev, dsgc_ws_size);
    if (s != INT8T_OK) return s;
    if (!batch_blocks_ok(count, items)) return INT8T_ERR_SHAPE;
    if (batch_absmax(count, items, ws_dev, g_dev, g_n, dsgc_ws_dev, (hipStream_t)stream) != hipSuccess) return INT8T_ERR_RUNTIME;
    return batch_codes(count, items, ws_dev, (hipStream_t)stream);
}
}  // namespace

extern "C" {

int8t_status int8t_quantize_batch(int count, const int8t_quantize_item* items, void* ws_dev, size_t ws_bytes,
                                  void* stream) {
    return quantize_batch_impl(count, items, ws_dev, ws_bytes, nullptr, 0, nullptr, 0, stream);
}

int8t_status int8t_quantize_batch_prepare(int count, const int8t_quantize_item* items, void* ws_dev, size_t ws_bytes,
                                          const float* g_dev, size_t n, void* dsgc_ws_dev, size_t dsgc_ws_size,
                                          void* stream) {
    if (!g_dev) return INT8T_ERR_NULL;
    return quantize_batch_impl(count, items, ws_dev, ws_bytes, g_dev, n, dsgc_ws_dev, dsgc_ws_size, stream);
}

namespace {
DsgcWs dsgc_ws_layout(void* ws_dev) {
    char* p = (char*)ws_dev;
    DsgcWs ws;
    const size_t nacc = dsgc_acc_words();
    ws.absmax_part = (float*)p;                 p += align256(kMaxPartials * sizeof(float));
    ws.acc = (unsigned long long*)p;
    ws.ticket = (unsigned int*)(ws.acc + nacc);  p += align256((nacc + 1) * sizeof(unsigned long long));
    ws.partG = (double*)p;
    return ws;
}
}  // namespace

int8t_status int8t_dsgc_prepare(const float* g_dev, size_t n, void* ws_dev, size_t ws_bytes, void* stream) {
    if (!g_dev || !ws_dev) return INT8T_ERR_NULL;
    if (n == 0 || n > kMaxElems) return INT8T_ERR_SHAPE;
    if (!aligned16(g_dev) || !aligned16(ws_dev)) return INT8T_ERR_ARG;
    if (ws_bytes < dsgc_ws_bytes(n)) return INT8T_ERR_WORKSPACE;
    const DsgcWs ws = dsgc_ws_layout(ws_dev);
    int nparts = 0;
    if (launch_absmax(g_dev, n, ws.absmax_part, &nparts, (hipStream_t)stream, ws.partG, ws.acc,
                      (int)dsgc_acc_words() + 1) != hipSuccess)
        return INT8T_ERR_RUNTIME;
    return INT8T_OK;
}

int8t_status int8t_dsgc_search(const float* g_dev, size_t n, const float* ratios_dev, int n_cand,
                               int8t_round mode, uint64_t seed, float* clip_dev, double* deviation_dev,
                               double* deviation_all_dev, void* ws_dev, size_t ws_bytes, void* stream) {
    if (!g_dev || !ratios_dev || !clip_dev || !deviation_dev || !ws_dev) return INT8T_ERR_NULL;
    if (n == 0 || n > kMaxElems) return INT8T_ERR_SHAPE;
    if (n_cand < 1 || n_cand > INT8T_MAX_CANDIDATES) return INT8T_ERR_ARG;
    if (mode != INT8T_ROUND_NEAREST_EVEN && mode != INT8T_ROUND_STOCHASTIC) return INT8T_ERR_ARG;
    if (!aligned16(g_dev) || !aligned16(ws_dev) || !aligned4(ratios_dev) || !aligned4(clip_dev) ||
        !aligned8(deviation_dev) || !aligned8(deviation_all_dev))
        return INT8T_ERR_ARG;
    if (ws_bytes < dsgc_ws_bytes(n)) return INT8T_ERR_WORKSPACE;
    const DsgcWs ws = dsgc_ws_layout(ws_dev);
    if (launch_dsgc(g_dev, n, ratios_dev, n_cand, mode == INT8T_ROUND_STOCHASTIC, seed, ws, absmax_blocks(n), clip_dev,
                    deviation_dev, deviation_all_dev, (hipStream_t)stream) != hipSuccess)
        return INT8T_ERR_RUNTIME;
    return INT8T_OK;
}

int8t_status int8t_dsgc_clip(const float* g_dev, size_t n, const float* ratios_dev, int n_cand,
                             int8t_round mode, uint64_t seed, float* clip_dev, double* deviation_dev,
                             double* deviation_all_dev, void* ws_dev, size_t ws_bytes, void* stream) {
    // argument checks of both phases first, so that nothing is launched on bad input
    if (!g_dev || !ratios_dev || !clip_dev || !deviation_dev || !ws_dev) return INT8T_ERR_NULL;
    if (n == 0 || n > kMaxElems) return INT8T_ERR_SHAPE;
    if (n_cand < 1 || n_cand > INT8T_MAX_CANDIDATES) return INT8T_ERR_ARG;
    if (mode != INT8T_ROUND_NEAREST_EVEN && mode != INT8T_ROUND_STOCHASTIC) return INT8T_ERR_ARG;
    if (!aligned16(g_dev) || !aligned16(ws_dev) || !aligned4(ratios_dev) || !aligned4(clip_dev) ||
        !aligned8(deviation_dev) || !aligned8(deviation_all_dev))
        return INT8T_ERR_ARG;
    if (ws_bytes < dsgc_ws_bytes(n)) return INT8T_ERR_WORKSPACE;
    int8t_status s = int8t_dsgc_prepare(g_dev, n, ws_dev, ws_bytes, stream);
    if (s != INT8T_OK) return s;
    return int8t_dsgc_search(g_dev, n, ratios_dev, n_cand, mode, seed, clip_dev, deviation_dev, deviation_all_dev,
                             ws_dev, ws_bytes, stream);
}

namespace {
// Device address of `scratch` on each GPU (every GPU holds its own copy of the array at its own
// address); looked up once per device, with that device current, by the first call on it.
constexpr int kMaxDevices = 64;
std::atomic<void*> g_static_scratch[kMaxDevices];

int8t_status static_scratch(void** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return INT8T_ERR_RUNTIME;
    void* p = g_static_scratch[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return INT8T_ERR_RUNTIME;
        g_static_scratch[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return INT8T_OK;
}
}  // namespace

int8t_status int8t_dsgc_clip_static(const float* g_dev, size_t n, const float* ratios_dev, int n_cand,
                                    int8t_round mode, uint64_t seed, float* clip_dev, double* deviation_dev,
                                    double* deviation_all_dev, void* stream) {
    if (!g_dev || !ratios_dev || !clip_dev || !deviation_dev) return INT8T_ERR_NULL;
    if (n == 0) return INT8T_ERR_SHAPE;
    if (n > INT8T_DSGC_STATIC_MAX_ELEMS || n_cand > INT8T_MAX_CANDIDATES) return INT8T_ERR_LIMIT;
    static_assert(INT8T_DSGC_STATIC_MAX_ELEMS <= kMaxElems, "the static variant's limit is the kernels' own");
    static_assert(kStaticDsgcBytes == INT8T_DSGC_STATIC_SCRATCH_BYTES, "size stated in the header");
    void* ws = nullptr;
    const int8t_status s = static_scratch(&ws);
    if (s != INT8T_OK) return s;
    if (dsgc_ws_bytes(n) > kStaticDsgcBytes) return INT8T_ERR_LIMIT;
    // the same two phases on the GPU's own array; the first pass clears the accumulators and the
    // ticket with its own stores (no memset node, so a caller may capture the call into a graph)
    return int8t_dsgc_clip(g_dev, n, ratios_dev, n_cand, mode, seed, clip_dev, deviation_dev, deviation_all_dev, ws,
                           kStaticDsgcBytes, stream);
}

static int8t_status conv_fwd(const int8t_conv_desc* desc, const int8_t* xq_dev, const float* sx_dev, const int8_t* wq_dev, const float* sw_dev,
                             float* y_dev, int32_t* acc_dev, void* ws_dev, size_t ws_bytes, bool s2d_ready, void* stream);
int8t_status int8t_conv_fwd(const int8t_conv_desc* desc, const int8_t* xq_dev, const float* sx_dev,
                            const int8_t* wq_dev, const float* sw_dev, float* y_dev, int32_t* acc_dev,
                            void* ws_dev, size_t ws_bytes, void* stream) {
    return conv_fwd(desc, xq_dev, sx_dev, wq_dev, sw_dev, y_dev, acc_dev, ws_dev, ws_bytes, false, stream);
}

// s2d_ready: the space-to-depth codes of a lie in the scratch already
static int8t_status conv_fwd(const int8t_conv_desc* desc, const int8_t* xq_dev, const float* sx_dev, const int8_t* wq_dev, const float* sw_dev,
                             float* y_dev, int32_t* acc_dev, void* ws_dev, size_t ws_bytes, bool s2d_ready, void* stream) {
    Geo g;
    int8t_status s = desc_ok(desc, &g);
    if (s != INT8T_OK) return s;
    if (!xq_dev || !sx_dev || !wq_dev || !sw_dev || !y_dev) return INT8T_ERR_NULL;
    if (!aligned16(xq_dev) || !aligned16(wq_dev) || !aligned16(y_dev) || !aligned4(acc_dev) || !aligned16(ws_dev))
        return INT8T_ERR_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (g.depthwise) {
        DwArgs a = dw_args(desc, g, false);
        a.a = xq_dev; a.b = wq_dev; a.sa = sx_dev; a.sb = sw_dev; a.out = y_dev; a.acc = acc_dev;
        return launch_dw_conv(a, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
    }
    IgemmArgs a{};
    fill_igemm_fwd(&a, desc, g);
    a.variant = selected_variant(INT8T_OP_CONV_FWD, desc);
    a.act = xq_dev; a.wgt = wq_dev; a.sa = sx_dev; a.sb = sw_dev; a.out = y_dev; a.acc = acc_dev;
    a.partial = (int32_t*)ws_dev; a.partial_bytes = ws_dev ? ws_bytes : 0;
    {
        // the rewritten codes of a layer s2d.hip covers come first in the scratch; without it the layer runs as it is
        IgemmArgs t = a;
        const size_t s2d_bytes = igemm_s2d(&t);
        if (s2d_bytes && a.partial_bytes >= s2d_bytes) {
            a.s2d = (int8_t*)ws_dev;
            a.s2d_ready = s2d_ready;
            a.partial = (int32_t*)((int8_t*)ws_dev + s2d_bytes);
            a.partial_bytes -= s2d_bytes;
        }
    }
    return launch_igemm(a, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
}

int8t_status int8t_conv_fwd_fused(const int8t_conv_desc* desc, const float* x_dev, const float* clip_dev,
                                  const int8_t* wq_dev, const float* sw_dev, float* y_dev, int32_t* acc_dev,
                                  int8_t* xq_dev, float* sx_dev, void* ws_dev, size_t ws_bytes, void* stream) {
    Geo g;
    int8t_status s = desc_ok(desc, &g);
    if (s != INT8T_OK) return s;
    if (g.depthwise || desc->R != 1 || desc->S != 1 || desc->stride_h != 1 || desc->stride_w != 1 || desc->pad_h || desc->pad_w)
        return INT8T_ERR_SHAPE;
    if (!x_dev || !wq_dev || !sw_dev || !y_dev || !sx_dev) return INT8T_ERR_NULL;
    if (!aligned16(x_dev) || !aligned16(wq_dev) || !aligned16(y_dev) || !aligned4(acc_dev) || !aligned16(xq_dev) ||
        !aligned4(sx_dev) || !aligned4(clip_dev) || !aligned16(ws_dev))
        return INT8T_ERR_ARG;
    if (!clip_dev) {
        if (!ws_dev) return INT8T_ERR_NULL;
        if (ws_bytes < kMaxPartials * sizeof(float)) return INT8T_ERR_WORKSPACE;
    }
    hipStream_t st = (hipStream_t)stream;
    IgemmArgs a{};
    fill_igemm_fwd(&a, desc, g);
    a.xf = x_dev; a.xclip = clip_dev; a.xq_out = xq_dev; a.sx_out = sx_dev;
    a.wgt = wq_dev; a.sb = sw_dev; a.out = y_dev; a.acc = acc_dev;
    if (!clip_dev) {
        a.xabs_part = (const float*)ws_dev;
        if (launch_absmax(x_dev, (size_t)desc->N * desc->C * desc->H * desc->W, (float*)ws_dev, &a.xabs_nparts, st) != hipSuccess)
            return INT8T_ERR_RUNTIME;
    }
    return launch_igemm_fused(a, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
}

int8t_status int8t_conv_bwd_data(const int8t_conv_desc* desc, const int8_t* dyq_dev, const float* sdy_dev,
                                 const int8_t* wq_dev, const float* sw_dev, float* dx_dev, int32_t* acc_dev,
                                 void* ws_dev, size_t ws_bytes, void* stream) {
    Geo g;
    int8t_status s = desc_ok(desc, &g);
    if (s != INT8T_OK) return s;
    if (!dyq_dev || !sdy_dev || !wq_dev || !sw_dev || !dx_dev) return INT8T_ERR_NULL;
    if (!aligned16(dyq_dev) || !aligned16(wq_dev) || !aligned16(dx_dev) || !aligned4(acc_dev) || !aligned16(ws_dev))
        return INT8T_ERR_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (g.depthwise) {
        DwArgs a = dw_args(desc, g, true);
        a.a = dyq_dev; a.b = wq_dev; a.sa = sdy_dev; a.sb = sw_dev; a.out = dx_dev; a.acc = acc_dev;
        return launch_dw_conv(a, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
    }
    IgemmArgs a{};
    fill_igemm_bwd_data(&a, desc, g);
    a.variant = selected_variant(INT8T_OP_CONV_BWD_DATA, desc);
    a.act = dyq_dev;
    // second copy of the weight codes: [C][R][S][Kp]
    a.wgt = wq_dev + align256((size_t)desc->K * desc->R * desc->S * pad16(desc->C));
    a.sa = sdy_dev; a.sb = sw_dev; a.out = dx_dev; a.acc = acc_dev;
    a.partial = (int32_t*)ws_dev; a.partial_bytes = ws_dev ? ws_bytes : 0;
    return launch_igemm(a, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
}

int8t_status int8t_conv_bwd_weight(const int8t_conv_desc* desc, const int8_t* xq_dev, const float* sx_dev,
                                   const int8_t* dyq_dev, const float* sdy_dev, float* dw_dev, int32_t* acc_dev,
                                   void* ws_dev, size_t ws_bytes, void* stream) {
    return int8t_conv_bwd_weight_fwd(desc, xq_dev, sx_dev, dyq_dev, sdy_dev, dw_dev, acc_dev, ws_dev, ws_bytes, nullptr, 0, stream);
}

int8t_status int8t_conv_bwd_weight_fwd(const int8t_conv_desc* desc, const int8_t* xq_dev, const float* sx_dev,
                                       const int8_t* dyq_dev, const float* sdy_dev, float* dw_dev, int32_t* acc_dev,
                                       void* ws_dev, size_t ws_bytes, const void* fwd_ws_dev, size_t fwd_ws_bytes, void* stream) {
    Geo g;
    int8t_status s = desc_ok(desc, &g);
    if (s != INT8T_OK) return s;
    if (!xq_dev || !sx_dev || !dyq_dev || !sdy_dev || !dw_dev || !ws_dev) return INT8T_ERR_NULL;
    if (!aligned16(xq_dev) || !aligned16(dyq_dev) || !aligned16(dw_dev) || !aligned4(acc_dev) || !aligned16(ws_dev) || !aligned16(fwd_ws_dev))
        return INT8T_ERR_ARG;
    if (ws_bytes < int8t_workspace_bytes(INT8T_OP_CONV_BWD_WEIGHT, desc, 0, 0)) return INT8T_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    if (g.depthwise) {
        DwArgs a = dw_wgrad_args(desc, g);
        a.a = xq_dev; a.b = dyq_dev; a.sa = sx_dev; a.sb = sdy_dev; a.out = dw_dev; a.acc = acc_dev;
        a.partial = (int32_t*)ws_dev;
        return launch_dw_wgrad(a, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
    }
    WgradArgs a{};
    fill_wgrad_geometry(&a, desc, g);
    wgrad_s2d(&a);
    a.variant = selected_variant(INT8T_OP_CONV_BWD_WEIGHT, desc);
    wgrad_plan(&a);
    a.x = xq_dev; a.dy = dyq_dev; a.sa = sx_dev; a.sb = sdy_dev; a.dw = dw_dev; a.acc = acc_dev;
    a.partial = (int32_t*)ws_dev;
    a.xs = (int8_t*)ws_dev + wgrad_partial_bytes(a);
    const size_t fwd_bytes = fwd_s2d_bytes(desc, g);
    const bool apart = (uintptr_t)fwd_ws_dev + fwd_bytes <= (uintptr_t)ws_dev || (uintptr_t)ws_dev + ws_bytes <= (uintptr_t)fwd_ws_dev;
    if (fwd_ws_dev && fwd_bytes && fwd_ws_bytes >= fwd_bytes && apart) {
        a.xs = (int8_t*)const_cast<void*>(fwd_ws_dev);      // (read only)
        a.xs_ready = 1;
    }
    // (the result of a reduction may go where the codes lay, that of a tile may not)
    const int xd[4] = {desc->N, desc->C, desc->H, desc->W}, yd[4] = {desc->N, desc->K, g.P, g.Q};
    const size_t nw = (size_t)desc->K * desc->C * desc->R * desc->S * 4;
    a.direct = wgrad_single_share(a);
    for (const void* out : {(const void*)dw_dev, (const void*)acc_dev})
        if (out && (overlap(out, nw, xq_dev, int8t_code_bytes(xd, INT8T_ACT)) || overlap(out, nw, dyq_dev, int8t_code_bytes(yd, INT8T_ACT)) ||
                    overlap(out, nw, sx_dev, 4) || overlap(out, nw, sdy_dev, 4)))
            a.direct = 0;
    return launch_wgrad(a, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
}

// Whether the codes of a that the forward pass of a step leaves in its scratch (int8t_conv_bwd_weight_fwd) are still there when
// backward-weight runs: nothing that is written from then on overlaps them.
static bool fwd_scratch_kept(const int8t_conv_desc* d, const Geo& g, const int8t_layer_buffers* b, bool bwd_data) {
    const size_t bytes = fwd_s2d_bytes(d, g);
    if (!b->ws_fwd || !bytes || b->ws_fwd_bytes < bytes) return false;
    struct Range { const void* p; size_t n; };
    const size_t nx = (size_t)d->N * d->C * d->H * d->W * 4, ny = (size_t)d->N * d->K * g.P * g.Q * 4, nw = (size_t)d->K * d->C * d->R * d->S * 4;
    const Range r[] = {{b->y, ny}, {b->y_acc, ny}, {bwd_data ? b->dx : nullptr, nx}, {bwd_data ? b->dx_acc : nullptr, nx},
                       {bwd_data ? b->ws_bwd_data : nullptr, b->ws_bwd_data_bytes}, {b->ws_bwd_weight, b->ws_bwd_weight_bytes}, {b->dw, nw}, {b->dw_acc, nw}};
    const uintptr_t q = (uintptr_t)b->ws_fwd;
    for (const Range& t : r) {
        const uintptr_t p = (uintptr_t)t.p;
        if (p && p < q + bytes && q < p + t.n) return false;
    }
    return true;
}

// Where a step that forms the codes of a (and of g_z: quant_g) and runs the forward pass may put the space-to-depth codes of a with the ordinary
// ones: the forward pass's scratch, if nothing that is read or written up to that pass lies in it.  nullptr: the pass rewrites the codes itself (so
// do the autograd modules, whose partial maxima and forward scratch are one buffer).
static int8_t* s2d_with_codes(const int8t_conv_desc* d, const Geo& g, const int8t_layer_buffers* b, bool quant_g) {
    const size_t bytes = fwd_s2d_bytes(d, g);
    if (!bytes || !b->ws_fwd || b->ws_fwd_bytes < bytes) return nullptr;
    struct Range { const void* p; size_t n; };
    const size_t nx = (size_t)d->N * d->C * d->H * d->W * 4, ny = (size_t)d->N * d->K * g.P * g.Q * 4, nw = (size_t)d->K * d->C * d->R * d->S * 4;
    const int xd[4] = {d->N, d->C, d->H, d->W}, wd[4] = {d->K, d->C, d->R, d->S}, yd[4] = {d->N, d->K, g.P, g.Q};
    const Range r[] = {{b->x, nx}, {b->w, nw}, {b->ws_quant, b->ws_quant_bytes}, {b->xq, int8t_code_bytes(xd, INT8T_ACT)}, {b->sx, 4},
                       {b->wq, int8t_code_bytes(wd, INT8T_WGT)}, {b->sw, 4}, {quant_g ? b->dy : nullptr, ny}, {quant_g ? b->clip : nullptr, 4},
                       {quant_g ? b->dyq : nullptr, int8t_code_bytes(yd, INT8T_ACT)}, {quant_g ? b->sdy : nullptr, 4},
                       {quant_g ? b->ws_dy : nullptr, b->ws_dy_bytes}, {quant_g ? b->dev_final : nullptr, 8}};
    for (const Range& t : r)
        if (t.p && overlap(t.p, t.n, b->ws_fwd, bytes)) return nullptr;
    return (int8_t*)b->ws_fwd;
}

// Whether what the three passes of a step write overlaps nothing that one of them reads or writes, so that they may run
// side by side (one after the other, a pass may reuse the buffers of the passes before it).
static bool disjoint_results(const int8t_conv_desc* d, const Geo& g, const int8t_layer_buffers* b, bool fwd) {
    struct Range { const void* p; size_t n; };
    const size_t nx = (size_t)d->N * d->C * d->H * d->W * 4, ny = (size_t)d->N * d->K * g.P * g.Q * 4;
    const int Cg = d->C / d->groups;
    const size_t nw = (size_t)d->K * Cg * d->R * d->S * 4;
    const int8t_kind ak = g.depthwise ? INT8T_ACT_PLANAR : INT8T_ACT, wk = g.depthwise ? INT8T_WGT_PLANAR : INT8T_WGT;
    const int xd[4] = {d->N, d->C, d->H, d->W}, wd[4] = {d->K, Cg, d->R, d->S}, yd[4] = {d->N, d->K, g.P, g.Q};
    // (dw comes from the second launch: it may not overlap a result or an input of the first, which are written or read before)
    const Range r[] = {{fwd ? b->y : nullptr, ny}, {fwd ? b->y_acc : nullptr, ny}, {b->dx, nx}, {b->dx_acc, nx}, {b->ws_bwd_weight, b->ws_bwd_weight_bytes},
                       {b->dw, nw}, {b->dw_acc, nw},
                       {b->xq, int8t_code_bytes(xd, ak)}, {b->wq, int8t_code_bytes(wd, wk)}, {b->dyq, int8t_code_bytes(yd, ak)},
                       {b->sx, 4}, {b->sw, 4}, {b->sdy, 4}};
    for (int i = 0; i < 7; ++i)
        for (int j = i + 1; j < 13; ++j) {
            const uintptr_t p = (uintptr_t)r[i].p, q = (uintptr_t)r[j].p;
            if (p && q && p < q + r[j].n && q < p + r[i].n) return false;
        }
    return true;
}

// The same for quantization and passes side by side: what they write overlaps nothing that they read or write.  x: codes of a and
// W and the forward pass, dy: codes of g_z and the backward passes.
static bool disjoint_step(const int8t_conv_desc* d, const Geo& g, const int8t_layer_buffers* b, bool x, bool dy) {
    struct Range { const void* p; size_t n; bool written; };
    const size_t nx = (size_t)d->N * d->C * d->H * d->W * 4, ny = (size_t)d->N * d->K * g.P * g.Q * 4;
    const int Cg = d->C / d->groups;
    const size_t nw = (size_t)d->K * Cg * d->R * d->S * 4;
    const int8t_kind ak = g.depthwise ? INT8T_ACT_PLANAR : INT8T_ACT, wk = g.depthwise ? INT8T_WGT_PLANAR : INT8T_WGT;
    const int xd[4] = {d->N, d->C, d->H, d->W}, wd[4] = {d->K, Cg, d->R, d->S}, yd[4] = {d->N, d->K, g.P, g.Q};
    const Range r[] = {{x ? b->x : nullptr, nx, false}, {x ? b->w : nullptr, nw, false}, {x ? b->ws_quant : nullptr, b->ws_quant_bytes, false},
                       {dy ? b->dy : nullptr, ny, false}, {dy ? b->clip : nullptr, 4, false},
                       {b->xq, int8t_code_bytes(xd, ak), x}, {b->wq, int8t_code_bytes(wd, wk), x}, {b->sx, 4, x}, {b->sw, 4, x},
                       {x ? b->y : nullptr, ny, true}, {x ? b->y_acc : nullptr, ny, true},
                       {dy ? b->dyq : nullptr, int8t_code_bytes(yd, ak), true}, {dy ? b->sdy : nullptr, 4, true},
                       {dy ? b->dx : nullptr, nx, true}, {dy ? b->dx_acc : nullptr, nx, true}, {dy ? b->dw : nullptr, nw, true},
                       {dy ? b->dw_acc : nullptr, nw, true}, {dy ? b->ws_bwd_weight : nullptr, b->ws_bwd_weight_bytes, true}};
    constexpr int count = sizeof(r) / sizeof(r[0]);
    for (int i = 0; i < count; ++i)
        for (int j = i + 1; j < count; ++j) {
            const uintptr_t p = (uintptr_t)r[i].p, q = (uintptr_t)r[j].p;
            if ((r[i].written || r[j].written) && p && q && p < q + r[j].n && q < p + r[i].n) return false;
        }
    return true;
}

// Depthwise layers whose codes are formed in the launch of the passes (conv_dw_fused.hip): the parts that belong together
// are all asked for, codes of a and W with the forward pass (x), codes of g_z with the two backward ones (dy).
static bool dw_fused_parts(const int8t_conv_desc* d, const Geo& g, int parts, bool* x, bool* dy) {
    constexpr int kX = INT8T_STEP_QUANT_XW | INT8T_STEP_FWD, kDy = INT8T_STEP_QUANT_G | INT8T_STEP_BWD_DATA | INT8T_STEP_BWD_WEIGHT;
    *x = (parts & kX) == kX;
    *dy = (parts & kDy) == kDy;
    return g.depthwise && d->R == 3 && d->S == 3 && d->stride_h == 1 && d->stride_w == 1 && d->pad_h == 1 && d->pad_w == 1 &&
           (*x || *dy) && *x == ((parts & kX) != 0) && *dy == ((parts & kDy) != 0);
}

// The passes of a dense layer as their launches plan them: geometry, selected variants, backward-weight's plan, and the scratch that
// a split reduction would take.  (all other pointers are set by the caller)
struct DensePasses {
    IgemmArgs f{}, d{};
    WgradArgs w{};
};
static void dense_passes(DensePasses* p, const int8t_conv_desc* desc, const Geo& g, void* ws_fwd, size_t ws_fwd_bytes, void* ws_bwd_data,
                         size_t ws_bwd_data_bytes) {
    fill_igemm_fwd(&p->f, desc, g);
    p->f.variant = selected_variant(INT8T_OP_CONV_FWD, desc);
    p->f.partial = (int32_t*)ws_fwd; p->f.partial_bytes = ws_fwd_bytes;
    fill_igemm_bwd_data(&p->d, desc, g);
    p->d.variant = selected_variant(INT8T_OP_CONV_BWD_DATA, desc);
    p->d.partial = (int32_t*)ws_bwd_data; p->d.partial_bytes = ws_bwd_data_bytes;
    fill_wgrad_geometry(&p->w, desc, g);
    wgrad_s2d(&p->w);
    p->w.variant = selected_variant(INT8T_OP_CONV_BWD_WEIGHT, desc);
    wgrad_plan(&p->w);
}

int8t_form int8t_layer_step_form(const int8t_conv_desc* desc, int parts) {
    Geo g;
    if (desc_ok(desc, &g) != INT8T_OK || parts <= 0 || parts > INT8T_STEP_ALL) return INT8T_FORM_APART;
    const bool fwd = parts & INT8T_STEP_FWD, both = (parts & INT8T_STEP_BWD_DATA) && (parts & INT8T_STEP_BWD_WEIGHT);
    if (g.depthwise) {
        const DwArgs w = dw_wgrad_args(desc, g);
        bool x, dy;
        if (dw_fused_parts(desc, g, parts, &x, &dy) && dw_fused_applies(desc->H, desc->W, w)) return INT8T_FORM_DW_CODES;
        return both && dw_trio_applies(dw_args(desc, g, true), w) ? INT8T_FORM_DW_PASSES : INT8T_FORM_APART;
    }
    if (!both) return INT8T_FORM_APART;
    DensePasses p;
    int scratch;      // (its address is only looked at)
    dense_passes(&p, desc, g, &scratch, int8t_workspace_bytes(INT8T_OP_CONV_FWD, desc, 0, 0), &scratch,
                 int8t_workspace_bytes(INT8T_OP_CONV_BWD_DATA, desc, 0, 0));
    if (desc->stride_h != 1 || desc->stride_w != 1) {
        if (!conv_trio_strided(fwd ? &p.f : nullptr, p.d, p.w)) return INT8T_FORM_APART;
        int form = STRIDED_PLAIN;
        (void)igemm_strided_blocks(&p.d, &form);
        return form == STRIDED_PLAIN     ? INT8T_FORM_STRIDED
               : form == STRIDED_CLASSES ? INT8T_FORM_STRIDED_CLASSES
               : form == STRIDED_CELL    ? INT8T_FORM_STRIDED_CELL
                                         : INT8T_FORM_STRIDED_CELLS;
    }
    const TrioTile tile = conv_trio_tile(fwd && !conv_trio_fwd_apart(p.f, p.d) ? &p.f : nullptr, p.d, p.w);
    if (!tile.bn) return conv_band_trio(nullptr, p.d, p.w) ? INT8T_FORM_BANDS : INT8T_FORM_APART;
    if (tile.rows64) return tile.bn == 64 ? INT8T_FORM_64X128 : INT8T_FORM_64X128_AND_128X128;
    return tile.bn == 64 ? INT8T_FORM_128X64 : INT8T_FORM_128X128;
}

// int8t_layer_step, int8t_layer_backward (the first phase of the search without max|a| and max|W|, and the column sums db of g_z)
// and int8t_layer_infer (codes and scales may be left out).
enum class StepForm { kStep, kBackward, kInfer };
static int8t_status layer_step(const int8t_conv_desc* desc, const int8t_layer_buffers* b, int parts, uint64_t seed, StepForm form, float* db,
                               void* stream) {
    const bool backward = form == StepForm::kBackward;
    Geo g;
    int8t_status s = desc_ok(desc, &g);
    if (s != INT8T_OK) return s;
    if (!b) return INT8T_ERR_NULL;
    if (parts <= 0 || parts > INT8T_STEP_ALL) return INT8T_ERR_ARG;
    const bool absmax = parts & INT8T_STEP_ABSMAX, prepare = parts & INT8T_STEP_PREPARE, search = parts & INT8T_STEP_SEARCH;
    const bool quant_xw = parts & INT8T_STEP_QUANT_XW, quant_g = parts & INT8T_STEP_QUANT_G;
    const bool fwd = parts & INT8T_STEP_FWD, bwd_data = parts & INT8T_STEP_BWD_DATA, bwd_weight = parts & INT8T_STEP_BWD_WEIGHT;
    if (backward ? absmax || quant_xw || fwd || prepare != search || (db && g.P * g.Q != 1) : prepare && !absmax) return INT8T_ERR_ARG;
    if (db && !b->dy) return INT8T_ERR_NULL;
    if (db && (!aligned4(db) || !aligned4(b->dy))) return INT8T_ERR_ARG;
    const int8t_kind ak = g.depthwise ? INT8T_ACT_PLANAR : INT8T_ACT, wk = g.depthwise ? INT8T_WGT_PLANAR : INT8T_WGT;
    const size_t n_y = (size_t)desc->N * desc->K * g.P * g.Q;
    const int ydims[4] = {desc->N, desc->K, g.P, g.Q};
    // a, W and g_z as a batch; g_z goes with the other two where its codes are wanted at the same time and no deviation is
    int8t_quantize_item it[3] = {};
    it[0].x_dev = b->x; it[0].q_dev = b->xq; it[0].scale_dev = b->sx; it[0].kind = ak;
    it[1].x_dev = b->w; it[1].q_dev = b->wq; it[1].scale_dev = b->sw; it[1].kind = wk;
    it[2].x_dev = b->dy; it[2].q_dev = b->dyq; it[2].scale_dev = b->sdy; it[2].kind = ak;
    it[2].clip_dev = b->clip; it[2].mode = INT8T_ROUND_STOCHASTIC; it[2].seed = seed;
    const int xd[4] = {desc->N, desc->C, desc->H, desc->W}, wd[4] = {desc->K, desc->C / desc->groups, desc->R, desc->S};
    for (int i = 0; i < 4; ++i) { it[0].dims[i] = xd[i]; it[1].dims[i] = wd[i]; it[2].dims[i] = ydims[i]; }
    const bool g_in_batch = quant_xw && quant_g && !b->dev_final;
    // ---- everything that can be wrong, before the first launch
    if (quant_g && !b->clip) return INT8T_ERR_NULL;
    if (absmax || quant_xw) {
        s = quantize_batch_check(g_in_batch ? 3 : 2, it, quant_xw, b->ws_quant, b->ws_quant_bytes, prepare ? b->dy : nullptr, n_y, b->ws_dy, b->ws_dy_bytes);
        if (s != INT8T_OK) return s;
        if (quant_xw && !batch_blocks_ok(g_in_batch ? 3 : 2, it)) return INT8T_ERR_SHAPE;
        if (prepare && !b->dy) return INT8T_ERR_NULL;
    }
    if (search) {
        if (!b->dy || !b->ratios || !b->clip || !b->dev_search || !b->ws_dy) return INT8T_ERR_NULL;
        if (b->n_cand < 1 || b->n_cand > INT8T_MAX_CANDIDATES || !aligned16(b->dy) || !aligned16(b->ws_dy) || !aligned4(b->ratios) ||
            !aligned4(b->clip) || !aligned8(b->dev_search) || !aligned8(b->dev_all))
            return INT8T_ERR_ARG;
        if (b->ws_dy_bytes < dsgc_ws_bytes(n_y)) return INT8T_ERR_WORKSPACE;
    }
    // the partials of a and W and the search's scratch are in use at the same time
    if ((absmax || quant_xw) && (prepare || search)) {
        const uintptr_t p = (uintptr_t)b->ws_quant, q = (uintptr_t)b->ws_dy;
        if (p < q + dsgc_ws_bytes(n_y) && q < p + int8t_quantize_batch_workspace_bytes(2, it)) return INT8T_ERR_ARG;
    }
    if (quant_g && !g_in_batch) {
        if (!b->dy || !b->dyq || !b->sdy || (b->dev_final && !b->ws_dy)) return INT8T_ERR_NULL;
        if (!aligned16(b->dy) || !aligned16(b->dyq) || !aligned4(b->sdy) || (b->dev_final && !aligned16(b->ws_dy))) return INT8T_ERR_ARG;
        if (ak == INT8T_ACT && desc->N > 65535) return INT8T_ERR_SHAPE;      // grid.z of the channels-last pass, as in int8t_quantize
        if (b->dev_final && b->ws_dy_bytes < int8t_quantize_workspace_bytes(ydims, ak)) return INT8T_ERR_WORKSPACE;
    }
    if (((fwd || bwd_weight) && (!b->xq || !b->sx)) || ((fwd || bwd_data) && (!b->wq || !b->sw)) ||
        ((bwd_data || bwd_weight) && (!b->dyq || !b->sdy)) || (fwd && !b->y) || (bwd_data && !b->dx) ||
        (bwd_weight && (!b->dw || !b->ws_bwd_weight)))
        return INT8T_ERR_NULL;
    if (((fwd || bwd_weight) && !aligned16(b->xq)) || ((fwd || bwd_data) && !aligned16(b->wq)) || ((bwd_data || bwd_weight) && !aligned16(b->dyq)) ||
        (fwd && (!aligned16(b->y) || !aligned4(b->y_acc))) || (bwd_data && (!aligned16(b->dx) || !aligned4(b->dx_acc))) ||
        (bwd_weight && (!aligned16(b->dw) || !aligned4(b->dw_acc) || !aligned16(b->ws_bwd_weight))) ||
        !aligned16(b->ws_fwd) || !aligned16(b->ws_bwd_data))
        return INT8T_ERR_ARG;
    if (bwd_weight && b->ws_bwd_weight_bytes < int8t_workspace_bytes(INT8T_OP_CONV_BWD_WEIGHT, desc, 0, 0)) return INT8T_ERR_WORKSPACE;
    // Depthwise layers whose codes are formed in this call: quantization and passes in one launch (conv_dw_fused.hip), where nothing
    // overlaps what another part of the call reads or writes.
    bool dw_x = false, dw_g = false;
    const bool dw_fused = dw_fused_parts(desc, g, parts, &dw_x, &dw_g) && !(quant_g && b->dev_final) && disjoint_step(desc, g, b, dw_x, dw_g);
    int8_t* const s2d = quant_xw && fwd ? s2d_with_codes(desc, g, b, quant_g) : nullptr;
    // ---- launches
    hipStream_t st = (hipStream_t)stream;
    if (absmax && batch_absmax(2, it, b->ws_quant, prepare ? b->dy : nullptr, n_y, b->ws_dy, st) != hipSuccess) return INT8T_ERR_RUNTIME;
    if (backward && (prepare || db) && batch_absmax(0, nullptr, nullptr, prepare ? b->dy : nullptr, n_y, b->ws_dy, st, db, b->dy, desc->K) != hipSuccess)
        return INT8T_ERR_RUNTIME;
    if (form == StepForm::kInfer && !g.depthwise && desc->R == 1 && desc->S == 1 && desc->stride_h == 1 && desc->stride_w == 1 && desc->pad_h == 0 &&
        desc->pad_w == 0 && !b->y_acc && selected_variant(INT8T_OP_CONV_FWD, desc) == VAR_AUTO) {
        size_t nx = 0, nw = 0;
        (void)dims_ok(xd, &nx);
        (void)dims_ok(wd, &nw);
        InferArgs a{};
        a.x = b->x; a.w = b->w; a.y = b->y;
        a.N = desc->N; a.C = desc->C; a.K = desc->K; a.HW = desc->H * desc->W;
        a.part_x = batch_partials(b->ws_quant, 0); a.np_x = absmax_blocks(nx);
        a.part_w = batch_partials(b->ws_quant, 1); a.np_w = absmax_blocks(nw);
        const uintptr_t y = (uintptr_t)b->y, ye = y + n_y * 4;      // the results are written while the tensors are read
        const bool apart = (ye <= (uintptr_t)b->x || (uintptr_t)b->x + nx * 4 <= y) && (ye <= (uintptr_t)b->w || (uintptr_t)b->w + nw * 4 <= y) &&
                           (ye <= (uintptr_t)b->ws_quant || (uintptr_t)b->ws_quant + b->ws_quant_bytes <= y);
        if (apart && infer_1x1_applies(a)) return launch_infer_1x1(a, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
    }
    if (search) {
        s = int8t_dsgc_search(b->dy, n_y, b->ratios, b->n_cand, INT8T_ROUND_STOCHASTIC, seed, b->clip, b->dev_search, b->dev_all, b->ws_dy,
                              b->ws_dy_bytes, stream);
        if (s != INT8T_OK) return s;
    }
    if (dw_fused) {
        DwFused f{};
        f.N = desc->N; f.C = desc->C; f.H = desc->H; f.W = desc->W;
        f.xq = b->xq; f.wq = b->wq; f.gq = b->dyq;
        f.sx = b->sx; f.sw = b->sw; f.sg = b->sdy;
        if (dw_x) {
            size_t nx = 0, nw = 0;
            (void)dims_ok(xd, &nx);
            (void)dims_ok(wd, &nw);
            f.x = b->x; f.w = b->w; f.y = b->y; f.y_acc = b->y_acc;
            f.part_x = batch_partials(b->ws_quant, 0); f.np_x = absmax_blocks(nx);
            f.part_w = batch_partials(b->ws_quant, 1); f.np_w = absmax_blocks(nw);
        }
        DwArgs w = dw_wgrad_args(desc, g);
        if (dw_g) {
            f.g = b->dy; f.clip = b->clip; f.dx = b->dx; f.dx_acc = b->dx_acc;
            f.key_x = seed_key_x(seed); f.key_a = seed_key_a(seed);
            f.partial = w.partial = (int32_t*)b->ws_bwd_weight;
            w.sa = b->sx; w.sb = b->sdy; w.out = b->dw; w.acc = b->dw_acc;
        }
        hipError_t e = hipSuccess;
        if (launch_dw_fused(f, w, st, &e)) return e == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
    }
    if (quant_xw) {
        s = batch_codes(g_in_batch ? 3 : 2, it, b->ws_quant, st, s2d);
        if (s != INT8T_OK) return s;
    }
    if (quant_g && !g_in_batch) {
        s = int8t_quantize(b->dy, ydims, ak, b->clip, INT8T_ROUND_STOCHASTIC, seed, b->dyq, b->sdy, b->dev_final, b->ws_dy, b->ws_dy_bytes, stream);
        if (s != INT8T_OK) return s;
    }
    const bool together = bwd_data && bwd_weight && disjoint_results(desc, g, b, fwd);
    bool fwd_left = fwd;
    if (together && g.depthwise) {
        DwArgs f = dw_args(desc, g, false), d = dw_args(desc, g, true), w = dw_wgrad_args(desc, g);
        f.a = b->xq; f.b = b->wq; f.sa = b->sx; f.sb = b->sw; f.out = b->y; f.acc = b->y_acc;
        d.a = b->dyq; d.b = b->wq; d.sa = b->sdy; d.sb = b->sw; d.out = b->dx; d.acc = b->dx_acc;
        w.a = b->xq; w.b = b->dyq; w.sa = b->sx; w.sb = b->sdy; w.out = b->dw; w.acc = b->dw_acc;
        w.partial = (int32_t*)b->ws_bwd_weight;
        hipError_t e = hipSuccess;
        if (launch_dw_trio(fwd ? &f : nullptr, d, w, st, &e)) return e == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
    } else if (together && !g.depthwise) {
        DensePasses p;
        dense_passes(&p, desc, g, b->ws_fwd, b->ws_fwd ? b->ws_fwd_bytes : 0, b->ws_bwd_data, b->ws_bwd_data ? b->ws_bwd_data_bytes : 0);
        IgemmArgs &f = p.f, &d = p.d;
        WgradArgs& w = p.w;
        f.act = b->xq; f.wgt = b->wq; f.sa = b->sx; f.sb = b->sw; f.out = b->y; f.acc = b->y_acc;
        d.act = b->dyq; d.wgt = b->wq + align256((size_t)desc->K * desc->R * desc->S * pad16(desc->C));
        d.sa = b->sdy; d.sb = b->sw; d.out = b->dx; d.acc = b->dx_acc;
        w.x = b->xq; w.dy = b->dyq; w.sa = b->sx; w.sb = b->sdy; w.dw = b->dw; w.acc = b->dw_acc;
        w.partial = (int32_t*)b->ws_bwd_weight;
        w.direct = wgrad_single_share(w);        // (disjoint_results)
        if (desc->stride_h != 1 || desc->stride_w != 1) {
            if (conv_trio_strided(fwd ? &f : nullptr, d, w))
                return launch_conv_trio_strided(fwd ? &f : nullptr, d, w, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
        } else {
            if (fwd && conv_trio_fwd_apart(f, d)) {
                if (launch_igemm(f, st) != hipSuccess) return INT8T_ERR_RUNTIME;
                fwd_left = false;
            }
            const IgemmArgs* fp = fwd_left ? &f : nullptr;
            const TrioTile tile = conv_trio_tile(fp, d, w);
            if (tile.bn) return launch_conv_trio(fp, d, w, tile, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
            if (const int passes = conv_band_trio(fp, d, w)) {
                if (fp && passes == 2) {
                    if (launch_igemm(f, st) != hipSuccess) return INT8T_ERR_RUNTIME;
                    fp = nullptr;
                }
                return launch_conv_band_trio(fp, d, w, st) == hipSuccess ? INT8T_OK : INT8T_ERR_RUNTIME;
            }
        }
    }
    if (fwd_left) {
        s = conv_fwd(desc, b->xq, b->sx, b->wq, b->sw, b->y, b->y_acc, b->ws_fwd, b->ws_fwd_bytes, s2d != nullptr, stream);
        if (s != INT8T_OK) return s;
    }
    if (bwd_data) {
        s = int8t_conv_bwd_data(desc, b->dyq, b->sdy, b->wq, b->sw, b->dx, b->dx_acc, b->ws_bwd_data, b->ws_bwd_data_bytes, stream);
        if (s != INT8T_OK) return s;
    }
    if (bwd_weight) {
        const bool kept = fwd && fwd_scratch_kept(desc, g, b, bwd_data);
        return int8t_conv_bwd_weight_fwd(desc, b->xq, b->sx, b->dyq, b->sdy, b->dw, b->dw_acc, b->ws_bwd_weight, b->ws_bwd_weight_bytes,
                                         kept ? b->ws_fwd : nullptr, kept ? b->ws_fwd_bytes : 0, stream);
    }
    return INT8T_OK;
}

int8t_status int8t_layer_step(const int8t_conv_desc* desc, const int8t_layer_buffers* b, int parts, uint64_t seed, void* stream) {
    return layer_step(desc, b, parts, seed, StepForm::kStep, nullptr, stream);
}

int8t_status int8t_layer_backward(const int8t_conv_desc* desc, const int8t_layer_buffers* b, int parts, uint64_t seed, float* db_dev,
                                  void* stream) {
    return layer_step(desc, b, parts, seed, StepForm::kBackward, db_dev, stream);
}

int8t_status int8t_layer_infer(const int8t_conv_desc* desc, const int8t_layer_buffers* b, void* stream) {
    return layer_step(desc, b, INT8T_STEP_ABSMAX | INT8T_STEP_QUANT_XW | INT8T_STEP_FWD, 0, StepForm::kInfer, nullptr, stream);
}

double int8t_dclr_scale(double d_c, double alpha, double beta) {
    const double e = exp(-alpha * d_c);
    return e > beta ? e : beta;
}

}  // extern "C"
