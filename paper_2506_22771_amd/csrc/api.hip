// C-ABI entry points of libffint8: argument validation on the host, then kernel launches on the
// caller's stream.  Nothing here allocates device memory or synchronises.
#include <string.h>

#include <mutex>

#include "ff_internal.hpp"

namespace ffi {

constexpr int64_t INT32_SAFE_LEN = 2147483647ll / (127 * 127);  // longest reduction that cannot overflow int32
constexpr int MAX_LAYERS = 32;
constexpr int MAX_LANES = 3;   // streams that run the update chains of different layers side by side
constexpr int MAX_CHUNKS = 2;  // weight-gradient accumulators per pass (k_update combines at most 4 terms)

// Shapes of one layer as the kernels see them.
struct Dims {
    int kind;
    int64_t B, M, K, N, rps;   // M rows per pass (dense: B; conv: B*Ho*Wo), rps rows per sample
    int64_t in_rows, in_cols;  // 2-D view of the layer input: dense [B, K]; conv [B*H*W, C_in]
    bool implicit;             // conv whose forward runs as an implicit GEMM (C_in % 4 == 0, more than a handful of channels)
    bool pointwise;            // 1x1 stride-1 convolution: its patch matrix is the NHWC input itself
    ConvGeom g;                // conv only
    int n_chunks;              // weight-gradient accumulators per pass
    int64_t chunk_b;           // samples per accumulator
    int src;                   // ff_train_step: index of the layer whose output is this layer's input (-1: the net input)
    int role, skip;            // residual-block wiring (ff_layer_desc)
};

// Sizes the quantise kernels accept: fewer than 2^32 elements (32-bit element index in the random stream) and at
// most 65535 row blocks of 128 rows (grid.y).
static bool quant_shape_ok(int64_t rows, int64_t cols)
{
    return rows >= 0 && cols >= 0 && (cols == 0 || rows < (int64_t(1) << 32) / cols) && (rows + 127) / 128 <= 65535;
}

static ff_status layer_dims(const ff_layer_desc* L, Dims* d)
{
    if (!L) return FF_ERR_INVALID_ARG;
    if (L->batch < 0) return FF_ERR_INVALID_ARG;
    memset(d, 0, sizeof(*d));
    d->kind = L->kind;
    d->B = L->batch;
    if (L->kind == FF_DENSE) {
        if (L->in_features <= 0 || L->out_features <= 0) return FF_ERR_SHAPE;
        d->M = L->batch;
        d->K = L->in_features;
        d->N = L->out_features;
        d->rps = 1;
        d->in_rows = L->batch;
        d->in_cols = L->in_features;
    } else if (L->kind == FF_CONV2D || L->kind == FF_DWCONV2D) {
        if (L->H <= 0 || L->W <= 0 || L->C_in <= 0 || L->C_out <= 0) return FF_ERR_SHAPE;
        if (L->kind == FF_DWCONV2D && (L->C_in != L->C_out || L->ksize != 3)) return FF_ERR_SHAPE;
        if ((L->ksize != 1 && L->ksize != 3) || (L->stride != 1 && L->stride != 2) || L->pad != L->ksize / 2)
            return FF_ERR_SHAPE;
        ConvGeom& g = d->g;
        g.H = L->H;
        g.W = L->W;
        g.Cin = L->C_in;
        g.cpitch = (int32_t)pitch8(L->C_in);
        g.ks = L->ksize;
        g.stride = L->stride;
        g.pad = L->pad;
        g.Ho = (L->H + 2 * L->pad - L->ksize) / L->stride + 1;
        g.Wo = (L->W + 2 * L->pad - L->ksize) / L->stride + 1;
        d->rps = (int64_t)g.Ho * g.Wo;
        d->M = d->B * d->rps;
        d->K = L->kind == FF_DWCONV2D ? (int64_t)L->ksize * L->ksize : (int64_t)L->ksize * L->ksize * L->C_in;
        d->N = L->C_out;
        d->in_rows = d->B * L->H * L->W;
        d->in_cols = L->C_in;
        d->implicit = L->kind == FF_CONV2D && (L->C_in & 3) == 0 && L->C_in > 4;
        d->pointwise = L->kind == FF_CONV2D && L->ksize == 1 && L->stride == 1;
        if (d->in_rows * g.cpitch >= (int64_t(1) << 31) || d->M >= (int64_t(1) << 31)) return FF_ERR_UNSUPPORTED;
    } else {
        return FF_ERR_INVALID_ARG;
    }
    // Launch limits of the kernels behind this layer, checked here so that an unsupported size is reported before
    // anything has been enqueued: the quantisers index elements with 32 bits and put 128 rows per workgroup on
    // grid.y; the depthwise forward kernel one sample.  (65535 output features is a limit of the interface; the update, which
    // once put a weight row on grid.y, walks the matrix flat and no longer needs it.)
    if (!quant_shape_ok(d->in_rows, d->in_cols) || !quant_shape_ok(d->M, d->N) || !quant_shape_ok(d->N, d->K) ||
        d->N > 65535 || (L->kind == FF_DWCONV2D && d->B > 65535))
        return FF_ERR_UNSUPPORTED;
    // Weight-gradient reduction: one accumulator if M * 127^2 fits int32, otherwise equal blocks of `per`
    // samples, per = the largest power of two with per * rps <= 133144.
    if (d->M <= INT32_SAFE_LEN) {
        d->n_chunks = 1;
        d->chunk_b = d->B;
    } else {
        int64_t per = 1;
        if (d->rps > INT32_SAFE_LEN) return FF_ERR_OVERFLOW_BOUND;
        while (per * 2 * d->rps <= INT32_SAFE_LEN) per *= 2;
        d->chunk_b = per;
        d->n_chunks = (int)((d->B + per - 1) / per);
        if ((per * d->rps) & 15) return FF_ERR_UNSUPPORTED;  // chunk starts must fall on 16-byte boundaries
    }
    return FF_OK;
}

static bool aligned16(const void* p) { return (((uintptr_t)p) & 15) == 0; }
static bool aligned4(const void* p) { return (((uintptr_t)p) & 3) == 0; }
#define HIPCHK(e) do { if ((e) != hipSuccess) return FF_ERR_HIP; } while (0)
// launch bracketed by timing events of kernel class `cls` on the stream `s` of the enclosing function
#define HIPCHK_T(cls, e) do { hipError_t _err; { Timed _t((cls), s); _err = (e); } if (_err != hipSuccess) return FF_ERR_HIP; } while (0)

static int32_t goodness_shift(int64_t K, int64_t terms)
{
    const unsigned __int128 a = (unsigned __int128)16129u * (unsigned __int128)K;
    const unsigned __int128 bound = a * a * (unsigned __int128)terms;
    int r = 0;
    while ((bound >> r) >> 64) ++r;
    return r;
}

// Scratch the single-operation entry points ask their callers for per pass beyond FF_WS_MIN_BYTES
// (ff_layer_workspace_bytes): a size of the interface, at least what the routes below use and for convolutions a good deal
// more.  `col`: room for a row-major patch matrix [M, pitch(K)], and for a transposed one of a weight-gradient chunk, which no
// route writes any more.  `part`: partial accumulators of a split weight-gradient reduction.
static size_t layer_col_bytes(const Dims& d)
{
    if (d.kind != FF_CONV2D) return 0;   // dense and depthwise layers need no patch matrix
    const size_t fwd = (d.g.Cin & 15) == 0 || d.pointwise ? 0 : (size_t)(d.M * pitch8(d.K));
    const size_t bwd = (size_t)(d.K * pitch8(d.chunk_b * d.rps));
    return align_up(fwd > bwd ? fwd : bwd, 256);
}
static size_t layer_part_bytes(const Dims& d, int nb)
{
    if (d.kind == FF_DWCONV2D) return 0;
    const int splits = gemm_plan(d.N, d.K, min(d.M, d.chunk_b * d.rps), nb, true, false).most_splits;
    if (splits <= 1) return 0;
    return align_up((size_t)splits * (size_t)(d.N * pitch32(d.K)) * sizeof(int32_t), 256);
}
// Convolutions whose forward pass materialises the row-major patch matrix (1x1 stride-1 ones never do).
static bool explicit_patches(const Dims& d) { return d.kind == FF_CONV2D && !d.implicit && !d.pointwise; }
// ... and whose weight gradient reads it again, reduction-major: up to four channels, where the NHWC input is mostly pad
// channels (9 * 16 columns for 27).  Other layers' weight gradients read the NHWC input itself.
static bool wgrad_from_patches(const Dims& d) { return explicit_patches(d) && d.g.Cin <= 4; }
// Columns of the weight-gradient contraction: operands read reduction-major are worked on in whole 16-byte chunks
// (GemmArgs::conv == 2).
static int64_t wgrad_cols(const Dims& d)
{
    if (d.kind != FF_CONV2D) return d.K;
    if (wgrad_from_patches(d)) return (d.K + 15) & ~int64_t(15);
    return (int64_t)d.g.ks * d.g.ks * ((d.g.Cin + 15) & ~15);
}
// Sample chunks of equal size go into one launch as further problems of the batch.
static bool chunks_together(const Dims& d) { return d.n_chunks > 1 && d.B == d.n_chunks * d.chunk_b; }
// Splits of a weight gradient's reduction of R rows, nb problems in a launch; *window: the launch reads its input through windows (wgrad3.hip).
static int wgrad_splits(const Dims& d, int64_t R, int nb, bool* window)
{
    const int w3 = d.kind == FF_CONV2D && !wgrad_from_patches(d) ? wgrad3_splits(d.g, d.N, R, nb) : 0;
    *window = w3 > 0;
    return w3 > 0 ? w3 : gemm_plan(d.N, wgrad_cols(d), R, nb, true, d.kind != FF_DENSE).splits;
}
// Scratch for the partial results of a split weight gradient: [launch][pass][chunk of the launch][split][N, pitch32(K)].
static size_t wgrad_part_bytes(const Dims& d, int nb)
{
    if (d.kind == FF_DWCONV2D)
        return align_up((size_t)(nb * d.n_chunks) * (size_t)dwconv_wgrad_splits(d.g, d.chunk_b, nb * d.n_chunks) *
                            (size_t)(d.N * pitch32(d.K)) * sizeof(int32_t), 256);
    const int problems = nb * (chunks_together(d) ? d.n_chunks : 1);
    const int64_t chunk_rows = min(d.M, d.chunk_b * d.rps), last_rows = d.M - (d.n_chunks - 1) * chunk_rows;
    int splits = 1;   // (the last chunk of a pass may be shorter and cut into other tiles)
    bool window;
    for (const int64_t rows : {chunk_rows, last_rows}) splits = max(splits, wgrad_splits(d, rows, problems, &window));
    if (splits <= 1) return 0;
    return align_up((size_t)(nb * d.n_chunks) * (size_t)splits * (size_t)(d.N * pitch32(d.K)) * sizeof(int32_t), 256);
}
static size_t layer_scratch_bytes(const Dims& d) { return layer_col_bytes(d) + layer_part_bytes(d, 1); }

// ---- workspace of ff_train_step ------------------------------------------------------------------
struct WsLayout {
    int k;
    int64_t B;
    Dims d[MAX_LAYERS];
    // byte offsets
    size_t off_slots;      // uint32: out_amax[k+1][2] (slot 0: the net input, slot j+1: output of layer j),
                           // g_amax[k][2], w_amax[k] (single-launch step)
    size_t off_gsum;       // uint64 [k][2][B]
    size_t off_vmax;       // int32  [k][2][B]
    size_t off_gl;         // scratch of the goodness / loss kernel (see GoodnessArgs::loss_part)
    size_t zero_bytes;     // the region [0, zero_bytes) is cleared at the start of a step
    size_t off_scales;     // fp32: s_a[k][2], s_g[k][2]
    // Scratch of one layer's update chain (local gradient -> weight gradient -> update -> requantise), `lanes` copies
    // `lane_stride` bytes apart: off_wbmax, off_gy, off_dw and off_part below are those of lane 0.  The chains
    // of different layers are independent of each other (layer-local learning), so a step may run them on several
    // streams at once, each with a scratch of its own.
    int lanes;
    size_t lane_stride;
    size_t off_wbmax;      // uint32 [UPDATE_MAX_BLOCKS]
    size_t off_c, off_ct;  // fp32 [k][2][B]
    size_t off_gy, st_gy;  // int8 scratch [2][st_gy]: transposed quantised local gradient
    size_t off_dw, st_dw, dw_bytes;  // int32 scratch [2][MAX_CHUNKS][dw_bytes]; st_dw = pass stride (bytes)
    // explicit patch matrices [2][st]: retained where the weight gradient reads them again (wgrad_from_patches); all other
    // layers that have one share a scratch, which only their forward contraction on the caller's stream reads
    size_t off_col[MAX_LAYERS], st_col[MAX_LAYERS];
    size_t off_part, part_bytes;     // int32 scratch: partial sums of split weight gradients (see wgrad_part_bytes)
    size_t off_xmax;                 // uint32 [2][ABSMAX_MAX_BLOCKS]: per-workgroup absmax of the net input
    size_t off_aq[MAX_LAYERS], st_aq[MAX_LAYERS];    // quantised layer input [2][st]: dense layers share one scratch
    size_t off_aqt[MAX_LAYERS], st_aqt[MAX_LAYERS];  // dense: transposed quantised input [2][st], retained
    size_t off_acc[MAX_LAYERS], st_acc[MAX_LAYERS];  // int32 accumulators [2][st] (bytes), retained
    size_t off_y[MAX_LAYERS], st_y[MAX_LAYERS];      // residual layers: fp32 block output [2][st] (bytes), retained
    // exact-derivative look-ahead only (all sizes 0 otherwise)
    int chain;
    size_t off_hf, off_gf, st_f;   // fp32 scratch [2][st_f] each: the two gradients of a layer before quantisation
    size_t off_hq, st_hq;          // int8 scratch [2][st_hq]: the gradient handed down, row-major
    size_t off_e, st_e;            // int32 scratch [2][st_e] (bytes): input-gradient accumulators
    size_t off_wqt;                // int8 scratch: transposed int8 weights of one layer
    size_t off_cmax;               // uint32 [2][2][CHAIN_MAX_BLOCKS]: per-workgroup absmax of the two gradients
    // single-launch step of a small dense stack (all sizes 0 when the stack does not qualify)
    int fused_ok;                  // the stack qualifies for the single-launch kernel
    int fused_auto;                // ... and is small enough that FF_LAUNCH_AUTO picks it
    int fused_wgs;                 // workgroups of that launch
    bool rework[MAX_LAYERS];       // the layer's accumulators are not kept: every pass that needs them contracts again (rows.hip)
    size_t off_fgy[MAX_LAYERS], st_fgy[MAX_LAYERS];   // per layer: transposed int8 local gradient [2][st]
    size_t total;
};

// Operands of a layer's forward contraction (not a depthwise one): P, Q and the shape.
static GemmArgs forward_args(const Dims& d, int relu, const int8_t* aq, int64_t st_aq, const int8_t* w_q, const int8_t* col,
                             int64_t st_col, int nb)
{
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.Q = w_q;
    g.I = (int32_t)d.M;
    g.J = (int32_t)d.N;
    g.R = (int32_t)d.K;
    g.ldq = pitch8(d.K);
    g.ldc = pitch32(d.N);
    g.rows_per_sample = (int32_t)d.rps;
    g.relu = relu;
    g.rshift = goodness_shift(d.K, d.rps * d.N);
    g.nb = nb;
    g.splits = 1;
    if (d.kind == FF_DENSE || d.pointwise) {
        // (a 1x1 stride-1 convolution: the NHWC input [B*H*W, pitch(C_in)] is its own patch matrix)
        g.P = aq;
        g.st_p = st_aq;
        g.ldp = pitch8(d.K);
    } else if (d.implicit) {
        g.P = aq;
        g.st_p = st_aq;
        g.ldp = 16;  // unused by the implicit loader
        g.conv = 1;
        g.R = d.g.ks * d.g.ks * ((d.g.Cin + 15) & ~15);
        g.H = d.g.H; g.W = d.g.W; g.Cin = (d.g.Cin + 15) & ~15; g.cin_out = d.g.Cin; g.cpitch = d.g.cpitch; g.ks = d.g.ks;
        g.stride = d.g.stride; g.pad = d.g.pad; g.Ho = d.g.Ho; g.Wo = d.g.Wo;
        g.p_bytes = d.in_rows * d.g.cpitch;
    } else {
        g.P = col;
        g.st_p = st_col;
        g.ldp = pitch8(d.K);
    }
    return g;
}

static DwArgs dw_forward_args(const Dims& d, int relu, const int8_t* aq, int64_t st_aq, const int8_t* w_q, int nb)
{
    DwArgs p;
    memset(&p, 0, sizeof(p));
    p.a = aq;
    p.st_a = st_aq;
    p.w_q = w_q;
    p.g = d.g;
    p.B = (int32_t)d.B;
    p.ldacc = pitch32(d.N);
    p.relu = relu;
    p.rshift = goodness_shift(d.K, d.rps * d.N);
    p.nb = nb;
    return p;
}

// Layers whose accumulators are worked out again by each pass that needs them instead of being stored: large depthwise ones
// (dwconv_rework_pays), and convolutions whose patch matrix exists as rows of up to ROWS_MAX_R bytes (1x1 stride-1 ones over their input,
// first layers over their patches).  Per output the stored form moves 12 bytes (written, read by the hand-off and by the
// local gradient), this one the row twice more, whose bytes are shared by the outputs it gives.  Up to four bytes of row per output
// are taken (a MobileNet-shaped step, whose 96 -> 24 layer lies on that line, 1681 -> 1635 us against a line at two).  Steps of three 1x1
// layers, the one in the middle stored and reworked, 256 images of 32x32: 32 -> 32 channels 193 and 153 us, 64 -> 16 213 and 180, 96 -> 24 236 and
// 216, 128 -> 32 260 and 246 (beyond the line: 96 -> 12 238 and 210, 128 -> 16 258 and 238).
// Rows of more than 96 bytes go through 32 KB of operands per 32 columns in every pass: into more than 64 columns they pay only once
// the stored accumulators leave the caches, at 3 x 2^23 outputs a pass: 128 -> 256 channels, 256 images of 32x32 (67 M) 676 and 598, 128 -> 512, 256 of
// 16x16 (34 M) 311 and 293, 128 -> 384 (25 M) 263 and 250; below, 128 -> 384, 256 of 14x14 (19 M) 228 and 238, 128 -> 256, 64 of 28x28 (13 M) 208
// and 226, 128 -> 512, 128 of 14x14 (13 M) 179 and 204, 128 -> 128, 256 of 14x14 (6.4 M) 153 and 161.  96 -> 384, 256 of 14x14 (19 M) 221 and 205.
// (512 columns: rows.hip stores a row of codes in whole items of 32 columns, and longer rows have a wider pitch; depthwise layers beyond were
// not measured.)
static bool rework_accumulators(const ff_net_desc* net, const WsLayout& w, int i)
{
    const Dims& d = w.d[i];
    const ff_layer_desc& L = net->layers[i];
    if (net->launch_mode == FF_LAUNCH_KERNELS) return false;   // one kernel per operation, every tensor in memory
    if (d.kind == FF_DENSE || d.role != FF_ROLE_LAYER || d.skip != FF_SKIP_NONE || L.l2norm_out || (d.N & 3) != 0 || d.N > 512) return false;
    if (d.kind == FF_CONV2D && (!(d.pointwise || wgrad_from_patches(d)) || d.K > ROWS_MAX_R || pitch8(d.K) > 4 * d.N)) return false;
    if (d.kind == FF_CONV2D && d.K > 96 && d.N > 64 && d.M * d.N < (int64_t(3) << 23)) return false;
    if (d.kind == FF_DWCONV2D && !dwconv_rework_pays(d.g, d.B)) return false;
    for (int j = i + 1; j < w.k; ++j)   // (a dense layer also takes its input transposed)
        if (w.d[j].src == i && w.d[j].kind == FF_DENSE) return false;
    return true;
}

static ff_status make_layout(const ff_net_desc* net, WsLayout* w)
{
    if (!net || !net->layers) return FF_ERR_INVALID_ARG;
    if (net->n_layers < 1 || net->n_layers > MAX_LAYERS) return FF_ERR_SHAPE;
    if (net->batch < 1) return FF_ERR_SHAPE;
    w->k = net->n_layers;
    w->B = net->batch;
    for (int i = 0; i < w->k; ++i) {
        const ff_status st = layer_dims(&net->layers[i], &w->d[i]);
        if (st != FF_OK) return st;
        const Dims& d = w->d[i];
        if (net->layers[i].batch != net->batch) return FF_ERR_SHAPE;
        if (d.K > INT32_SAFE_LEN) return FF_ERR_OVERFLOW_BOUND;
        if (d.n_chunks > MAX_CHUNKS) return FF_ERR_UNSUPPORTED;
        const ff_layer_desc& L = net->layers[i];
        Dims& dd = w->d[i];
        dd.role = L.role;
        dd.skip = L.skip;
        if (L.input_back < 0 || L.input_back > 1) return FF_ERR_UNSUPPORTED;
        if (L.role != FF_ROLE_LAYER && L.role != FF_ROLE_PROJECTION) return FF_ERR_INVALID_ARG;
        if (L.skip != FF_SKIP_NONE && L.skip != FF_SKIP_IDENTITY && L.skip != FF_SKIP_PROJECTION) return FF_ERR_INVALID_ARG;
        dd.src = i - 1 - L.input_back;
        if (dd.src < -1) return FF_ERR_SHAPE;
        if (dd.src >= 0) {
            const Dims& p = w->d[dd.src];
            if (p.role == FF_ROLE_PROJECTION) return FF_ERR_SHAPE;   // a projection has no output of its own
            if (p.kind == FF_DENSE && d.kind != FF_DENSE) return FF_ERR_UNSUPPORTED;   // no dense -> conv transition
            if (p.kind != FF_DENSE && d.kind == FF_DENSE) {
                // flatten: the NHWC output [B, H_out, W_out, C] read as [B, H_out * W_out * C]; its int32 rows must be
                // contiguous (C % 4 == 0)
                if ((p.N & 3) != 0) return FF_ERR_UNSUPPORTED;
                if (d.K != p.rps * p.N) return FF_ERR_SHAPE;
            } else if (d.kind == FF_DENSE && d.K != p.N) {
                return FF_ERR_SHAPE;
            }
            if (d.kind != FF_DENSE && (d.g.Cin != p.N || d.g.H != p.g.Ho || d.g.W != p.g.Wo)) return FF_ERR_SHAPE;
        }
        if (L.role == FF_ROLE_PROJECTION) {
            // [projection, conv1 (reads the same input), conv2 (adds the projection)]
            if (d.kind != FF_CONV2D || L.relu || L.l2norm_out || L.skip != FF_SKIP_NONE) return FF_ERR_INVALID_ARG;   // (a depthwise projection is not a case)
            if (i + 2 >= w->k || net->layers[i + 1].input_back != 1 || net->layers[i + 1].role != FF_ROLE_LAYER ||
                net->layers[i + 2].skip != FF_SKIP_PROJECTION)
                return FF_ERR_SHAPE;
        }
        if (L.skip != FF_SKIP_NONE) {
            if (d.kind != FF_CONV2D || L.role != FF_ROLE_LAYER || L.l2norm_out || (d.N & 3) || L.input_back != 0)
                return FF_ERR_UNSUPPORTED;
            if (d.B > 65535 || d.rps * (d.N >> 2) > (int64_t(1) << 28))   // launch limits of the block-output kernels
                return FF_ERR_UNSUPPORTED;
            if (L.skip == FF_SKIP_IDENTITY) {
                if (i < 1) return FF_ERR_SHAPE;
                const Dims& c1 = w->d[i - 1];   // the block input is the input of conv1
                if (c1.role != FF_ROLE_LAYER || c1.kind != FF_CONV2D || c1.g.Cin != d.N || c1.g.H != d.g.Ho ||
                    c1.g.W != d.g.Wo)
                    return FF_ERR_SHAPE;
            } else {
                if (i < 2) return FF_ERR_SHAPE;
                const Dims& pr = w->d[i - 2];
                if (pr.role != FF_ROLE_PROJECTION || pr.N != d.N || pr.g.Ho != d.g.Ho || pr.g.Wo != d.g.Wo)
                    return FF_ERR_SHAPE;
            }
        }
    }
    const size_t A = 256;
    size_t off = 0;
    const size_t k = (size_t)w->k, B = (size_t)w->B;
    w->off_slots = off;
    off = align_up(off + sizeof(uint32_t) * (k * 5 + 2), A);
    w->off_gsum = off;
    off = align_up(off + sizeof(uint64_t) * k * 2 * B, A);
    w->off_vmax = off;
    off = align_up(off + sizeof(int32_t) * k * 2 * B, A);
    w->off_gl = off;   // goodness / loss kernel with several workgroups: uint64 partial sums [2][GL_MAX_WG], uint32 counters [2]
    off = align_up(off + sizeof(uint64_t) * 2 * GL_MAX_WG + sizeof(uint32_t) * 2, A);
    w->zero_bytes = off;
    w->off_scales = off;
    off = align_up(off + sizeof(float) * (k * 4 + 4), A);   // + s_h[2], the scale of the transposed weight copy
    w->off_c = off;
    off = align_up(off + sizeof(float) * k * 2 * B, A);
    w->off_ct = off;
    off = align_up(off + sizeof(float) * k * 2 * B, A);
    size_t aq_dense = 0, gy = 0, dw = 0, part = 0, col = 0;
    for (int i = 0; i < w->k; ++i) {
        const Dims& d = w->d[i];
        if (d.kind == FF_DENSE) aq_dense = max(aq_dense, (size_t)(d.in_rows * pitch8(d.in_cols)));
        gy = max(gy, d.kind == FF_DWCONV2D ? (size_t)(d.M * pitch8(d.N)) : (size_t)(d.N * pitch8(d.M)));
        dw = max(dw, (size_t)(d.N * pitch32(d.K)) * sizeof(int32_t));
        part = max(part, wgrad_part_bytes(d, 2));
        if (explicit_patches(d) && !wgrad_from_patches(d)) col = max(col, (size_t)(d.M * pitch8(d.K)));
    }
    aq_dense = align_up(aq_dense, A);
    const size_t off_aq_dense = off;
    off += 2 * aq_dense;
    col = align_up(col, A);
    const size_t off_col_shared = off;
    off += 2 * col;
    if (net->launch_mode != FF_LAUNCH_AUTO && net->launch_mode != FF_LAUNCH_KERNELS && net->launch_mode != FF_LAUNCH_FUSED &&
        net->launch_mode != FF_LAUNCH_LANES)
        return FF_ERR_INVALID_ARG;
    // Single-launch step: plain dense stacks of at most FU_MAX_LAYERS layers and FU_MAX_B samples per pass.  It keeps
    // the local gradient of EVERY layer (the per-operation path reuses one scratch for all layers), hence the extra
    // buffers; weight gradients are applied straight from the accumulator registers.
    w->fused_ok = net->lookahead != FF_LOOKAHEAD_CHAIN && w->k <= FU_MAX_LAYERS && w->B <= FU_MAX_B;
    double macs = 0.0;
    int64_t fwd_tiles = 0, dw_tiles = 0;
    for (int i = 0; i < w->k && w->fused_ok; ++i) {
        const Dims& d = w->d[i];
        const ff_layer_desc& L = net->layers[i];
        if (d.kind != FF_DENSE || L.role != FF_ROLE_LAYER || L.skip != FF_SKIP_NONE || L.input_back != 0 || d.n_chunks != 1)
            w->fused_ok = 0;
        // (the kernel indexes with 32 bits)
        if (d.N * pitch8(d.K) > (int64_t(1) << 30) || d.K * pitch8(d.B) > (int64_t(1) << 30) || d.N * pitch8(d.B) > (int64_t(1) << 30))
            w->fused_ok = 0;
        macs += (double)d.B * (double)d.K * (double)d.N;
        fwd_tiles = max(fwd_tiles, 2 * ((d.B + 31) / 32) * ((d.N + 31) / 32));
        dw_tiles += ((d.N + 31) / 32) * ((d.K + 31) / 32);
    }
    w->fused_auto = w->fused_ok && macs <= (double)(int64_t(1) << 27);   // 41 M for 784 -> 500 -> 500 at 64 samples
    // workgroups: one per forward tile (both passes), and enough wavefronts (8 per workgroup) to take the weight-gradient
    // tiles of all layers in one round; an even number
    w->fused_wgs = (int)min((int64_t)256, max(max((int64_t)32, fwd_tiles), (dw_tiles + FU_THREADS / 64 - 1) / (FU_THREADS / 64)));
    w->fused_wgs = (w->fused_wgs + 1) & ~1;
    // Update chains on several streams: asked for (FF_LAUNCH_LANES), or chosen (FF_LAUNCH_AUTO) when the layers are small
    // enough that single launches leave compute units idle -- mean multiply-adds per layer and pass below 2^33 (three
    // lanes) or 2^36 (two).  Large dense layers fill the chip on their own and share one power budget: one lane.
    {
        double mean = 0.0;
        for (int i = 0; i < w->k; ++i) mean += (double)w->d[i].M * (double)w->d[i].K * (double)w->d[i].N;
        mean /= (double)w->k;
        int lanes = 1;
        if (net->lookahead == FF_LOOKAHEAD_COEFF && w->k >= 2) {
            if (net->launch_mode == FF_LAUNCH_LANES) lanes = MAX_LANES;
            else if (net->launch_mode == FF_LAUNCH_AUTO && !w->fused_auto)
                lanes = mean < 8589934592.0 ? MAX_LANES : (mean < 68719476736.0 ? 2 : 1);
        } else if (net->launch_mode == FF_LAUNCH_LANES) {
            return FF_ERR_UNSUPPORTED;
        }
        w->lanes = min(lanes, w->k);
    }
    w->off_xmax = off;
    off = align_up(off + sizeof(uint32_t) * 2 * ABSMAX_MAX_BLOCKS, A);
    const size_t lane0 = off;
    w->off_wbmax = off;   // per-workgroup maxima of a weight update (UpdateArgs::block_max)
    off = align_up(off + sizeof(uint32_t) * UPDATE_MAX_BLOCKS, A);
    w->st_gy = align_up(gy, A);
    w->off_gy = off;
    off += 2 * w->st_gy;
    w->dw_bytes = align_up(dw, A);
    w->st_dw = MAX_CHUNKS * w->dw_bytes;
    w->off_dw = off;
    off += 2 * w->st_dw;
    w->part_bytes = part;
    w->off_part = off;
    off += w->part_bytes;
    w->lane_stride = align_up(off - lane0, A);
    off = lane0 + (size_t)w->lanes * w->lane_stride;
    for (int i = 0; i < w->k; ++i) {
        const Dims& d = w->d[i];
        if (d.kind == FF_DENSE) {
            w->off_aq[i] = off_aq_dense;
            w->st_aq[i] = aq_dense;
            w->st_aqt[i] = align_up((size_t)(d.K * pitch8(d.M)), A);
            w->off_aqt[i] = off;
            off += 2 * w->st_aqt[i];
        } else {
            w->st_aq[i] = align_up((size_t)(d.in_rows * pitch8(d.in_cols)), A);
            w->off_aq[i] = off;
            off += 2 * w->st_aq[i];
            w->st_aqt[i] = w->off_aqt[i] = 0;
        }
        const bool keep = wgrad_from_patches(d);
        w->st_col[i] = keep ? align_up((size_t)(d.M * pitch8(d.K)), A) : (explicit_patches(d) ? col : 0);
        w->off_col[i] = keep ? off : off_col_shared;
        if (keep) off += 2 * w->st_col[i];
        w->st_acc[i] = align_up((size_t)(d.M * pitch32(d.N)) * sizeof(int32_t), A);
        w->off_acc[i] = off;
        off += 2 * w->st_acc[i];
        w->st_y[i] = d.skip != FF_SKIP_NONE ? align_up((size_t)(d.M * d.N) * sizeof(float), A) : 0;
        w->off_y[i] = off;
        off += 2 * w->st_y[i];
    }
    w->chain = net->lookahead == FF_LOOKAHEAD_CHAIN;
    w->st_f = w->st_hq = w->st_e = 0;
    w->off_hf = w->off_gf = w->off_hq = w->off_e = w->off_wqt = w->off_cmax = off;
    if (net->lookahead != FF_LOOKAHEAD_COEFF && net->lookahead != FF_LOOKAHEAD_CHAIN) return FF_ERR_INVALID_ARG;
    if (w->chain) {
        size_t f = 0, hq = 0, e = 0, wqt = 0;
        for (int i = 0; i < w->k; ++i) {
            const Dims& d = w->d[i];
            const ff_layer_desc& L = net->layers[i];
            if (d.kind != FF_DENSE || L.l2norm_out || L.role != FF_ROLE_LAYER || L.skip != FF_SKIP_NONE || L.input_back)
                return FF_ERR_UNSUPPORTED;
            if (d.N > INT32_SAFE_LEN) return FF_ERR_OVERFLOW_BOUND;   // reduction length of the input gradient
            f = max(f, (size_t)(d.M * d.N) * sizeof(float));
            if (i > 0) {
                hq = max(hq, (size_t)(d.M * pitch8(d.N)));
                e = max(e, (size_t)(d.M * pitch32(d.K)) * sizeof(int32_t));
                wqt = max(wqt, (size_t)(d.K * pitch8(d.N)));
            }
        }
        w->st_f = align_up(f, A);
        w->off_hf = off;
        off += 2 * w->st_f;
        w->off_gf = off;
        off += 2 * w->st_f;
        w->st_hq = align_up(hq, A);
        w->off_hq = off;
        off += 2 * w->st_hq;
        w->st_e = align_up(e, A);
        w->off_e = off;
        off += 2 * w->st_e;
        w->off_wqt = off;
        off += align_up(wqt, A);
        w->off_cmax = off;
        off += align_up(sizeof(uint32_t) * 4 * CHAIN_MAX_BLOCKS, A);
    }
    for (int i = 0; i < w->k; ++i) w->off_fgy[i] = w->st_fgy[i] = 0;
    if (net->launch_mode == FF_LAUNCH_FUSED && !w->fused_ok) return FF_ERR_UNSUPPORTED;
    if (w->fused_ok && (net->launch_mode == FF_LAUNCH_FUSED || (net->launch_mode == FF_LAUNCH_AUTO && w->fused_auto))) {
        for (int i = 0; i < w->k; ++i) {
            const Dims& d = w->d[i];
            w->st_fgy[i] = align_up((size_t)(d.N * pitch8(d.M)), A);
            w->off_fgy[i] = off;
            off += 2 * w->st_fgy[i];
        }
    } else {
        w->fused_auto = 0;
        if (net->launch_mode != FF_LAUNCH_FUSED) w->fused_ok = 0;
    }
    w->total = off;
    for (int i = 0; i < w->k; ++i) w->rework[i] = rework_accumulators(net, *w, i);
    return FF_OK;
}

// ---- instrumentation: HIP events around each launch, recorded on the launch stream -----------------
struct TimingState {
    uint32_t mask = 0;   // bit c set: launches of kernel class c are timed
    int n = 0;
    hipEvent_t* ev = nullptr;  // 2 per record
    int8_t* cls = nullptr;
    int created = 0;
};
static TimingState g_timing;
static unsigned long long* g_clock_probe = nullptr;   // device counters of ff_timing_clock_probe (null: off)
static unsigned long long* g_fused_stamps = nullptr;  // device buffer of ff_timing_fused_stamps (null: off)

struct Timed {
    hipStream_t s;
    int idx = -1;
    Timed(int kernel_class, hipStream_t stream) : s(stream)
    {
        TimingState& t = g_timing;
        if (!((t.mask >> kernel_class) & 1u) || t.n >= FF_TIMING_MAX_RECORDS) return;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;   // no event records into a graph under capture
        if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return;
        if (!t.ev) {
            t.ev = new hipEvent_t[2 * FF_TIMING_MAX_RECORDS];
            t.cls = new int8_t[FF_TIMING_MAX_RECORDS];
        }
        while (t.created <= t.n) {
            if (hipEventCreate(&t.ev[2 * t.created]) != hipSuccess) return;
            if (hipEventCreate(&t.ev[2 * t.created + 1]) != hipSuccess) return;
            ++t.created;
        }
        idx = t.n++;
        t.cls[idx] = (int8_t)kernel_class;
        (void)hipEventRecord(t.ev[2 * idx], s);
    }
    ~Timed()
    {
        if (idx >= 0) (void)hipEventRecord(g_timing.ev[2 * idx + 1], s);
    }
};

static Im2colArgs im2col_args(const Dims& d, const int8_t* aq, int64_t st_aq, int8_t* col, int64_t st_col, int nb)
{
    Im2colArgs ic;
    memset(&ic, 0, sizeof(ic));
    ic.a = aq;
    ic.st_a = st_aq;
    ic.out = col;
    ic.st_out = st_col;
    ic.g = d.g;
    ic.K = (int32_t)d.K;
    ic.B = (int32_t)d.B;
    ic.ld_out = pitch8(d.K);
    ic.nb = nb;
    return ic;
}

// One of the passes over a layer whose accumulators are not kept (RowsResult); q: what the codes are made of.
static hipError_t launch_rework(int what, const GemmArgs& g, const QuantArgs& q, hipStream_t s)
{
    RowsArgs r;
    memset(&r, 0, sizeof(r));
    r.P = g.P;
    r.Q = g.Q;
    r.ldp = g.ldp;
    r.ldq = g.ldq;
    r.st_p = g.st_p;
    r.I = g.I;
    r.J = g.J;
    r.R = g.R;
    r.nb = g.nb;
    r.rows_per_sample = g.rows_per_sample;
    r.relu = g.relu;
    r.rshift = g.rshift;
    r.gsum = g.gsum;
    r.vmax = g.vmax;
    r.st_g = g.st_g;
    return launch_rows(what, r, q, s);
}

// ---- the two contractions of a layer, for nb passes at once ------------------------------------------
// Forward: acc[z] = A_q[z] x W_q^T (+ per-sample sums).  `aq` is the quantised layer input (dense: [M, pitch(K)];
// conv: NHWC), `col` scratch for an explicit patch matrix (see explicit_patches).
static ff_status run_forward(const Dims& d, int relu, const int8_t* aq, int64_t st_aq, const int8_t* w_q, int32_t* acc,
                             int64_t st_acc, unsigned long long* gsum, int32_t* vmax, int64_t st_g, int8_t* col,
                             int64_t st_col, int nb, hipStream_t s, const ResidualArgs* res = nullptr)
{
    if (d.kind == FF_DWCONV2D) {
        DwArgs p = dw_forward_args(d, relu, aq, st_aq, w_q, nb);
        p.acc = acc;
        p.st_acc = st_acc;
        p.gsum = gsum;
        p.vmax = vmax;
        p.st_g = st_g;
        if (acc) HIPCHK_T(FF_K_DWCONV, launch_dwconv_forward(p, s));
        else HIPCHK_T(FF_K_DWCONV, launch_dwconv_rework(ROWS_GOODNESS, p, QuantArgs{}, s));
        return FF_OK;
    }
    GemmArgs g = forward_args(d, relu, aq, st_aq, w_q, col, st_col, nb);
    g.C = acc;
    g.st_c = st_acc;
    g.gsum = gsum;
    g.vmax = vmax;
    g.st_g = st_g;
    g.residual = res;
    if (explicit_patches(d)) HIPCHK_T(FF_K_IM2COL, launch_im2col(im2col_args(d, aq, st_aq, col, st_col, nb), s));
    if (!acc) {
        HIPCHK_T(FF_K_GEMM_FWD, launch_rework(ROWS_GOODNESS, g, QuantArgs{}, s));
        return FF_OK;
    }
    if (conv3_ok(g)) {
        HIPCHK_T(FF_K_GEMM_FWD, launch_conv3(g, s));
        return FF_OK;
    }
    if (conv3_wide_ok(g)) {
        HIPCHK_T(FF_K_GEMM_FWD, launch_conv3_wide(g, s));
        return FF_OK;
    }
    g.clk = g_clock_probe;
    HIPCHK_T(FF_K_GEMM_FWD, launch_gemm_nt_i8(g, s));
    return FF_OK;
}

// Where the accumulators of a weight gradient are: term[p][c] of pass p and sample chunk c is the sum of splits[c] partial
// results, st_split elements apart.
struct WgradTerms {
    const int32_t* term[2][MAX_CHUNKS];
    int splits[MAX_CHUNKS];
    int64_t st_split;
};

// Weight gradient: dw[z][c] = gy_q_t[z][:, chunk c] x (patches of chunk c)^T for every chunk c.
// `aqt` is the transposed quantised input (dense) or the NHWC quantised input (conv), which the contraction reads
// reduction-major as it is -- or the row-major patch matrix [M, pitch(K)] (wgrad_from_patches).  dw accumulators of one pass
// are dw_elems apart.  `part`: part_elems elements for the partial results of a split reduction.  terms == null (one pass
// only): split results are added up into dw; otherwise they are left as they are for the update, and *terms says where
// everything is.
static ff_status run_wgrad(const Dims& d, const int8_t* gy_t, int64_t st_gy, const int8_t* aqt, int64_t st_aqt,
                           int32_t* part, int64_t part_elems, int32_t* dw, int64_t st_dw, int64_t dw_elems, int nb,
                           hipStream_t s, WgradTerms* terms)
{
    const int64_t elems = d.N * pitch32(d.K);
    if (!terms && nb != 1) return FF_ERR_INVALID_ARG;
    if (terms) {
        terms->st_split = elems;
        for (int c = 0; c < d.n_chunks; ++c) {
            terms->splits[c] = 1;
            for (int z = 0; z < nb; ++z) terms->term[z][c] = dw + z * st_dw + c * dw_elems;
        }
    }
    if (d.kind == FF_DWCONV2D) {
        // gy_t holds the ROW-MAJOR int8 gradient [M, pitch(C)] for this layer kind
        DwArgs p;
        memset(&p, 0, sizeof(p));
        p.a = aqt;
        p.st_a = st_aqt;
        p.g = d.g;
        p.B = (int32_t)d.B;
        p.gy = gy_t;
        p.ldg = pitch8(d.N);
        p.st_gy = st_gy;
        p.nb = nb;
        p.nc = d.n_chunks;
        p.chunk_b = (int32_t)d.chunk_b;
        p.splits = dwconv_wgrad_splits(d.g, d.chunk_b, nb * d.n_chunks);
        if (terms && part_elems >= nb * d.n_chunks * p.splits * elems) {
            p.dw = part;
            p.st_split = elems;
            p.st_dw2 = p.splits * elems;
            p.st_dw = d.n_chunks * p.st_dw2;
            for (int c = 0; c < d.n_chunks; ++c) {
                terms->splits[c] = p.splits;
                for (int z = 0; z < nb; ++z) terms->term[z][c] = part + z * p.st_dw + c * p.st_dw2;
            }
        } else {   // accumulators that are added to with atomics start at zero
            p.dw = dw;
            p.st_dw = st_dw;
            p.st_dw2 = dw_elems;
            for (int z = 0; z < nb; ++z)
                for (int c = 0; c < d.n_chunks; ++c)
                    HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)(dw + z * st_dw + c * dw_elems), elems, 0u, s));
        }
        HIPCHK_T(FF_K_DWCONV, launch_dwconv_wgrad(p, s));
        return FF_OK;
    }
    // one launch for all chunks, or one per chunk (chunks of different sizes)
    const int together = chunks_together(d) ? d.n_chunks : 1;
    const int launches = d.n_chunks / together;
    for (int l = 0; l < launches; ++l) {
        const int64_t b0 = l * d.chunk_b, b1 = min(d.B, b0 + d.chunk_b);
        const int64_t m0 = b0 * d.rps, mc = (b1 - b0) * d.rps;
        GemmArgs g;
        memset(&g, 0, sizeof(g));
        g.P = gy_t + m0;
        g.st_p = st_gy;
        g.st_p2 = mc;
        g.ldp = pitch8(d.M);
        g.C = dw + l * dw_elems;
        g.st_c = st_dw;
        g.st_c2 = dw_elems;
        g.I = (int32_t)d.N;
        g.J = (int32_t)d.K;
        g.R = (int32_t)mc;
        g.ldc = pitch32(d.K);
        g.rows_per_sample = 1;
        g.nb = nb * together;
        g.nc = together;
        if (d.kind == FF_DENSE) {
            g.Q = aqt + m0;
            g.st_q = st_aqt;
            g.st_q2 = mc;
            g.ldq = pitch8(d.M);
        } else {
            // the operand as it lies in memory, read reduction-major: the NHWC input, or the patch matrix, which is the
            // NHWC input of a 1x1 convolution with K channels
            ConvGeom q = d.g;
            if (wgrad_from_patches(d)) {
                q.H = q.Ho;
                q.W = q.Wo;
                q.Cin = (int32_t)d.K;
                q.cpitch = (int32_t)pitch8(d.K);
                q.ks = q.stride = 1;
                q.pad = 0;
            }
            g.Q = aqt + b0 * q.H * q.W * q.cpitch;
            g.st_q = st_aqt;
            g.st_q2 = d.chunk_b * q.H * q.W * q.cpitch;
            g.ldq = 16;   // unused by this loader
            g.conv = 2;
            g.J = (int32_t)wgrad_cols(d);
            g.H = q.H; g.W = q.W; g.Cin = (q.Cin + 15) & ~15; g.cin_out = q.Cin; g.cpitch = q.cpitch; g.ks = q.ks;
            g.stride = q.stride; g.pad = q.pad; g.Ho = q.Ho; g.Wo = q.Wo;
            g.p_bytes = (b1 - b0) * q.H * q.W * q.cpitch;
        }
        bool window;
        g.splits = wgrad_splits(d, mc, g.nb, &window);
        const int64_t room = part_elems / launches;            // this launch's share of the scratch
        const int64_t fit = room / (elems * g.nb);             // partial results per accumulator it holds
        if (g.splits > fit) g.splits = window ? wgrad3_split_evenly(g.R, fit < 1 ? 1 : fit) : split_evenly(g.R, fit < 1 ? 1 : fit);
        auto contract = [&] { return window ? launch_wgrad3(g, d.g, s) : launch_gemm_nt_i8(g, s); };
        g.clk = g_clock_probe;
        if (g.splits > 1) {
            // problem (pass z, chunk c) keeps its partial results at ((z * together + c) * splits) * elems
            int32_t* const out = g.C;
            int32_t* const mine = part + l * room / 4 * 4;
            g.C = mine;
            g.st_split = elems;
            g.st_c2 = g.splits * elems;
            g.st_c = together * g.st_c2;
            HIPCHK_T(FF_K_GEMM_DW, contract());
            if (terms) {
                for (int c = 0; c < together; ++c) {
                    terms->splits[l + c] = g.splits;
                    for (int z = 0; z < nb; ++z) terms->term[z][l + c] = mine + z * g.st_c + c * g.st_c2;
                }
            } else {
                HIPCHK_T(FF_K_GEMM_DW, launch_reduce_splits(mine, g.splits, elems, g.st_c2, out, dw_elems, elems, together, s));
            }
        } else {
            HIPCHK_T(FF_K_GEMM_DW, contract());
        }
    }
    return FF_OK;
}

}  // namespace ffi

using namespace ffi;

extern "C" {

int64_t ff_pitch(int64_t cols) { return pitch8(cols); }
int64_t ff_pitch32(int64_t cols) { return pitch32(cols); }

uint64_t ff_stream_tag(uint64_t step, uint32_t layer, uint32_t pass_idx, uint32_t kind)
{
    return stream_tag_of(step, layer, pass_idx, kind);
}

const char* ff_status_string(ff_status s)
{
    switch (s) {
        case FF_OK: return "ok";
        case FF_ERR_INVALID_ARG: return "invalid argument";
        case FF_ERR_SHAPE: return "inconsistent or unsupported shape";
        case FF_ERR_ALIGN: return "buffer not aligned as required";
        case FF_ERR_WORKSPACE: return "workspace too small";
        case FF_ERR_OVERFLOW_BOUND: return "an int32 accumulator could overflow for this shape";
        case FF_ERR_UNSUPPORTED: return "not implemented in this build";
        case FF_ERR_HIP: return "HIP runtime error";
        default: return "unknown status";
    }
}

const char* ff_version(void) { return "ffint8 0.4 (gfx950)"; }

int32_t ff_goodness_shift(const ff_layer_desc* layer)
{
    Dims d;
    if (layer_dims(layer, &d) != FF_OK) return -1;
    return goodness_shift(d.K, d.rps * d.N);
}

int32_t ff_layer_dw_chunks(const ff_layer_desc* layer)
{
    Dims d;
    if (layer_dims(layer, &d) != FF_OK) return -1;
    return d.n_chunks;
}

size_t ff_layer_workspace_bytes(const ff_layer_desc* layer)
{
    Dims d;
    if (layer_dims(layer, &d) != FF_OK) return 0;
    return FF_WS_MIN_BYTES + layer_scratch_bytes(d);
}

ff_status ff_quantize(const float* x, int64_t rows, int64_t cols, int32_t round_mode, uint64_t seed,
                      uint64_t stream_tag, int8_t* q, int8_t* q_t, float* scale, void* ws, size_t ws_bytes,
                      void* stream)
{
    if (rows < 0 || cols < 0 || !scale || (!q && !q_t) || !ws) return FF_ERR_INVALID_ARG;
    if (round_mode != FF_ROUND_NEAREST_EVEN && round_mode != FF_ROUND_STOCHASTIC) return FF_ERR_INVALID_ARG;
    if (!quant_shape_ok(rows, cols)) return FF_ERR_UNSUPPORTED;
    if (ws_bytes < FF_WS_MIN_BYTES) return FF_ERR_WORKSPACE;
    if (!aligned16(ws) || (q && !aligned16(q)) || (q_t && !aligned16(q_t)) || !aligned4(scale)) return FF_ERR_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    if (rows == 0 || cols == 0) {
        const float one = 1.0f;
        uint32_t bits;
        memcpy(&bits, &one, 4);
        HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)scale, 1, bits, s));
        return FF_OK;
    }
    if (!x) return FF_ERR_INVALID_ARG;
    if (!aligned4(x)) return FF_ERR_ALIGN;
    static_assert(ABSMAX_MAX_BLOCKS * sizeof(uint32_t) <= FF_WS_MIN_BYTES, "one candidate per workgroup of the absmax");
    uint32_t* slot = (uint32_t*)ws;
    HIPCHK_T(FF_K_ABSMAX, launch_absmax(x, 0, 1, rows * cols, slot, s));
    QuantArgs a;
    memset(&a, 0, sizeof(a));
    a.x = x;
    a.amax_bits = slot;
    a.amax_n = absmax_blocks(rows * cols);
    a.round_mode = round_mode;
    a.key = make_sr_key(seed, stream_tag);
    a.rows = rows;
    a.cols = cols;
    a.q = q;
    a.ldq = pitch8(cols);
    a.q_t = q_t;
    a.ldqt = pitch8(rows);
    a.scale = scale;
    a.nb = 1;
    a.rows_per_sample = 1;
    HIPCHK_T(FF_K_QUANT_ACT, launch_quantize(QSRC_F32, a, s));
    return FF_OK;
}

ff_status ff_layer_forward(const ff_layer_desc* layer, const int8_t* a_q, const int8_t* w_q, int32_t* acc,
                           uint64_t* gsum_int, int32_t* vmax, void* ws, size_t ws_bytes, void* stream)
{
    Dims d;
    const ff_status st = layer_dims(layer, &d);
    if (st != FF_OK) return st;
    if (!a_q || !w_q || !acc || !gsum_int || !vmax) return FF_ERR_INVALID_ARG;
    if (!aligned16(a_q) || !aligned16(w_q) || !aligned16(acc) || (((uintptr_t)gsum_int) & 7) || !aligned4(vmax))
        return FF_ERR_ALIGN;
    if (d.K > INT32_SAFE_LEN) return FF_ERR_OVERFLOW_BOUND;
    const bool need_col = d.kind == FF_CONV2D && (d.g.Cin & 15) != 0;   // the layers that are asked for scratch (explicit_patches(d) use it)
    if (need_col) {
        if (!ws) return FF_ERR_INVALID_ARG;
        if (!aligned16(ws)) return FF_ERR_ALIGN;
        if (ws_bytes < FF_WS_MIN_BYTES + layer_scratch_bytes(d)) return FF_ERR_WORKSPACE;
    }
    hipStream_t s = (hipStream_t)stream;
    if (d.B == 0) return FF_OK;
    HIPCHK_T(FF_K_SMALL, launch_clear2_u32((uint32_t*)gsum_int, 2 * d.B, (uint32_t*)vmax, d.B, s));
    int8_t* col = need_col ? (int8_t*)ws + FF_WS_MIN_BYTES : nullptr;
    return run_forward(d, layer->relu ? 1 : 0, a_q, 0, w_q, acc, 0, (unsigned long long*)gsum_int, vmax, 0, col, 0, 1, s);
}

ff_status ff_goodness_loss(const ff_layer_desc* layer, const uint64_t* gsum_int, const int32_t* vmax,
                           const float* s_a, const float* s_w, int32_t pass_sign, float theta, float* goodness,
                           float* coeff, float* loss_mean, float* next_amax, void* stream)
{
    Dims d;
    const ff_status st = layer_dims(layer, &d);
    if (st != FF_OK) return st;
    if (!gsum_int || !vmax || !s_a || !s_w || !goodness || !coeff || !loss_mean) return FF_ERR_INVALID_ARG;
    if (pass_sign != FF_PASS_POS && pass_sign != FF_PASS_NEG) return FF_ERR_INVALID_ARG;
    if ((((uintptr_t)gsum_int) & 7) || !aligned4(vmax) || !aligned4(goodness) || !aligned4(coeff)) return FF_ERR_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    GoodnessArgs a;
    memset(&a, 0, sizeof(a));
    a.gsum = (const unsigned long long*)gsum_int;
    a.vmax = vmax;
    a.s_a = s_a;
    a.s_w = s_w;
    a.rshift = goodness_shift(d.K, d.rps * d.N);
    a.l2norm = layer->l2norm_out ? 1 : 0;
    a.pass_sign = pass_sign;
    a.theta = theta;
    a.B = d.B;
    a.goodness = goodness;
    a.coeff = coeff;
    a.loss_mean = loss_mean;
    a.next_amax_bits = (uint32_t*)next_amax;
    a.nb = 1;
    HIPCHK_T(FF_K_SMALL, launch_goodness_loss(a, s));
    return FF_OK;
}

ff_status ff_layer_handoff(const ff_layer_desc* layer, const int32_t* acc, const float* s_a, const float* s_w,
                           const float* goodness, const float* amax, int32_t round_mode, uint64_t seed,
                           uint64_t stream_tag, int8_t* q, int8_t* q_t, float* scale, void* stream)
{
    Dims d;
    const ff_status st = layer_dims(layer, &d);
    if (st != FF_OK) return st;
    if (!acc || !s_a || !s_w || !amax || !scale || (!q && !q_t)) return FF_ERR_INVALID_ARG;
    if (layer->l2norm_out && !goodness) return FF_ERR_INVALID_ARG;
    if (round_mode != FF_ROUND_NEAREST_EVEN && round_mode != FF_ROUND_STOCHASTIC) return FF_ERR_INVALID_ARG;
    if (!aligned16(acc) || (q && !aligned16(q)) || (q_t && !aligned16(q_t))) return FF_ERR_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    if (d.M == 0) {   // empty batch: no codes; the scale of an empty tensor is 1, as in ff_quantize
        HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)scale, 1, 0x3F800000u, s));
        return FF_OK;
    }
    QuantArgs a;
    memset(&a, 0, sizeof(a));
    a.acc = acc;
    a.ldacc = pitch32(d.N);
    a.s_a = s_a;
    a.s_w = s_w;
    a.per_sample = goodness;
    a.rows_per_sample = (int32_t)d.rps;
    a.relu = layer->relu ? 1 : 0;
    a.l2norm = layer->l2norm_out ? 1 : 0;
    a.amax_bits = (const uint32_t*)amax;
    a.round_mode = round_mode;
    a.key = make_sr_key(seed, stream_tag);
    a.rows = d.M;
    a.cols = d.N;
    a.q = q;
    a.ldq = pitch8(d.N);
    a.q_t = q_t;
    a.ldqt = pitch8(d.M);
    a.scale = scale;
    a.nb = 1;
    HIPCHK_T(FF_K_QUANT_ACT, launch_quantize(QSRC_HANDOFF, a, s));
    return FF_OK;
}

ff_status ff_lookahead(const float* coeff, int32_t n_layers, int64_t batch, float lambda, float* coeff_total,
                       void* stream)
{
    if (!coeff || !coeff_total || batch < 0) return FF_ERR_INVALID_ARG;
    if (n_layers < 1 || n_layers > MAX_LAYERS) return FF_ERR_SHAPE;
    if (batch == 0) return FF_OK;
    hipStream_t s = (hipStream_t)stream;
    LookaheadArgs a;
    memset(&a, 0, sizeof(a));
    a.coeff = coeff;
    a.coeff_total = coeff_total;
    a.k = n_layers;
    a.np = 1;
    a.B = batch;
    a.st_layer = batch;
    a.st_pass = 0;
    a.lambda = lambda;
    HIPCHK_T(FF_K_SMALL, launch_lookahead(a, s));
    return FF_OK;
}

ff_status ff_layer_backward_local(const ff_layer_desc* layer, const int32_t* acc, const int32_t* vmax,
                                  const float* s_a, const float* s_w, const float* coeff_total, int32_t round_mode,
                                  uint64_t seed, uint64_t stream_tag, const int8_t* a_q_t, int8_t* gy_q_t,
                                  float* s_g, int32_t* dw_acc, void* ws, size_t ws_bytes, void* stream)
{
    Dims d;
    const ff_status st = layer_dims(layer, &d);
    if (st != FF_OK) return st;
    if (!acc || !vmax || !s_a || !s_w || !coeff_total || !a_q_t || !gy_q_t || !s_g || !dw_acc || !ws)
        return FF_ERR_INVALID_ARG;
    if (round_mode != FF_ROUND_NEAREST_EVEN && round_mode != FF_ROUND_STOCHASTIC) return FF_ERR_INVALID_ARG;
    if (ws_bytes < FF_WS_MIN_BYTES + layer_scratch_bytes(d)) return FF_ERR_WORKSPACE;
    if (!aligned16(acc) || !aligned16(a_q_t) || !aligned16(gy_q_t) || !aligned16(dw_acc) || !aligned16(ws))
        return FF_ERR_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    if (d.B == 0) {   // empty batch: scale 1 (as for any empty tensor) and an all-zero weight gradient
        HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)s_g, 1, 0x3F800000u, s));
        HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)dw_acc, d.N * pitch32(d.K), 0u, s));
        return FF_OK;
    }
    uint32_t* slot = (uint32_t*)ws;
    QuantArgs a;
    memset(&a, 0, sizeof(a));
    // Range of the gradient: by the quantiser's workgroups themselves, or by a launch before it for batches of which each would read a
    // good part again (as for the hand-off).  Backward with the launch and without: 2000 -> 2000 features, 2048 samples 70.0 and 68.2
    // us, 3072 82.7 and 83.3, 8192 163 and 171; 64 -> 128 channels on 256 images of 32x32 167 and 160.  (Narrow layers gain beyond the line
    // too: 500 -> 500, 4096 samples 79.6 and 77.2.)
    if (d.B <= 2048) {
        a.vmax = vmax;
        a.B = (int32_t)d.B;
    } else {
        HIPCHK_T(FF_K_SMALL, launch_grad_amax(coeff_total, vmax, s_a, s_w, d.B, 1, slot, s));
    }
    a.acc = acc;
    a.ldacc = pitch32(d.N);
    a.s_a = s_a;
    a.s_w = s_w;
    a.per_sample = coeff_total;
    a.rows_per_sample = (int32_t)d.rps;
    a.relu = layer->relu ? 1 : 0;
    a.amax_bits = slot;
    a.round_mode = round_mode;
    a.key = make_sr_key(seed, stream_tag);
    a.rows = d.M;
    a.cols = d.N;
    if (d.kind == FF_DWCONV2D) {   // the depthwise weight gradient reads the gradient row-major
        a.q = gy_q_t;
        a.ldq = pitch8(d.N);
    } else {
        a.q_t = gy_q_t;
        a.ldqt = pitch8(d.M);
    }
    a.scale = s_g;
    a.nb = 1;
    HIPCHK_T(FF_K_QUANT_GRAD, launch_quantize(QSRC_GRAD, a, s));
    const int64_t dw_elems = d.N * pitch32(d.K);
    // scratch: [row-major patch matrix (wgrad_from_patches) | partial sums of a split reduction]
    char* scratch = (char*)ws + FF_WS_MIN_BYTES;
    size_t room = layer_scratch_bytes(d);
    const int8_t* operand = a_q_t;
    if (wgrad_from_patches(d)) {
        Im2colArgs ic = im2col_args(d, a_q_t, 0, (int8_t*)scratch, 0, 1);
        HIPCHK_T(FF_K_IM2COL, launch_im2col(ic, s));
        operand = (const int8_t*)scratch;
        scratch += layer_col_bytes(d);
        room -= layer_col_bytes(d);
    }
    return run_wgrad(d, gy_q_t, 0, operand, 0, (int32_t*)scratch, (int64_t)(room / sizeof(int32_t)), dw_acc, 0, dw_elems, 1, s,
                     nullptr);
}

// ---- the entry point that allocates nothing: its scratch is a fixed array in the library's own device image ----
// Each GPU holds its own copy of the array at its own address; in host code the array's name is only a handle for
// hipGetSymbolAddress, never a device address.  The address is looked up once per device (with that device current)
// and kept; launches and kernels only ever see that pointer.
static __device__ __align__(256) unsigned char scratch[FF_NOALLOC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static void* g_scratch_ptr[MAX_DEVICES];
static std::mutex g_scratch_mutex;

static ff_status scratch_of_current_device(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return FF_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return FF_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return FF_OK;
}

size_t ff_noalloc_scratch_bytes(void) { return FF_NOALLOC_SCRATCH_BYTES; }

ff_status ff_layer_backward_local_noalloc(const ff_layer_desc* layer, const int32_t* acc, const int32_t* vmax,
                                          const float* s_a, const float* s_w, const float* coeff_total,
                                          int32_t round_mode, uint64_t seed, uint64_t stream_tag, const int8_t* a_q_t,
                                          int8_t* gy_q_t, float* s_g, int32_t* dw_acc, void* stream)
{
    Dims d;
    const ff_status st = layer_dims(layer, &d);
    if (st != FF_OK) return st;
    // the layer's patch matrix and split partial sums must fit the fixed array
    if (FF_WS_MIN_BYTES + layer_scratch_bytes(d) > FF_NOALLOC_SCRATCH_BYTES) return FF_ERR_WORKSPACE;
    void* ws = nullptr;
    const ff_status ss = scratch_of_current_device(&ws);
    if (ss != FF_OK) return ss;
    // Nothing in the array has to start at zero: the absmax slot is stored (not accumulated into), the patch matrix
    // is written whole (pad bytes included) before the contraction reads it, and every split stores its own partial
    // sums before they are added up.
    return ff_layer_backward_local(layer, acc, vmax, s_a, s_w, coeff_total, round_mode, seed, stream_tag, a_q_t,
                                   gy_q_t, s_g, dw_acc, ws, FF_NOALLOC_SCRATCH_BYTES, stream);
}

ff_status ff_chain_gradients(const ff_layer_desc* layer, const int32_t* acc, const float* s_a, const float* s_w,
                             const float* coeff, const int32_t* e_acc, const float* s_h, const float* s_w_up,
                             float lambda, float* h, float* g, float* h_amax, float* g_amax, void* stream)
{
    Dims d;
    const ff_status st = layer_dims(layer, &d);
    if (st != FF_OK) return st;
    if (d.kind != FF_DENSE) return FF_ERR_UNSUPPORTED;
    if (!acc || !s_a || !s_w || !coeff || !g || !g_amax) return FF_ERR_INVALID_ARG;
    if (e_acc && (!s_h || !s_w_up)) return FF_ERR_INVALID_ARG;
    if ((h == nullptr) != (h_amax == nullptr)) return FF_ERR_INVALID_ARG;
    if (!aligned16(acc) || (e_acc && !aligned16(e_acc)) || !aligned4(g) || (h && !aligned4(h)) || !aligned4(g_amax) ||
        (h_amax && !aligned4(h_amax)))
        return FF_ERR_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)g_amax, 1, 0u, s));
    if (h_amax) HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)h_amax, 1, 0u, s));
    ChainArgs ca;
    memset(&ca, 0, sizeof(ca));
    ca.acc = acc;
    ca.ldacc = pitch32(d.N);
    ca.s_a = s_a;
    ca.s_w = s_w;
    ca.coeff = coeff;
    ca.e_acc = e_acc;
    ca.lde = pitch32(d.N);
    ca.s_h = s_h;
    ca.s_w_up = s_w_up;
    ca.lambda = lambda;
    ca.relu = layer->relu ? 1 : 0;
    ca.M = d.M;
    ca.N = d.N;
    ca.h = h;
    ca.g = g;
    ca.h_amax_bits = (uint32_t*)h_amax;   // the bit pattern of a non-negative fp32 is the value itself
    ca.g_amax_bits = (uint32_t*)g_amax;
    ca.amax_atomic = 1;
    ca.nb = 1;
    HIPCHK_T(FF_K_CHAIN, launch_chain_combine(ca, s));
    return FF_OK;
}

ff_status ff_layer_input_grad(const ff_layer_desc* layer, const int8_t* h_q, const int8_t* w_q_t, int32_t* e_acc,
                              void* ws, size_t ws_bytes, void* stream)
{
    Dims d;
    const ff_status st = layer_dims(layer, &d);
    if (st != FF_OK) return st;
    if (d.kind != FF_DENSE) return FF_ERR_UNSUPPORTED;
    if (!h_q || !w_q_t || !e_acc || !ws) return FF_ERR_INVALID_ARG;
    if (ws_bytes < FF_WS_MIN_BYTES) return FF_ERR_WORKSPACE;
    if (!aligned16(h_q) || !aligned16(w_q_t) || !aligned16(e_acc)) return FF_ERR_ALIGN;
    if (d.N > INT32_SAFE_LEN) return FF_ERR_OVERFLOW_BOUND;
    hipStream_t s = (hipStream_t)stream;
    GemmArgs ga;
    memset(&ga, 0, sizeof(ga));
    ga.P = h_q;
    ga.Q = w_q_t;
    ga.C = e_acc;
    ga.I = (int32_t)d.M;
    ga.J = (int32_t)d.K;
    ga.R = (int32_t)d.N;
    ga.ldp = pitch8(d.N);
    ga.ldq = pitch8(d.N);
    ga.ldc = pitch32(d.K);
    ga.nb = 1;
    ga.splits = 1;
    HIPCHK_T(FF_K_CHAIN, launch_gemm_nt_i8(ga, s));
    return FF_OK;
}

ff_status ff_layer_update(const ff_layer_desc* layer, float* w_master, const int32_t* dw_acc_pos,
                          const float* s_g_pos, const float* s_a_pos, const int32_t* dw_acc_neg,
                          const float* s_g_neg, const float* s_a_neg, float lr, int32_t total_samples,
                          int8_t* w_q, float* s_w, void* ws, size_t ws_bytes, void* stream)
{
    Dims d;
    const ff_status st = layer_dims(layer, &d);
    if (st != FF_OK) return st;
    if (!w_master || !dw_acc_pos || !s_g_pos || !s_a_pos || !dw_acc_neg || !s_g_neg || !s_a_neg || !w_q || !s_w || !ws)
        return FF_ERR_INVALID_ARG;
    if (total_samples < 1) return FF_ERR_INVALID_ARG;
    if (ws_bytes < FF_WS_MIN_BYTES) return FF_ERR_WORKSPACE;
    if (!aligned4(w_master) || !aligned16(dw_acc_pos) || !aligned16(dw_acc_neg) || !aligned16(w_q) || !aligned16(ws))
        return FF_ERR_ALIGN;
    if (d.n_chunks > MAX_CHUNKS) return FF_ERR_UNSUPPORTED;
    hipStream_t s = (hipStream_t)stream;
    uint32_t* slot = (uint32_t*)ws;
    const int64_t dw_elems = d.N * pitch32(d.K);
    UpdateArgs u;
    memset(&u, 0, sizeof(u));
    u.w = w_master;
    u.N = d.N;
    u.K = d.K;
    u.lddw = pitch32(d.K);
    u.n_terms = 2 * d.n_chunks;
    for (int c = 0; c < d.n_chunks; ++c) {
        u.dw[c] = dw_acc_pos + c * dw_elems;
        u.s_g[c] = s_g_pos;
        u.s_a[c] = s_a_pos;
        u.dw[d.n_chunks + c] = dw_acc_neg + c * dw_elems;
        u.s_g[d.n_chunks + c] = s_g_neg;
        u.s_a[d.n_chunks + c] = s_a_neg;
    }
    u.lr = lr;
    u.total_samples = total_samples;
    for (int j = 0; j < u.n_terms; ++j) u.splits[j] = 1;
    u.block_max = slot;
    u.max_blocks = FF_WS_MIN_BYTES / sizeof(uint32_t);
    HIPCHK_T(FF_K_UPDATE, launch_update(u, s));
    QuantArgs a;
    memset(&a, 0, sizeof(a));
    a.x = w_master;
    a.amax_bits = slot;
    a.amax_n = update_blocks(u);
    a.round_mode = FF_ROUND_NEAREST_EVEN;
    a.rows = d.N;
    a.cols = d.K;
    a.q = w_q;
    a.ldq = pitch8(d.K);
    a.scale = s_w;
    a.nb = 1;
    a.rows_per_sample = 1;
    HIPCHK_T(FF_K_QUANT_W, launch_quantize(QSRC_F32, a, s));
    return FF_OK;
}

size_t ff_workspace_bytes(const ff_net_desc* net)
{
    WsLayout w;
    if (make_layout(net, &w) != FF_OK) return 0;
    return w.total;
}

}  // extern "C"

// One iteration of Algorithm 1.  step_dev == null: the step number is `step`; otherwise it is read from device
// memory by the kernels (and advanced by one at the end when `advance` is set).
// Streams and events of the update-chain lanes: lane 0 is the caller's stream, lanes 1 .. MAX_LANES - 1 are streams
// the library creates once per device (default priority, non-blocking) and keeps until the process ends.  A step forks
// them off the caller's stream with an event after the look-ahead kernel and joins them back before it returns, so for
// the caller the step is still one piece of work in stream order (also under graph capture, where fork and join
// become graph edges).
struct LanePool {
    hipStream_t st[MAX_LANES - 1];
    hipEvent_t fork, join[MAX_LANES - 1];
    bool ready;
};
static LanePool g_lanes[MAX_DEVICES];
static std::mutex g_lanes_mutex;

static LanePool* lanes_of_current_device(bool may_create)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_lanes_mutex);
    LanePool& p = g_lanes[dev];
    if (p.ready) return &p;
    if (!may_create) return nullptr;
    bool ok = hipEventCreateWithFlags(&p.fork, hipEventDisableTiming) == hipSuccess;
    for (int i = 0; i < MAX_LANES - 1 && ok; ++i)
        ok = hipStreamCreateWithFlags(&p.st[i], hipStreamNonBlocking) == hipSuccess &&
             hipEventCreateWithFlags(&p.join[i], hipEventDisableTiming) == hipSuccess;
    if (!ok) return nullptr;   // (whatever was created stays allocated; the step then runs on one stream)
    p.ready = true;
    return &p;
}

static ff_status train_step_impl(const ff_net_desc* net, const ff_net_state* state, const float* x_pos,
                                 const float* x_neg, float theta, float lambda, float lr, uint64_t seed, uint64_t step,
                                 uint64_t* step_dev, int32_t advance, float* loss, float* goodness, void* ws,
                                 size_t ws_bytes, void* stream)
{
    WsLayout w;
    const ff_status st = make_layout(net, &w);
    if (st != FF_OK) return st;
    if (!state || !state->w_master || !state->w_q || !state->s_w || !x_pos || !x_neg || !loss || !goodness || !ws)
        return FF_ERR_INVALID_ARG;
    for (int i = 0; i < w.k; ++i) {
        if (!state->w_master[i] || !state->w_q[i] || !state->s_w[i]) return FF_ERR_INVALID_ARG;
        if (!aligned4(state->w_master[i]) || !aligned16(state->w_q[i])) return FF_ERR_ALIGN;
    }
    if (ws_bytes < w.total) return FF_ERR_WORKSPACE;
    if (!aligned16(ws) || !aligned4(x_pos) || !aligned4(x_neg) || !aligned4(loss) || !aligned4(goodness))
        return FF_ERR_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    char* base = (char*)ws;
    const int k = w.k;
    const int64_t B = w.B;
    uint32_t* out_amax = (uint32_t*)(base + w.off_slots);  // [k+1][2]: slot 0 the net input, slot j+1 the output of layer j
    uint32_t* g_amax = out_amax + 2 * (k + 1);             // [k][2]
    uint32_t* w_amax = g_amax + 2 * k;                     // [k]
    unsigned long long* gsum = (unsigned long long*)(base + w.off_gsum);
    int32_t* vmax = (int32_t*)(base + w.off_vmax);
    float* s_a = (float*)(base + w.off_scales);  // [k][2]
    float* s_g = s_a + 2 * k;                    // [k][2]
    float* c = (float*)(base + w.off_c);
    float* ct = (float*)(base + w.off_ct);

    const int64_t n_in = w.d[0].in_rows * w.d[0].in_cols;
    const int64_t st_x = ((intptr_t)x_neg - (intptr_t)x_pos) / (intptr_t)sizeof(float);
    if (w.fused_ok && (w.fused_auto || net->launch_mode == FF_LAUNCH_FUSED)) {
        // the whole step in one persistent launch (small dense stacks; see fused.hip): it clears what it adds to itself
        FusedArgs fa;
        memset(&fa, 0, sizeof(fa));
        fa.k = k;
        fa.B = (int32_t)B;
        fa.lambda = lambda;
        fa.lr = lr;
        fa.seed = seed;
        fa.step = step;
        fa.step_dev = step_dev;
        fa.advance = advance;
        fa.x = x_pos;
        fa.st_x = st_x;
        fa.wg_amax = (uint32_t*)(base + w.off_wbmax);   // (UPDATE_MAX_BLOCKS words: more than the 256 workgroups at most)
        fa.w_amax = w_amax;
        fa.gsum = gsum;
        fa.vmax = vmax;
        fa.s_a = s_a;
        fa.s_g = s_g;
        fa.c = c;
        fa.ct = ct;
        fa.goodness = goodness;
        fa.loss = loss;
        for (int i = 0; i < k; ++i) {
            const Dims& d = w.d[i];
            FusedLayer& fl = fa.L[i];
            fl.K = (int32_t)d.K;
            fl.N = (int32_t)d.N;
            fl.relu = net->layers[i].relu ? 1 : 0;
            fl.l2norm = net->layers[i].l2norm_out ? 1 : 0;
            fl.train = (!net->train_layer || net->train_layer[i]) ? 1 : 0;
            fl.rshift = goodness_shift(d.K, d.rps * d.N);
            fl.theta = net->theta_layer ? net->theta_layer[i] : theta;
            fl.w = state->w_master[i];
            fl.wq = state->w_q[i];
            fl.sw = state->s_w[i];
            fl.aq = (int8_t*)(base + w.off_aq[i]);
            fl.st_aq = (int64_t)w.st_aq[i];
            fl.aqt = (int8_t*)(base + w.off_aqt[i]);
            fl.st_aqt = (int64_t)w.st_aqt[i];
            fl.acc = (int32_t*)(base + w.off_acc[i]);
            fl.st_acc = (int64_t)(w.st_acc[i] / sizeof(int32_t));
            fl.gy = (int8_t*)(base + w.off_fgy[i]);
            fl.st_gy = (int64_t)w.st_fgy[i];
        }
        fa.stamps = g_fused_stamps;
        HIPCHK_T(FF_K_FUSED, launch_fused_dense_step(fa, w.fused_wgs, s));
        return FF_OK;
    }
    uint32_t* const xmax = (uint32_t*)(base + w.off_xmax);
    HIPCHK_T(FF_K_ABSMAX, launch_absmax(x_pos, st_x, 2, n_in, xmax, s, (uint32_t*)base, (int64_t)(w.zero_bytes / 4)));
    // One kernel forms every layer's goodness, loss and coefficients after the forward pass; the hand-off needs only the range
    // of a layer's output.  Small batches: each of the quantiser's workgroups takes it from the per-sample maxima (256
    // threads: a few loads each; with normalisation also a square root and a division per sample).  Larger ones: a small
    // launch of its own, one workgroup per pass, and beyond that the kernels per layer, which spread a layer's samples over
    // several workgroups.
    // The small launch against taking the range in the quantiser: 784-1000-1000-1000 with 512 samples 120 -> 118 us, 2000
    // 164 -> 163, 3000 213 -> 215, 8000 396 -> 416; with normalisation 512 116 -> 114, 1500 153 -> 153, 2000 171 -> 174, 4000
    // 298 -> 307; 16-64-128 channels on 4x4 maps cross at the same batches.
    // The kernels per layer against this, with normalisation: 784-1000-1000-1000 with 5000 samples 356 -> 354 us, 8192 402 ->
    // 408, 16384 645 -> 677, 300-64-64-64 with 5000 122 -> 117, 12000 146 -> 151; without: 5000 345 -> 337 and 114 -> 105,
    // 12000 505 -> 503 and 142 -> 138, 16384 634 -> 638 and 153 -> 159.
    bool normalised = false;   // a hand-off range of square roots and divisions
    for (int i = 0; i + 1 < k; ++i) normalised = normalised || net->layers[i].l2norm_out;
    const bool goodness_last = B <= (normalised ? 6144 : 12288);
    auto range_launch = [&](const ff_layer_desc& L) { return B > (L.l2norm_out ? 1024 : 2048); };
    // ---- streams: the caller's, plus the library's own where the step runs independent work side by side
    hipStream_t lane_stream[MAX_LANES];
    for (int l = 0; l < MAX_LANES; ++l) lane_stream[l] = s;
    int n_lanes = 1;
    LanePool* pool = nullptr;
    if (w.lanes > 1 && !w.chain) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        const bool capturing = hipStreamIsCapturing(s, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone;
        pool = lanes_of_current_device(!capturing);   // nothing is created while a graph is being captured
        if (pool) {
            n_lanes = w.lanes;
            for (int l = 1; l < n_lanes; ++l) lane_stream[l] = pool->st[l - 1];
        }
    }
    const hipStream_t s_main = s;

    // a pass over layer t, whose accumulators are not kept (both passes; the weights are those before the layer's update)
    auto rework = [&](int what, int t, const QuantArgs& qa, hipStream_t s) {
        if (w.d[t].kind == FF_DWCONV2D)
            return launch_dwconv_rework(what, dw_forward_args(w.d[t], qa.relu, (const int8_t*)(base + w.off_aq[t]), (int64_t)w.st_aq[t], state->w_q[t], 2), qa, s);
        const GemmArgs g = forward_args(w.d[t], qa.relu, (const int8_t*)(base + w.off_aq[t]), (int64_t)w.st_aq[t], state->w_q[t],
                                  (const int8_t*)(base + w.off_col[t]), (int64_t)w.st_col[t], 2);
        return launch_rework(what, g, qa, s);
    };

    // The goodness sums of a residual block's output need its range over the pass first, and so does the quantiser of the next
    // layer: where nothing asks for them before the end of the pass, the quantiser forms them as it reads the tensor (its workgroups
    // read the B maxima each, hence the bound).  fx_reader[i]: that layer, or -1: a launch of its own (the last block).
    // 64 channels, two passes of 256 images of 32x32: 26 + 29 us as two launches.
    int fx_reader[MAX_LAYERS];
    for (int i = 0; i < k; ++i) {
        fx_reader[i] = -1;
        if (w.d[i].skip == FF_SKIP_NONE || !goodness_last || B > 2048 || net->launch_mode == FF_LAUNCH_KERNELS) continue;
        for (int j = k - 1; j > i; --j)
            if (w.d[j].src == i && w.d[j].role == FF_ROLE_LAYER) fx_reader[i] = j;
    }

    // ---- forward pass through all layers, both data sets together (Algorithm 1) -----------------
    bool proj_pending = false;   // a projection's forward pass is running on the second stream
    for (int i = 0; i < k; ++i) {
        const Dims& d = w.d[i];
        const ff_layer_desc& L = net->layers[i];
        const bool dense = d.kind == FF_DENSE;
        // The 1x1 projection of a residual block and the block's first convolution read the same input and do not
        // depend on each other: with a second stream at hand the projection (quantiser + contraction; no patch
        // scratch: it reads the input tensor directly) runs there, and the block's second convolution waits for it.
        const bool side = n_lanes > 1 && d.role == FF_ROLE_PROJECTION && (d.implicit || d.pointwise) && !proj_pending;
        hipStream_t s = s_main;
        if (side) {
            if (hipEventRecord(pool->fork, s_main) != hipSuccess || hipStreamWaitEvent(lane_stream[1], pool->fork, 0) != hipSuccess)
                return FF_ERR_HIP;
            s = lane_stream[1];
        }
        QuantArgs a;
        memset(&a, 0, sizeof(a));
        int src;
        if (d.src < 0) {
            src = QSRC_F32;
            a.x = x_pos;
            a.st_x = st_x;
            a.rows_per_sample = 1;
        } else if (w.d[d.src].skip != FF_SKIP_NONE) {
            // the source is a residual layer: its block output is held as fp32
            src = QSRC_F32;
            a.x = (const float*)(base + w.off_y[d.src]);
            a.st_x = (int64_t)(w.st_y[d.src] / sizeof(float));
            a.rows_per_sample = dense ? 1 : (int32_t)w.d[d.src].rps;
            if (fx_reader[d.src] == i) {
                src = QSRC_F32_FX;
                a.fx_gsum = gsum + (int64_t)d.src * 2 * B;
                a.st_b = B;
                a.fx_amax = out_amax + 2 * (d.src + 1);
            }
        } else {
            const int j = d.src;
            const Dims& dp = w.d[j];
            const ff_layer_desc& Lp = net->layers[j];
            src = QSRC_HANDOFF;
            a.acc = (const int32_t*)(base + w.off_acc[j]);
            a.st_acc = (int64_t)(w.st_acc[j] / sizeof(int32_t));
            a.ldacc = pitch32(dp.N);
            a.s_a = s_a + 2 * j;
            a.st_s_a = 1;
            a.s_w = state->s_w[j];
            a.st_s_w = 0;
            a.per_sample = goodness + (int64_t)j * 2 * B;
            a.st_per_sample = B;
            a.rows_per_sample = (int32_t)dp.rps;
            if (dp.kind != FF_DENSE && dense) {   // flatten: one row of H_out * W_out * C contiguous accumulators per sample
                a.ldacc = d.K;
                a.rows_per_sample = 1;
            }
            a.relu = Lp.relu ? 1 : 0;
            a.l2norm = Lp.l2norm_out ? 1 : 0;
            if (goodness_last) {
                if (!range_launch(Lp)) a.vmax = vmax + (int64_t)j * 2 * B;
                a.gsum = gsum + (int64_t)j * 2 * B;
                a.B = (int32_t)B;
                a.rshift = goodness_shift(dp.K, dp.rps * dp.N);
                a.st_b = B;
            }
        }
        a.amax_bits = d.src < 0 ? xmax : out_amax + 2 * (d.src + 1);
        a.st_amax = d.src < 0 ? ABSMAX_MAX_BLOCKS : 1;
        a.amax_n = d.src < 0 ? absmax_blocks(n_in) : 0;
        if (d.src >= 0 && fx_reader[d.src] >= 0) {   // the range straight from the block's per-sample maxima
            a.amax_bits = (const uint32_t*)(vmax + (int64_t)d.src * 2 * B);
            a.st_amax = (int32_t)B;
            a.amax_n = (int32_t)B;
        }
        a.round_mode = FF_ROUND_STOCHASTIC;
        a.key = make_sr_key(seed, ff_stream_tag(step, (uint32_t)i, 0, FF_KIND_ACT));
        a.key2 = make_sr_key(seed, ff_stream_tag(step, (uint32_t)i, 1, FF_KIND_ACT));
        a.step_dev = step_dev;
        a.seed = seed;
        a.tag_layer = (uint32_t)i;
        a.tag_kind = FF_KIND_ACT;
        a.rows = d.in_rows;
        a.cols = d.in_cols;
        a.q = (int8_t*)(base + w.off_aq[i]);
        a.st_q = (int64_t)w.st_aq[i];
        a.ldq = pitch8(d.in_cols);
        if (dense) {
            a.q_t = (int8_t*)(base + w.off_aqt[i]);
            a.st_qt = (int64_t)w.st_aqt[i];
            a.ldqt = pitch8(d.M);
            a.qt_streaming = 1;   // read again only by this layer's weight gradient, after every forward pass
        }
        a.scale = s_a + 2 * i;
        a.st_scale = 1;
        a.nb = 2;
        const bool plain = d.role == FF_ROLE_LAYER && d.skip == FF_SKIP_NONE;   // goodness straight from the accumulators
        ResidualArgs ra;
        memset(&ra, 0, sizeof(ra));
        if (!plain && d.role != FF_ROLE_PROJECTION) {
            ra.acc = (const int32_t*)(base + w.off_acc[i]);
            ra.ldacc = pitch32(d.N);
            ra.st_acc = (int64_t)(w.st_acc[i] / sizeof(int32_t));
            ra.s_a = s_a + 2 * i;
            ra.st_s_a = 1;
            ra.s_w = state->s_w[i];
            ra.skip = d.skip;
            if (d.skip == FF_SKIP_IDENTITY) {
                ra.xq = (const int8_t*)(base + w.off_aq[i - 1]);
                ra.ldx = pitch8(w.d[i - 1].in_cols);
                ra.st_xq = (int64_t)w.st_aq[i - 1];
                ra.s_x = s_a + 2 * (i - 1);
                ra.st_s_x = 1;
            } else {
                ra.accp = (const int32_t*)(base + w.off_acc[i - 2]);
                ra.ldaccp = pitch32(w.d[i - 2].N);
                ra.st_accp = (int64_t)(w.st_acc[i - 2] / sizeof(int32_t));
                ra.s_ap = s_a + 2 * (i - 2);
                ra.st_s_ap = 1;
                ra.s_wp = state->s_w[i - 2];
            }
            ra.relu = L.relu ? 1 : 0;
            ra.M = d.M;
            ra.N = d.N;
            ra.rows_per_sample = (int32_t)d.rps;
            ra.y = (float*)(base + w.off_y[i]);
            ra.st_y = (int64_t)(w.st_y[i] / sizeof(float));
            ra.ymax_bits = (uint32_t*)(vmax + (int64_t)i * 2 * B);
            ra.st_b = B;
            ra.nb = 2;
        }
        // Implicit contractions form the block output from the accumulators; behind others a launch of its own does, and where a
        // wavefront's rows belong to more than two samples (measured with one atomic per row there: 512 channels on 4x4 maps 87 us
        // against 39 + 10).
        const bool in_contraction = ra.y && d.implicit && !d.pointwise && d.rps >= RESIDUAL_MIN_ROWS && net->launch_mode != FF_LAUNCH_KERNELS;
        // The projection's accumulators are read by whichever launch forms the block output: until then its stream runs beside this one.
        // (At 38 and 237 images with maps of 49 and 16 pixels last, a step takes as long with the wait ahead of every second
        // convolution: 820 and 1780 us.)
        auto join_projection = [&] {
            if (d.skip != FF_SKIP_PROJECTION || !proj_pending) return true;
            proj_pending = false;
            return hipStreamWaitEvent(s_main, pool->join[0], 0) == hipSuccess;
        };
        ff_status fs = [&]() -> ff_status {
            if (d.role == FF_ROLE_PROJECTION && !goodness_last) {
                // no activity of its own: zero coefficients (nothing enters the look-ahead sums), zero loss / goodness rows
                // (on the projection's own stream: nothing reads them before the look-ahead kernel)
                HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)(c + (int64_t)i * 2 * B), 2 * B, 0u, s));
                HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)(goodness + (int64_t)i * 2 * B), 2 * B, 0u, s));
                HIPCHK_T(FF_K_SMALL, launch_fill_u32((uint32_t*)(loss + 2 * i), 2, 0u, s));
            }
            if (src == QSRC_HANDOFF && w.rework[d.src]) HIPCHK_T(FF_K_QUANT_ACT, rework(ROWS_HANDOFF, d.src, a, s));
            else HIPCHK_T(FF_K_QUANT_ACT, launch_quantize(src, a, s));
            if (in_contraction && !join_projection()) return FF_ERR_HIP;
            return run_forward(d, L.relu ? 1 : 0, (const int8_t*)(base + w.off_aq[i]), (int64_t)w.st_aq[i], state->w_q[i],
                               w.rework[i] ? nullptr : (int32_t*)(base + w.off_acc[i]), (int64_t)(w.st_acc[i] / sizeof(int32_t)),
                               plain ? gsum + (int64_t)i * 2 * B : nullptr, vmax + (int64_t)i * 2 * B, B,
                               (int8_t*)(base + w.off_col[i]), (int64_t)w.st_col[i], 2, s, in_contraction ? &ra : nullptr);
        }();
        if (side) {   // (whatever happened on the second stream, it is joined back)
            if (hipEventRecord(pool->join[0], s) != hipSuccess) fs = fs != FF_OK ? fs : FF_ERR_HIP;
            proj_pending = true;
            if (fs != FF_OK) (void)hipStreamWaitEvent(s_main, pool->join[0], 0);
        }
        if (fs != FF_OK) return fs;
        if (d.role == FF_ROLE_PROJECTION) continue;
        if (!plain) {
            if (!in_contraction) {
                if (!join_projection()) return FF_ERR_HIP;
                HIPCHK_T(FF_K_RESIDUAL, launch_residual_act(ra, s));
            }
            if (fx_reader[i] >= 0) continue;
            GoodnessFxArgs fa;
            memset(&fa, 0, sizeof(fa));
            fa.y = ra.y;
            fa.st_y = ra.st_y;
            fa.M = d.M;
            fa.N = d.N;
            fa.rows_per_sample = (int32_t)d.rps;
            fa.ymax_bits = ra.ymax_bits;
            fa.amax_bits = out_amax + 2 * (i + 1);
            fa.st_amax = 1;
            fa.gsum = gsum + (int64_t)i * 2 * B;
            fa.st_b = B;
            fa.nb = 2;
            HIPCHK_T(FF_K_RESIDUAL, launch_goodness_fx(fa, s));
        }

        if (goodness_last) {
            if (plain && i + 1 < k && range_launch(L)) {
                RangeArgs r;
                memset(&r, 0, sizeof(r));
                r.vmax = vmax + (int64_t)i * 2 * B;
                r.gsum = gsum + (int64_t)i * 2 * B;
                r.s_a = s_a + 2 * i;
                r.s_w = state->s_w[i];
                r.rshift = goodness_shift(d.K, d.rps * d.N);
                r.l2norm = L.l2norm_out ? 1 : 0;
                r.B = B;
                r.out = out_amax + 2 * (i + 1);
                HIPCHK_T(FF_K_SMALL, launch_handoff_range(r, s));
            }
            continue;
        }
        GoodnessArgs ga;
        memset(&ga, 0, sizeof(ga));
        ga.gsum = gsum + (int64_t)i * 2 * B;
        ga.vmax = vmax + (int64_t)i * 2 * B;
        ga.s_a = s_a + 2 * i;
        ga.s_w = state->s_w[i];
        ga.rshift = goodness_shift(d.K, d.rps * d.N);
        ga.l2norm = L.l2norm_out ? 1 : 0;
        ga.pass_sign = FF_PASS_POS;
        ga.theta = net->theta_layer ? net->theta_layer[i] : theta;
        ga.B = B;
        ga.goodness = goodness + (int64_t)i * 2 * B;
        ga.coeff = c + (int64_t)i * 2 * B;
        ga.loss_mean = loss + 2 * i;
        // the absmax of this layer's output, i.e. of the input of whichever layers read it
        ga.next_amax_bits = plain ? out_amax + 2 * (i + 1) : nullptr;
        ga.fx_amax_bits = plain ? nullptr : out_amax + 2 * (i + 1);
        ga.nb = 2;
        ga.st_b = B;
        ga.st_scalar = 1;
        ga.loss_part = (unsigned long long*)(base + w.off_gl);
        ga.wg_counter = (uint32_t*)(base + w.off_gl + sizeof(uint64_t) * 2 * GL_MAX_WG);
        HIPCHK_T(FF_K_SMALL, launch_goodness_loss(ga, s));
    }

    if (proj_pending && hipStreamWaitEvent(s_main, pool->join[0], 0) != hipSuccess) return FF_ERR_HIP;

    // ---- look-ahead coefficients of every layer (Eq. (3)/(4)) and the absmax of every local gradient
    if (goodness_last) {
        GoodnessAllArgs ga;
        memset(&ga, 0, sizeof(ga));
        ga.k = k;
        ga.B = B;
        ga.lambda = w.chain ? 0.0f : lambda;   // (the chain combines the layers' own coefficients)
        ga.gsum = gsum;
        ga.vmax = vmax;
        ga.s_a = s_a;
        ga.out_amax = out_amax;
        ga.goodness = goodness;
        ga.coeff = c;
        ga.coeff_total = ct;
        ga.loss = loss;
        ga.g_amax_bits = g_amax;
        for (int i = 0; i < k; ++i) {
            const Dims& d = w.d[i];
            ga.L[i].s_w = state->s_w[i];
            ga.L[i].theta = net->theta_layer ? net->theta_layer[i] : theta;
            ga.L[i].rshift = goodness_shift(d.K, d.rps * d.N);
            ga.L[i].fx = d.skip != FF_SKIP_NONE;
            ga.L[i].projection = d.role == FF_ROLE_PROJECTION;
        }
        HIPCHK_T(FF_K_SMALL, launch_goodness_all(ga, s));
    } else if (!w.chain) {
        LookaheadArgs la;
        memset(&la, 0, sizeof(la));
        la.coeff = c;
        la.coeff_total = ct;
        la.k = k;
        la.np = 2;
        la.B = B;
        la.st_layer = 2 * B;
        la.st_pass = B;
        la.lambda = lambda;
        la.vmax = vmax;
        la.s_a = s_a;
        la.s_w = state->s_w;
        la.g_amax_bits = g_amax;
        for (int i = 0; i < k; ++i)
            if (w.d[i].skip != FF_SKIP_NONE) la.fx_mask |= 1u << i;
        HIPCHK_T(FF_K_SMALL, launch_lookahead(la, s));
    }

    // ---- per layer: int8 local gradient, int8 weight gradient, update (Algorithm 1, inner loop) ----
    // weights of layer `t` from the transposed int8 gradient in the scratch (quantised for layer `gl`): weight-gradient
    // contraction per pass and chunk, combined update, requantisation
    // ---- lanes: which copy of the chain scratch and which stream a layer's update chain uses
    int lane_of[MAX_LAYERS];
    {
        // longest chain first onto the lane with the least work so far (cost ~ multiply-adds of the layer)
        double load[MAX_LANES];
        for (int l = 0; l < MAX_LANES; ++l) load[l] = 0.0;
        bool placed[MAX_LAYERS];
        for (int i = 0; i < k; ++i) { placed[i] = false; lane_of[i] = 0; }
        for (int n = 0; n < k && n_lanes > 1; ++n) {
            int best = -1;
            double bc = -1.0;
            for (int i = 0; i < k; ++i) {
                const double c = (double)w.d[i].M * (double)w.d[i].K * (double)w.d[i].N;
                if (!placed[i] && c > bc) { bc = c; best = i; }
            }
            int l = 0;
            for (int j = 1; j < n_lanes; ++j)
                if (load[j] < load[l]) l = j;
            placed[best] = true;
            lane_of[best] = l;
            load[l] += bc;
        }
        // a projection is updated by the chain of the block's second convolution
        for (int i = 0; i < k; ++i)
            if (w.d[i].skip == FF_SKIP_PROJECTION && i >= 2) lane_of[i - 2] = lane_of[i];
    }
    // joins the lanes back into the caller's stream: explicitly at the end of the chains, and on every early way out
    struct Join {
        LanePool* pool;
        hipStream_t* st;
        int n;
        ff_status finish()
        {
            bool ok = true;
            for (int l = 1; l < n; ++l) {
                ok = hipEventRecord(pool->join[l - 1], st[l]) == hipSuccess && ok;
                ok = hipStreamWaitEvent(st[0], pool->join[l - 1], 0) == hipSuccess && ok;
            }
            n = 1;
            return ok ? FF_OK : FF_ERR_HIP;
        }
        ~Join() { (void)finish(); }
    };

    auto wgrad_update = [&](int t, int gl) -> ff_status {
        const Dims& d = w.d[t];
        const int lane = lane_of[gl];
        hipStream_t s = lane_stream[lane];                        // (shadows the caller's stream inside the chain)
        char* base = (char*)ws + (size_t)lane * w.lane_stride;   // lane-scoped scratch: gy, dw, part, wbmax
        char* const base0 = (char*)ws;                            // what lives outside the lanes
        const bool dense = d.kind == FF_DENSE;   // layers that keep a transposed copy of their input
        const int64_t dw_elems = (int64_t)(w.dw_bytes / sizeof(int32_t));
        const bool patches = wgrad_from_patches(d);
        const size_t off_q = dense ? w.off_aqt[t] : (patches ? w.off_col[t] : w.off_aq[t]);
        const size_t st_q = dense ? w.st_aqt[t] : (patches ? w.st_col[t] : w.st_aq[t]);
        uint32_t* wbmax = (uint32_t*)(base + w.off_wbmax);
        int candidates = 0;   // absmax candidates the update leaves at wbmax
        // Both passes in one workgroup halve the launch's workgroups: alone on the chip it has to have two per compute unit all
        // the same (1500 x 1500 at 1500 samples, 288 tiles: the chain's step 259 -> 269 us); beside other lanes it need not.
        const int fused = d.kind == FF_DENSE && d.n_chunks == 1 && aligned16(state->w_master[t]) ? gemm_update_blocks(d.N, d.K, d.M) : 0;
        if (fused && (n_lanes > 1 || fused >= 2 * num_cus())) {
            GemmArgs g;
            memset(&g, 0, sizeof(g));
            g.P = (const int8_t*)(base + w.off_gy);
            g.st_p = (int64_t)w.st_gy;
            g.ldp = pitch8(d.M);
            g.Q = (const int8_t*)(base0 + off_q);
            g.st_q = (int64_t)st_q;
            g.ldq = pitch8(d.M);
            g.I = (int32_t)d.N;
            g.J = (int32_t)d.K;
            g.R = (int32_t)d.M;
            g.rows_per_sample = 1;
            g.nb = 2;
            g.splits = 1;
            g.upd_w = state->w_master[t];
            for (int p = 0; p < 2; ++p) {
                g.upd_s_g[p] = s_g + 2 * gl + p;
                g.upd_s_a[p] = s_a + 2 * t + p;
            }
            g.upd_lr = lr;
            g.upd_samples = (int32_t)(2 * B);
            g.upd_max = wbmax;
            g.clk = g_clock_probe;
            HIPCHK_T(FF_K_GEMM_DW, launch_gemm_nt_i8(g, s));
            candidates = fused;
        } else {
            WgradTerms terms;
            const ff_status ws_ = run_wgrad(d, (const int8_t*)(base + w.off_gy), (int64_t)w.st_gy,
                                            (const int8_t*)(base0 + off_q), (int64_t)st_q, (int32_t*)(base + w.off_part),
                                            (int64_t)(w.part_bytes / sizeof(int32_t)), (int32_t*)(base + w.off_dw),
                                            (int64_t)(w.st_dw / sizeof(int32_t)), dw_elems, 2, s, &terms);
            if (ws_ != FF_OK) return ws_;

            UpdateArgs u;
            memset(&u, 0, sizeof(u));
            u.w = state->w_master[t];
            u.N = d.N;
            u.K = d.K;
            u.lddw = pitch32(d.K);
            u.n_terms = 2 * d.n_chunks;
            u.st_split = terms.st_split;
            for (int p = 0; p < 2; ++p)
                for (int cc = 0; cc < d.n_chunks; ++cc) {
                    const int tt = p * d.n_chunks + cc;
                    u.dw[tt] = terms.term[p][cc];
                    u.splits[tt] = terms.splits[cc];
                    u.s_g[tt] = s_g + 2 * gl + p;
                    u.s_a[tt] = s_a + 2 * t + p;
                }
            u.lr = lr;
            u.total_samples = (int32_t)(2 * B);
            u.block_max = wbmax;
            u.max_blocks = UPDATE_MAX_BLOCKS;
            HIPCHK_T(FF_K_UPDATE, launch_update(u, s));
            candidates = update_blocks(u);
        }

        QuantArgs qa;
        memset(&qa, 0, sizeof(qa));
        qa.x = state->w_master[t];
        qa.amax_bits = wbmax;
        qa.amax_n = candidates;
        qa.round_mode = FF_ROUND_NEAREST_EVEN;
        qa.rows = d.N;
        qa.cols = d.K;
        qa.q = state->w_q[t];
        qa.ldq = pitch8(d.K);
        qa.scale = state->s_w[t];
        qa.nb = 1;
        qa.rows_per_sample = 1;
        HIPCHK_T(FF_K_QUANT_W, launch_quantize(QSRC_F32, qa, s));
        return FF_OK;
    };
    auto trained = [&](int t) { return !net->train_layer || net->train_layer[t]; };

    if (w.chain) {
        // ---- Eq. (4) as an exact derivative: from the last layer down, the int8 gradient h_i is handed through the
        // pre-step weights of layer i to the layer below (dense layers only, checked by make_layout)
        uint32_t* h_amax = (uint32_t*)(base + w.off_cmax);   // [2][CHAIN_MAX_BLOCKS] each
        uint32_t* g_cand = h_amax + 2 * CHAIN_MAX_BLOCKS;
        float* s_h = s_g + 2 * k;             // [2]
        float* s_wt = s_h + 2;                // scale of the transposed weight copy (equals s_w of the layer)
        float* hf = (float*)(base + w.off_hf);
        float* gf = (float*)(base + w.off_gf);
        const int64_t st_f = (int64_t)(w.st_f / sizeof(float));
        int8_t* hq = (int8_t*)(base + w.off_hq);
        int32_t* eacc = (int32_t*)(base + w.off_e);
        int8_t* wqt = (int8_t*)(base + w.off_wqt);
        for (int i = k - 1; i >= 0; --i) {
            const Dims& d = w.d[i];
            const ff_layer_desc& L = net->layers[i];
            ChainArgs ca;
            memset(&ca, 0, sizeof(ca));
            ca.acc = (const int32_t*)(base + w.off_acc[i]);
            ca.ldacc = pitch32(d.N);
            ca.st_acc = (int64_t)(w.st_acc[i] / sizeof(int32_t));
            ca.s_a = s_a + 2 * i;
            ca.st_s_a = 1;
            ca.s_w = state->s_w[i];
            ca.coeff = c + (int64_t)i * 2 * B;
            ca.st_coeff = B;
            if (i < k - 1) {
                ca.e_acc = eacc;
                ca.lde = pitch32(d.N);
                ca.st_e = (int64_t)(w.st_e / sizeof(int32_t));
                ca.s_h = s_h;
                ca.st_s_h = 1;
                ca.s_w_up = s_wt;   // pre-step weight scale of layer i + 1 (state->s_w[i + 1] already holds the updated one)
            }
            ca.lambda = lambda;
            ca.relu = L.relu ? 1 : 0;
            ca.M = d.M;
            ca.N = d.N;
            ca.h = i > 0 ? hf : nullptr;
            ca.g = gf;
            ca.st_out = st_f;
            ca.h_amax_bits = h_amax;
            ca.g_amax_bits = g_cand;
            ca.nb = 2;
            // The last layer has nothing ahead of it: h = g = 2 c y, which the quantiser forms straight from the
            // accumulators (absmax by monotonicity, as in the default step); no fp32 tensors are written.
            const bool top = i == k - 1;
            int qsrc = QSRC_F32;
            QuantArgs a;
            memset(&a, 0, sizeof(a));
            if (top) {
                if (!goodness_last)
                    HIPCHK_T(FF_K_SMALL, launch_grad_amax(c + (int64_t)i * 2 * B, vmax + (int64_t)i * 2 * B, s_a + 2 * i,
                                                      state->s_w[i], B, 2, g_amax + 2 * i, s));
                qsrc = QSRC_GRAD;
                a.acc = ca.acc;
                a.st_acc = ca.st_acc;
                a.ldacc = ca.ldacc;
                a.s_a = ca.s_a;
                a.st_s_a = 1;
                a.s_w = ca.s_w;
                a.per_sample = ca.coeff;
                a.st_per_sample = B;
                a.relu = ca.relu;
            } else {
                HIPCHK_T(FF_K_CHAIN, launch_chain_combine(ca, s));
                a.x = gf;
                a.st_x = st_f;
            }
            a.rows_per_sample = 1;
            a.amax_bits = top ? g_amax + 2 * i : g_cand;
            a.st_amax = top ? 1 : CHAIN_MAX_BLOCKS;
            a.amax_n = top ? 0 : chain_blocks(d.M, d.N);
            a.round_mode = FF_ROUND_STOCHASTIC;
            a.key = make_sr_key(seed, ff_stream_tag(step, (uint32_t)i, 0, FF_KIND_GRAD));
            a.key2 = make_sr_key(seed, ff_stream_tag(step, (uint32_t)i, 1, FF_KIND_GRAD));
            a.step_dev = step_dev;
            a.seed = seed;
            a.tag_layer = (uint32_t)i;
            a.tag_kind = FF_KIND_GRAD;
            a.rows = d.M;
            a.cols = d.N;
            a.q_t = (int8_t*)(base + w.off_gy);
            a.st_qt = (int64_t)w.st_gy;
            a.ldqt = pitch8(d.M);
            a.scale = s_g + 2 * i;
            a.st_scale = 1;
            a.nb = 2;
            if (trained(i)) HIPCHK_T(FF_K_QUANT_GRAD, launch_quantize(qsrc, a, s));

            if (i > 0) {
                QuantArgs hqa = a;
                if (!top) {
                    hqa.x = hf;
                    hqa.amax_bits = h_amax;
                }
                hqa.key = make_sr_key(seed, ff_stream_tag(step, (uint32_t)i, 0, FF_KIND_CHAIN));
                hqa.key2 = make_sr_key(seed, ff_stream_tag(step, (uint32_t)i, 1, FF_KIND_CHAIN));
                hqa.tag_kind = FF_KIND_CHAIN;
                hqa.q_t = nullptr;
                hqa.st_qt = 0;
                hqa.ldqt = 0;
                hqa.q = hq;
                hqa.st_q = (int64_t)w.st_hq;
                hqa.ldq = pitch8(d.N);
                hqa.scale = s_h;
                HIPCHK_T(FF_K_CHAIN, launch_quantize(qsrc, hqa, s));

                // transposed int8 copy of the pre-step weights: the same codes as w_q, [K, pitch(N)]
                HIPCHK_T(FF_K_CHAIN, launch_transpose_i8(state->w_q[i], wqt, d.N, d.K, state->s_w[i], s_wt, s));

                GemmArgs ga;
                memset(&ga, 0, sizeof(ga));
                ga.P = hq;
                ga.Q = wqt;
                ga.C = eacc;
                ga.I = (int32_t)d.M;
                ga.J = (int32_t)d.K;
                ga.R = (int32_t)d.N;
                ga.ldp = pitch8(d.N);
                ga.ldq = pitch8(d.N);
                ga.ldc = pitch32(d.K);
                ga.nb = 2;
                ga.st_p = (int64_t)w.st_hq;
                ga.st_q = 0;
                ga.st_c = (int64_t)(w.st_e / sizeof(int32_t));
                ga.splits = 1;
                HIPCHK_T(FF_K_CHAIN, launch_gemm_nt_i8(ga, s));
            }
            if (trained(i)) {
                const ff_status us = wgrad_update(i, i);
                if (us != FF_OK) return us;
            }
        }
        if (step_dev && advance) HIPCHK_T(FF_K_SMALL, launch_advance_u64(step_dev, s));
        return FF_OK;
    }

    {
    Join join{pool, lane_stream, n_lanes};
    if (n_lanes > 1) {   // fork: the lanes start where the caller's stream stands now (all forward passes, the look-ahead)
        if (hipEventRecord(pool->fork, s) != hipSuccess) return FF_ERR_HIP;
        for (int l = 1; l < n_lanes; ++l)
            if (hipStreamWaitEvent(lane_stream[l], pool->fork, 0) != hipSuccess) return FF_ERR_HIP;
    }
    for (int i = 0; i < k; ++i) {
        const Dims& d = w.d[i];
        if (d.role == FF_ROLE_PROJECTION) continue;   // updated with the gradient of the block output, layer i + 2
        const bool with_proj = d.skip == FF_SKIP_PROJECTION && trained(i - 2);
        if (!trained(i) && !with_proj) continue;      // frozen layer: forward only
        const ff_layer_desc& L = net->layers[i];
        hipStream_t ls = lane_stream[lane_of[i]];
        char* const lbase = base + (size_t)lane_of[i] * w.lane_stride;   // this chain's copy of the scratch
        QuantArgs a;
        memset(&a, 0, sizeof(a));
        int src = QSRC_GRAD;
        if (d.skip != FF_SKIP_NONE) {
            src = QSRC_F32_GRAD;
            a.x = (const float*)(base + w.off_y[i]);
            a.st_x = (int64_t)(w.st_y[i] / sizeof(float));
        } else {
            a.acc = (const int32_t*)(base + w.off_acc[i]);
            a.st_acc = (int64_t)(w.st_acc[i] / sizeof(int32_t));
            a.ldacc = pitch32(d.N);
            a.s_a = s_a + 2 * i;
            a.st_s_a = 1;
            a.s_w = state->s_w[i];
        }
        a.per_sample = ct + (int64_t)i * 2 * B;
        a.st_per_sample = B;
        a.rows_per_sample = (int32_t)d.rps;
        a.relu = L.relu ? 1 : 0;
        a.amax_bits = g_amax + 2 * i;
        a.st_amax = 1;
        a.round_mode = FF_ROUND_STOCHASTIC;
        a.key = make_sr_key(seed, ff_stream_tag(step, (uint32_t)i, 0, FF_KIND_GRAD));
        a.key2 = make_sr_key(seed, ff_stream_tag(step, (uint32_t)i, 1, FF_KIND_GRAD));
        a.step_dev = step_dev;
        a.seed = seed;
        a.tag_layer = (uint32_t)i;
        a.tag_kind = FF_KIND_GRAD;
        a.rows = d.M;
        a.cols = d.N;
        if (d.kind == FF_DWCONV2D) {   // the depthwise weight gradient reads the gradient row-major
            a.q = (int8_t*)(lbase + w.off_gy);
            a.st_q = (int64_t)w.st_gy;
            a.ldq = pitch8(d.N);
        } else {
            a.q_t = (int8_t*)(lbase + w.off_gy);
            a.st_qt = (int64_t)w.st_gy;
            a.ldqt = pitch8(d.M);
        }
        a.scale = s_g + 2 * i;
        a.st_scale = 1;
        a.nb = 2;
        {
            hipStream_t s = ls;   // (the launch's stream, for its timing events)
            if (w.rework[i]) HIPCHK_T(FF_K_QUANT_GRAD, rework(ROWS_GRAD, i, a, s));
            else HIPCHK_T(FF_K_QUANT_GRAD, launch_quantize(src, a, s));
        }

        if (trained(i)) {
            const ff_status us = wgrad_update(i, i);
            if (us != FF_OK) return us;
        }
        if (with_proj) {
            const ff_status us = wgrad_update(i - 2, i);
            if (us != FF_OK) return us;
        }
    }
    const ff_status js = join.finish();
    if (js != FF_OK) return js;
    }
    if (step_dev && advance) HIPCHK_T(FF_K_SMALL, launch_advance_u64(step_dev, s));
    return FF_OK;
}

extern "C" {

ff_status ff_train_step(const ff_net_desc* net, const ff_net_state* state, const float* x_pos, const float* x_neg,
                        float theta, float lambda, float lr, uint64_t seed, uint64_t step, float* loss,
                        float* goodness, void* ws, size_t ws_bytes, void* stream)
{
    return train_step_impl(net, state, x_pos, x_neg, theta, lambda, lr, seed, step, nullptr, 0, loss, goodness, ws,
                           ws_bytes, stream);
}

ff_status ff_train_step_at(const ff_net_desc* net, const ff_net_state* state, const float* x_pos, const float* x_neg,
                           float theta, float lambda, float lr, uint64_t seed, uint64_t* step_dev, int32_t advance,
                           float* loss, float* goodness, void* ws, size_t ws_bytes, void* stream)
{
    if (!step_dev || ((uintptr_t)step_dev & 7)) return step_dev ? FF_ERR_ALIGN : FF_ERR_INVALID_ARG;
    return train_step_impl(net, state, x_pos, x_neg, theta, lambda, lr, seed, 0, step_dev, advance, loss, goodness, ws,
                           ws_bytes, stream);
}

ff_status ff_timing_enable(int32_t class_mask)
{
    g_timing.mask = (uint32_t)class_mask & ((1u << FF_K_COUNT) - 1u);
    return FF_OK;
}

ff_status ff_timing_clock_probe(uint64_t* counters)
{
    if (counters && ((uintptr_t)counters & 7)) return FF_ERR_ALIGN;
    g_clock_probe = (unsigned long long*)counters;
    return FF_OK;
}

ff_status ff_probe_mfma_ceiling(int32_t operand_kind, int32_t iterations, int32_t* sink, size_t sink_bytes,
                                uint64_t* counters, double* ops, void* stream)
{
    if (operand_kind < 0 || operand_kind > 2 || iterations < 1 || !sink || !ops) return FF_ERR_INVALID_ARG;
    if (!aligned4(sink) || (counters && ((uintptr_t)counters & 7))) return FF_ERR_ALIGN;
    const int g = num_cus();
    if (sink_bytes < (size_t)g * 512 * sizeof(int32_t)) return FF_ERR_WORKSPACE;
    int wgs = 0;
    if (launch_mfma_ceiling(sink, iterations, operand_kind, (unsigned long long*)counters, &wgs, (hipStream_t)stream) != hipSuccess)
        return FF_ERR_HIP;
    *ops = (double)wgs * 8.0 * (double)iterations * 8.0 * 65536.0;   // workgroups x wavefronts x iterations x MFMAs x ops
    return FF_OK;
}

ff_status ff_timing_fused_stamps(uint64_t* stamps)
{
    if (stamps && ((uintptr_t)stamps & 7)) return FF_ERR_ALIGN;
    g_fused_stamps = (unsigned long long*)stamps;
    return FF_OK;
}

ff_status ff_timing_reset(void)
{
    g_timing.n = 0;
    return FF_OK;
}

ff_status ff_timing_read(int32_t kernel_class, double* total_ms, int64_t* launches)
{
    if (!total_ms || !launches || kernel_class < 0 || kernel_class >= FF_K_COUNT) return FF_ERR_INVALID_ARG;
    double tot = 0.0;
    int64_t cnt = 0;
    for (int i = 0; i < g_timing.n; ++i) {
        if (g_timing.cls[i] != kernel_class) continue;
        if (hipEventSynchronize(g_timing.ev[2 * i + 1]) != hipSuccess) return FF_ERR_HIP;
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, g_timing.ev[2 * i], g_timing.ev[2 * i + 1]) != hipSuccess) return FF_ERR_HIP;
        tot += (double)ms;
        ++cnt;
    }
    *total_ms = tot;
    *launches = cnt;
    return FF_OK;
}

}  // extern "C"
