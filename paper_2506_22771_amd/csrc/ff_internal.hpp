// Internal declarations shared by the HIP translation units of libffint8 (gfx950 only).
// Host-side launchers are declared here; each is defined next to its kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/ffint8.h"

namespace ffi {

// ---- layout helpers -------------------------------------------------------------------------
// Row pitch of an int8 matrix in bytes: a multiple of 16 (the copy granule); rows longer than 512 bytes start on 128-byte
// lines, so that the 128-byte chunks the contraction copies per reduction step never straddle two cache lines (reduction
// lengths such as 784 or 2000 would otherwise cost every copy two line requests).  Kernels read a row only up to its
// length rounded up to 16; the bytes after that are padding that nothing reads.
__host__ __device__ static inline int64_t pitch8(int64_t cols)
{
    return cols <= 512 ? (cols + 15) & ~int64_t(15) : (cols + 127) & ~int64_t(127);
}
__host__ __device__ static inline int64_t pitch32(int64_t cols) { return (cols + 3) & ~int64_t(3); }
static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- stochastic-rounding key (Section IV-B cites stochastic rounding; the generator is ours) --
struct SrKey {
    uint32_t k0;  // low word of the 64-bit key
    uint32_t k1;  // (high word | 1), multiplies the high half of the element index
};
// key = finaliser of splitmix64 over (seed, stream tag); the same code runs on the host and, when the step
// number lives in device memory, at the head of the quantise kernels
__host__ __device__ inline SrKey make_sr_key(uint64_t seed, uint64_t tag)
{
    uint64_t z = seed + 0x9E3779B97F4A7C15ull * (tag + 1ull);
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    SrKey k;
    k.k0 = (uint32_t)z;
    k.k1 = (uint32_t)(z >> 32) | 1u;
    return k;
}
// stream tag of (step, layer, pass, kind): step << 20 | layer << 4 | pass << 2 | kind
__host__ __device__ inline uint64_t stream_tag_of(uint64_t step, uint32_t layer, uint32_t pass_idx, uint32_t kind)
{
    return (step << 20) | ((uint64_t)layer << 4) | ((uint64_t)pass_idx << 2) | (uint64_t)kind;
}

// ---- quantise kernels (elementwise.hip) -----------------------------------------------------
// QSRC_F32_GRAD: fp32 activities times the per-sample factor 2*coeff_total (local gradient of a residual layer)
// QSRC_HANDOFF_NORM: a hand-off with QuantArgs::l2norm; launch_quantize picks it
// QSRC_F32_FX: the fp32 output of a residual block; the launch also forms its goodness sums (fx_gsum)
enum QSource { QSRC_F32 = 0, QSRC_HANDOFF = 1, QSRC_GRAD = 2, QSRC_F32_GRAD = 3, QSRC_HANDOFF_NORM = 4, QSRC_F32_FX = 5 };

// One quantisation problem; `nb` problems (1 or 2) are launched together with the strides below.
struct QuantArgs {
    // source
    const float* x;          // QSRC_F32: [rows, cols] contiguous
    const int32_t* acc;      // QSRC_HANDOFF / QSRC_GRAD: [rows, ldacc]
    int64_t ldacc;
    const float* s_a;        // device scalars (HANDOFF / GRAD)
    const float* s_w;
    const float* per_sample; // HANDOFF with l2norm: goodness[B]; GRAD, F32_GRAD: coeff_total[B]
    int32_t rows_per_sample;
    int32_t relu, l2norm;
    // HANDOFF, optional: gsum: with l2norm the goodness of a row's sample straight from the contraction's sums (st_b apart
    // per pass) instead of per_sample.  vmax: the range straight from its per-sample maxima (and sums) instead of
    // amax_bits; every workgroup reads all B of them, for batches small beside the tensor.  GRAD, optional: vmax, likewise (with
    // the per-sample factors).
    const int32_t* vmax;
    const unsigned long long* gsum;
    int32_t B, rshift;
    int64_t st_b;
    // F32_FX: per-sample fixed-point goodness sums (as launch_goodness_fx; added to, st_b apart) and a word per pass for the absmax
    unsigned long long* fx_gsum;
    uint32_t* fx_amax;
    // quantiser
    const uint32_t* amax_bits;  // device: bit pattern of the non-negative fp32 absmax
    int32_t amax_n;             // > 1: amax_bits is an array of that many candidates, the absmax is their maximum
    int32_t round_mode;
    SrKey key;
    // destination
    int64_t rows, cols;
    int8_t* q;    // [rows, ldq] or null
    int64_t ldq;
    int8_t* q_t;  // [cols, ldqt] or null
    int64_t ldqt;
    int32_t qt_streaming;  // q_t is not read again soon: store it with a streaming hint
    int32_t row_per_xcd;   // filled in by the launch: a row of tiles is worked on by one XCD
    float* scale;  // device scalar out
    // batching (second problem = first + strides, in elements of the respective type)
    int32_t nb;
    int64_t st_x, st_acc, st_per_sample, st_q, st_qt;
    int32_t st_s_a, st_s_w, st_amax, st_scale;
    SrKey key2;  // key of the second problem
    // step number in device memory (null: the keys above are used).  The kernel then derives its key from
    // (seed, stream tag of (*step_dev, tag_layer, problem index, tag_kind)).
    const uint64_t* step_dev;
    uint64_t seed;
    uint32_t tag_layer, tag_kind;
};
hipError_t launch_quantize(int src, const QuantArgs& a, hipStream_t s);

// absmax of |x| over n floats of tensor z (x + z*st_x, z < nb): workgroup b stores the bit pattern of its maximum at
// part[z*ABSMAX_MAX_BLOCKS + b], b < absmax_blocks(n); the quantiser that follows takes the maximum of the array
// (QuantArgs::amax_n).
constexpr int ABSMAX_MAX_BLOCKS = 256;
int absmax_blocks(int64_t n);
// The launch also clears clear_n words at `clear` (work of a step that would be a launch of its own).
hipError_t launch_absmax(const float* x, int64_t st_x, int nb, int64_t n, uint32_t* part, hipStream_t s,
                         uint32_t* clear = nullptr, int64_t clear_n = 0);
hipError_t launch_clear2_u32(uint32_t* p, int64_t n, uint32_t* p2, int64_t n2, hipStream_t s);   // two ranges, one launch
hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s);
hipError_t launch_advance_u64(uint64_t* counter, hipStream_t s);   // *counter += 1, in stream order

// ---- per-sample kernels ----------------------------------------------------------------------
struct GoodnessArgs {
    const unsigned long long* gsum;
    const int32_t* vmax;
    const float* s_a;
    const float* s_w;
    int32_t rshift, l2norm;
    int32_t pass_sign;  // sign of the first problem; the second problem (nb == 2) uses the opposite
    float theta;
    int64_t B;
    float* goodness;
    float* coeff;
    float* loss_mean;
    uint32_t* next_amax_bits;  // may be null
    // non-null: gsum holds the fixed-point sums of a residual layer, G = fp32(gsum * 2^-40 * amax^2) with amax
    // from this slot (stride st_scalar); s_a, s_w and vmax are then unused
    const uint32_t* fx_amax_bits;
    int32_t nb;
    int64_t st_b;  // stride between problems for the [B] arrays
    int32_t st_scalar;  // stride for s_a / loss_mean / next_amax (s_w is shared)
    // Optional (large batches): several workgroups per pass.  loss_part: [nb][GL_MAX_WG] partial loss sums, wg_counter:
    // [nb]; the counters and the next_amax slots must be zero on entry, and the kernel leaves the counters zero.  The
    // workgroup that finishes last adds the partial sums in index order, so the mean does not depend on timing.
    unsigned long long* loss_part;
    uint32_t* wg_counter;
};
constexpr int GL_MAX_WG = 32;
hipError_t launch_goodness_loss(const GoodnessArgs& a, hipStream_t s);

// max over the samples of the handed-on activity (act(s_y acc), or that divided by sqrt(goodness)), both passes -> out[0], out[1]
struct RangeArgs {
    const int32_t* vmax;              // [2][B]
    const unsigned long long* gsum;   // [2][B]
    const float* s_a;                 // [2]
    const float* s_w;
    int32_t rshift, l2norm;
    int64_t B;
    uint32_t* out;
};
hipError_t launch_handoff_range(const RangeArgs& a, hipStream_t s);

// Goodness, loss, dL/dG and look-ahead of all layers of a step in one launch (two passes, [k][2][B] arrays).
struct GoodnessLayer {
    const float* s_w;
    float theta;
    int32_t rshift;
    int32_t fx;          // residual layer: fixed-point sums, vmax holds fp32 bit patterns
    int32_t projection;  // no activity of its own: zero goodness, loss and coefficient
};
struct GoodnessAllArgs {
    int32_t k;
    int64_t B;
    float lambda;
    const unsigned long long* gsum;
    const int32_t* vmax;
    const float* s_a;            // [k][2]
    const uint32_t* out_amax;    // [k+1][2]: slot i + 1 the output of layer i (fx layers)
    float* goodness;
    float* coeff;
    float* coeff_total;
    float* loss;                 // [k][2]
    uint32_t* g_amax_bits;       // [k][2], zeroed
    GoodnessLayer L[32];
};
hipError_t launch_goodness_all(const GoodnessAllArgs& a, hipStream_t s);

// coeff / coeff_total: [k][np][B] with strides; also (optionally) the absmax of each layer's local gradient.
struct LookaheadArgs {
    const float* coeff;
    float* coeff_total;
    int32_t k, np;
    int64_t B;
    int64_t st_layer, st_pass;
    float lambda;
    // optional gradient absmax (null vmax => skipped)
    const int32_t* vmax;       // same [k][np][B] strides
    const float* s_a;          // [k][np]
    const float* const* s_w;   // device array of k pointers to the layers' weight scales (may be null if vmax null)
    uint32_t* g_amax_bits;     // [k][np], zeroed
    uint32_t fx_mask;          // bit i: layer i's vmax entries are the fp32 bit patterns of max|y| (residual layer)
};
hipError_t launch_lookahead(const LookaheadArgs& a, hipStream_t s);

// ---- residual layers: block output y = act(s*acc + skip) as fp32, and its order-free goodness sums ------------
struct ResidualArgs {
    const int32_t* acc;  // [M, ldacc]
    int64_t ldacc, st_acc;
    const float* s_a;    // [z * st_s_a]
    const float* s_w;
    int32_t st_s_a;
    int32_t skip;        // FF_SKIP_IDENTITY / FF_SKIP_PROJECTION
    const int8_t* xq;    // identity: int8 [M, ldx] with scale s_x[z * st_s_x]
    int64_t ldx, st_xq;
    const float* s_x;
    int32_t st_s_x;
    const int32_t* accp; // projection: int32 [M, ldaccp] with scale s_ap[z * st_s_ap] * s_wp[0]
    int64_t ldaccp, st_accp;
    const float* s_ap;
    int32_t st_s_ap;
    const float* s_wp;
    int32_t relu;
    int64_t M, N;        // N % 4 == 0
    int32_t rows_per_sample;
    float* y;            // [M, N] contiguous
    int64_t st_y;
    uint32_t* ymax_bits; // [B] per pass (stride st_b), zeroed: bit pattern of max|y| per sample
    int64_t st_b;
    int32_t nb;
};
hipError_t launch_residual_act(const ResidualArgs& a, hipStream_t s);
constexpr int RESIDUAL_MIN_ROWS = 64;   // rows of a sample, where a contraction forms the block output (residual_max_store)

struct GoodnessFxArgs {
    const float* y;      // [M, N] contiguous
    int64_t st_y;
    int64_t M, N;
    int32_t rows_per_sample;
    const uint32_t* ymax_bits; // [B] per pass (stride st_b): bit patterns of max|y| per sample
    uint32_t* amax_bits;       // slot per pass (stride st_amax), written: max|y| over the pass
    int32_t st_amax;
    unsigned long long* gsum;  // [B] per pass (stride st_b), zeroed
    int64_t st_b;
    int32_t nb;
};
hipError_t launch_goodness_fx(const GoodnessFxArgs& a, hipStream_t s);

// ---- exact-derivative look-ahead (Eq. (4) taken literally; dense ReLU stacks) -----------------------------------
// Per element of one layer and pass: y = act(fp32(acc) * (s_a*s_w)), t = (2 c[b]) * y, E = fp32(e_acc) * (s_h*s_w_up)
// (0 without e_acc: the last layer), mask = acc > 0 under ReLU:
//   h = (t + E) * mask          -- handed down to the layer below (null h: not needed, first layer)
//   g = fma(lambda, E, t) * mask -- this layer's own local gradient
// and the absmax of both tensors (bit patterns, atomic max into zeroed slots).
struct ChainArgs {
    const int32_t* acc;  // [M, ldacc]
    int64_t ldacc, st_acc;
    const float* s_a;    // [z * st_s_a]
    int32_t st_s_a;
    const float* s_w;
    const float* coeff;  // [B] per pass (stride st_coeff): dL/dG of THIS layer
    int64_t st_coeff;
    const int32_t* e_acc;  // [M, lde] or null
    int64_t lde, st_e;
    const float* s_h;      // [z * st_s_h]: scale of the int8 gradient handed down by the layer above
    int32_t st_s_h;
    const float* s_w_up;   // weight scale of the layer above
    float lambda;
    int32_t relu;
    int64_t M, N;
    float* h;  // [M, N] contiguous per pass (stride st_out), may be null
    float* g;  // [M, N] contiguous per pass
    int64_t st_out;
    // absmax of both tensors: one candidate per workgroup at [z * CHAIN_MAX_BLOCKS + workgroup] (chain_blocks() of them), or,
    // with amax_atomic, one zeroed word each; h_amax_bits may be null with h
    uint32_t* h_amax_bits;
    uint32_t* g_amax_bits;
    int32_t amax_atomic;
    int32_t nb;
};
constexpr int CHAIN_MAX_BLOCKS = 1024;
int chain_blocks(int64_t M, int64_t N);
// q_t[k][n] = q[n][k] for an int8 matrix [N, pitch8(K)] (pad bytes of q_t zero); *s_out = *s_in
hipError_t launch_transpose_i8(const int8_t* q, int8_t* q_t, int64_t N, int64_t K, const float* s_in, float* s_out, hipStream_t s);
hipError_t launch_chain_combine(const ChainArgs& a, hipStream_t s);

// absmax of the local gradient of one layer: max_b |2 c[b]| * (float(vmax[b]) * s_y) -> slot[z], for nb passes (coefficients
// and maxima B apart, s_a one apart).
hipError_t launch_grad_amax(const float* coeff_total, const int32_t* vmax, const float* s_a, const float* s_w, int64_t B,
                            int nb, uint32_t* slot, hipStream_t s);

struct UpdateArgs {
    float* w;  // [N, K] contiguous
    int64_t N, K, lddw;
    int32_t n_terms;  // <= 4
    // accumulators of each term: the sum of splits[j] partial results, st_split elements apart (1: the accumulator itself)
    const int32_t* dw[4];
    int32_t splits[4];
    int64_t st_split;
    const float* s_g[4];
    const float* s_a[4];
    float lr;
    int32_t total_samples;
    // every workgroup stores the maximum of its new weights here (thousands of atomics on one word cost more than the rest
    // of an update); the quantiser that follows takes the maximum of the array (QuantArgs::amax_n)
    uint32_t* block_max;
    int32_t max_blocks;   // words at block_max
};
constexpr int UPDATE_MAX_BLOCKS = 1024;
int update_blocks(const UpdateArgs& a);   // workgroups launch_update starts
hipError_t launch_update(const UpdateArgs& a, hipStream_t s);

// ---- int8 contraction (gemm_i8.hip):  C[i][j] = sum_r P[i][r] * Q[j][r] -----------------------
struct GemmArgs {
    const int8_t* P;  // [I, ldp]
    const int8_t* Q;  // [J, ldq]
    int32_t* C;       // [I, ldc]
    int32_t I, J, R;  // R = reduction length in bytes (pad bytes beyond it are zero)
    int64_t ldp, ldq, ldc;
    // fused per-sample reductions (forward only; null gsum => plain contraction)
    unsigned long long* gsum;
    int32_t* vmax;
    int32_t rows_per_sample, relu, rshift;
    // nb problems in one launch: problem z = p * nc + c lies p strides st_* and c strides st_*2 further on (weight gradients:
    // pass p, sample chunk c; elsewhere nc = 1)
    int32_t nb, nc;
    int64_t st_p, st_q, st_c, st_g;
    int64_t st_p2, st_q2, st_c2;
    // split reduction (blockIdx.y): split s stores its partial sums at C + s*st_split; launch_reduce_splits
    // adds them up (integer sums: exact and order-free).  1 = no split.  Not combined with the fused reductions.
    int32_t splits;
    int64_t st_split;
    // implicit-GEMM convolution (conv != 0): P is an NHWC int8 tensor [B, H, W, cpitch] and row i of the
    // contraction is output pixel (b, ho, wo); reduction index r = (kh*ks + kw)*Cin + ci.  Cin is the channel count rounded
    // up to 16 (the pad channels of P are zero, so what Q holds at their place does not matter: it is the next tap's
    // weights), cin_out the real one, a multiple of 4: the tap stride of Q's rows.
    // conv == 2: Q is the NHWC int8 tensor [B, H, W, cpitch] itself, column j of C is (kh, kw, ci) and the reduction runs over
    // the output pixels of whole samples.  Cin is then the channel count rounded up to 16 (J = ks*ks*Cin) and cin_out the
    // real one: columns of the channels in between are not stored.
    int32_t conv, H, W, Cin, cpitch, ks, stride, pad, Ho, Wo;
    int32_t cin_out;
    int32_t adv_b, adv_h, adv_w;   // conv == 2, filled in by launch_gemm_nt_i8: images / rows / columns 128 pixels further on
    int64_t p_bytes;  // bytes of one implicit operand tensor (conv only; must be < 2^31)
    // log2 of C_in (conv == 1) when that is a power of two, else -1: the loader then indexes with shifts instead of
    // integer divisions.  Filled in by launch_gemm_nt_i8.
    int32_t cin_shift;
    // weight gradient and update in one launch (upd_w non-null; nb == 2 passes, no split, no fused reductions): C is not
    // written; the weights [I, J] (contiguous, 16-byte aligned, J % 4 == 0) are updated from the accumulators of both passes and
    // workgroup b leaves the largest magnitude of its new weights at upd_max[b]
    float* upd_w;
    const float* upd_s_g[2];
    const float* upd_s_a[2];
    float upd_lr;
    int32_t upd_samples;
    uint32_t* upd_max;
    // instrumentation (null normally): every workgroup adds the shader-clock cycles and the 100 MHz constant-clock
    // ticks it was alive to clk[0] and clk[1] (their ratio is the mean shader clock during the launch) and the
    // shader clocks of each tile by phase to clk[2..6] / clk[8..12]
    unsigned long long* clk;   // 16 counters, see ff_timing_clock_probe
    // residual layer, or null (implicit convolutions, no split, no fused reductions): C is not written, the block output is formed
    // from the accumulators.  [host] The kernels that form one take a copy behind these arguments (GemmResidualArgs); with it in every
    // launch's arguments the single operations of a forward pass, 128 -> 256 channels on 256 images of 16x16, took 74.5 us, 73.7 without
    const ResidualArgs* residual;
};
struct GemmResidualArgs : GemmArgs {
    ResidualArgs res;
};
hipError_t launch_gemm_nt_i8(const GemmArgs& a, hipStream_t s);
// workgroups of the launch with the fused update, or 0 where that is not the better way (see gemm_update_blocks)
int gemm_update_blocks(int64_t I, int64_t J, int64_t R);
int num_cus();   // compute units of the current device (256 when the query fails)
// register-resident MFMA loop (see ff_probe_mfma_ceiling): one workgroup of 512 threads per compute unit
hipError_t launch_mfma_ceiling(int32_t* sink, int iters, int kind, unsigned long long* clk, int* workgroups, hipStream_t s);
struct GemmPlan {
    int bm, bn, splits;
    int most_splits;   // splits at two workgroups per compute unit for every tile but 256 x 256: what scratch is sized for
};
// reduction_major: the launch is a GemmArgs::conv == 2 one
GemmPlan gemm_plan(int64_t I, int64_t J, int64_t R, int nb, bool allow_split, bool reduction_major);
constexpr int GEMM_TABLE_BYTES = 2048;   // LDS the reduction-major loader (conv == 2) takes beside the operand stages
int split_evenly(int64_t R, int64_t splits);   // at most `splits` shares of a reduction of R, none of them empty
// out[z][e] = sum over s < splits of part[z][s][e], e < n (n a multiple of 4); strides in elements
hipError_t launch_reduce_splits(const int32_t* part, int splits, int64_t st_split, int64_t st_part_z, int32_t* out,
                                int64_t st_out_z, int64_t n, int nb, hipStream_t s);

// ---- 3x3 stride-1 convolutions with resident weights (conv3.hip) --------------------------------------------------------
struct Conv3Geom {   // filled in by the launch: 16-byte chunks of a pixel, of a pixel in LDS, pixels and chunks of a window, ...
    int32_t cpp, pc, swz_mask, window, chunks, ncb, per;
};
bool conv3_ok(const GemmArgs& a);   // covers this implicit convolution, and there are enough tiles
hipError_t launch_conv3(const GemmArgs& a, hipStream_t s);

// ---- 3x3 stride-1 convolutions of more than 64 input channels (conv3_wide.hip) ----------------------------------------------
bool conv3_wide_ok(const GemmArgs& a);   // covers this implicit convolution, and is the better way
hipError_t launch_conv3_wide(const GemmArgs& a, hipStream_t s);
// dense contractions with few outputs (see gemm_few.hip); launch_gemm_nt_i8 has checked the arguments
bool gemm_few_ok(const GemmArgs& a);
hipError_t launch_gemm_few(const GemmArgs& a, hipStream_t s);

// ---- weight gradient of 3x3 convolutions from one input window per step (wgrad3.hip) --------------------------------------
struct ConvGeom {
    int32_t H, W, Cin, cpitch, ks, stride, pad, Ho, Wo;
};
// splits of the reduction of a launch over nb problems of R output pixels each, or 0 where it does not cover the layer (GemmArgs::conv == 2
// for the rest)
int wgrad3_splits(const ConvGeom& g, int64_t N, int64_t R, int nb);
int wgrad3_split_evenly(int64_t R, int64_t splits);   // at most `splits` shares of a reduction of R, none of them empty
hipError_t launch_wgrad3(const GemmArgs& a, const ConvGeom& g, hipStream_t s);

// ---- contraction of short rows without stored accumulators (rows.hip) ------------------------------------------------
// Rows P [I, ldp] x Q [J, ldq]^T over R <= ROWS_MAX_R bytes, nb passes (st_p, st_g apart), J a multiple of four.
constexpr int ROWS_MAX_R = 128;
enum RowsResult {
    ROWS_GOODNESS = 0,   // per-sample goodness sums and maxima into gsum, vmax (added to what is there)
    ROWS_HANDOFF = 1,    // codes of the activities, row-major: what launch_quantize(QSRC_HANDOFF) makes of the accumulators
    ROWS_GRAD = 2        // codes of the local gradient, transposed: what launch_quantize(QSRC_GRAD) makes of them
};
struct RowsArgs {
    const int8_t* P;
    const int8_t* Q;
    int64_t ldp, ldq, st_p;
    int32_t I, J, R, nb;
    int32_t rows_per_sample, relu, rshift;
    unsigned long long* gsum;
    int32_t* vmax;
    int64_t st_g;
};
hipError_t launch_rows(int what, const RowsArgs& r, const QuantArgs& a, hipStream_t s);

// ---- single-launch step of a small dense stack (fused.hip) ---------------------------------------------------------
constexpr int FU_MAX_LAYERS = 8;
constexpr int FU_THREADS = 512;
constexpr int FU_MAX_B = 2 * FU_THREADS;   // samples per pass
struct FusedLayer {
    int32_t K, N, relu, l2norm, train, rshift;
    float theta;
    float* w;      // fp32 master weights [N, K]
    int8_t* wq;    // [N, pitch8(K)]
    float* sw;
    // workspace of the step, two passes each (strides in elements of the respective type)
    int8_t* aq;    int64_t st_aq;    // quantised layer input [B, pitch8(K)]
    int8_t* aqt;   int64_t st_aqt;   // its transposed copy [K, pitch8(B)]
    int32_t* acc;  int64_t st_acc;   // accumulators [B, pitch32(N)]
    int8_t* gy;    int64_t st_gy;    // transposed int8 local gradient [N, pitch8(B)]
};
struct FusedArgs {
    int32_t k, B;
    float lambda, lr;
    uint64_t seed, step;
    uint64_t* step_dev;   // null: `step` is used
    int32_t advance;
    const float* x;       // positive set; the negative set is st_x elements further on
    int64_t st_x;
    uint32_t* wg_amax;    // [workgroups]: per-workgroup absmax of the net input
    uint32_t* w_amax;     // [k]
    unsigned long long* gsum;   // [k][2][B]
    int32_t* vmax;        // [k][2][B]
    float* s_a;           // [k][2]
    float* s_g;           // [k][2]
    float* c;             // [k][2][B]
    float* ct;            // [k][2][B]
    float* goodness;      // [k][2][B]
    float* loss;          // [k][2]
    unsigned* bar;        // device-wide barrier counters (filled in by the launcher)
    unsigned long long* stamps;   // instrumentation, see ff_timing_fused_stamps (null normally)
    FusedLayer L[FU_MAX_LAYERS];
};
hipError_t launch_fused_dense_step(const FusedArgs& a, int workgroups, hipStream_t s);

// ---- explicit im2col (conv.hip) ----------------------------------------------------------------------
struct Im2colArgs {
    const int8_t* a;  // NHWC int8 [B, H, W, cpitch]
    int8_t* out;      // [B*Ho*Wo, ld_out]
    ConvGeom g;
    int32_t K, B;
    int64_t ld_out;
    int32_t nb;
    int64_t st_a, st_out;
};
hipError_t launch_im2col(const Im2colArgs& p, hipStream_t s);
// ---- depthwise convolution (conv.hip): one ks x ks filter per channel, HBM-bound -----------------------------
struct DwArgs {
    const int8_t* a;    // NHWC int8 [B, H, W, cpitch]
    int64_t st_a;
    const int8_t* w_q;  // [C, 16]: nine taps (kh, kw) per channel, zero pad bytes
    ConvGeom g;         // Cin = C
    int32_t B;
    // forward
    int32_t* acc;       // [B*Ho*Wo, ldacc]
    int64_t ldacc, st_acc;
    unsigned long long* gsum;  // [B] per pass (stride st_g), zeroed; may be null
    int32_t* vmax;
    int64_t st_g;
    int32_t relu, rshift;
    // weight gradient over nc chunks of chunk_b samples each (the last may be shorter)
    const int8_t* gy;   // row-major int8 local gradient [B*Ho*Wo, ldg]
    int64_t ldg, st_gy;
    int32_t* dw;        // [C, 12] int32 per pass and chunk (st_dw, st_dw2 apart): splits partial results st_split apart, or
    int64_t st_dw, st_dw2, st_split;   // (st_split == 0) one zeroed accumulator
    int32_t nc, chunk_b, splits;
    int32_t nb;
};
int dwconv_wgrad_splits(const ConvGeom& g, int64_t chunk_b, int problems);
hipError_t launch_dwconv_forward(const DwArgs& p, hipStream_t s);
// a pass over a layer whose accumulators are not stored: `what` is a RowsResult, codes row-major either way
hipError_t launch_dwconv_rework(int what, const DwArgs& p, const QuantArgs& q, hipStream_t s);
bool dwconv_rework_pays(const ConvGeom& g, int64_t B);
hipError_t launch_dwconv_wgrad(const DwArgs& p, hipStream_t s);

}  // namespace ffi
