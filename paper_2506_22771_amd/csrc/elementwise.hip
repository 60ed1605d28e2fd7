// HBM-bound kernels of the FF-INT8 layer step for gfx950: absmax, the int8 quantiser in its three
// source flavours (fp32 tensor, hand-off from accumulators, local gradient from accumulators),
// goodness / loss, look-ahead, and the weight update.
//
// Numerics follow the paper's Section IV (symmetric uniform quantiser), Section IV-B (stochastic
// rounding of the layer input, int8 local gradient), Eq. (1)/(2) (losses) and Eq. (3)/(4)
// (look-ahead).  Every fp32 operation that decides an int8 code is a single correctly rounded IEEE
// operation in a fixed order; this file must be compiled with -ffp-contract=off.
#include <type_traits>

#include "ff_internal.hpp"
#include "device_math.hpp"

namespace ffi {

// Block-wide maximum of non-negative values' bit patterns, then one atomic per block.
template <int THREADS>
__device__ __forceinline__ void block_atomic_max_bits(uint32_t bits, uint32_t* slot)
{
    __shared__ uint32_t red[THREADS / 64];
    const uint32_t w = wave_max_u32(bits);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t m = red[0];
#pragma unroll
        for (int i = 1; i < THREADS / 64; ++i) m = max(m, red[i]);
        // thousands of workgroups target one word: skip the atomic when the slot already holds a larger value
        // (the slot only grows, so a stale read can only cause a harmless extra atomic)
        if (m != 0 && m > __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(slot, m);
    }
}

// The same, stored: one candidate per workgroup for the kernel that follows.
template <int THREADS>
__device__ __forceinline__ void block_store_max_bits(uint32_t bits, uint32_t* out)
{
    __shared__ uint32_t red[THREADS / 64];
    const uint32_t w = wave_max_u32(bits);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t m = red[0];
#pragma unroll
        for (int i = 1; i < THREADS / 64; ++i) m = max(m, red[i]);
        *out = m;
    }
}

// ------------------------------------------------------------------------------------------------
// fill
// ------------------------------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

__global__ void k_clear2_u32(uint32_t* p, int64_t n, uint32_t* p2, int64_t n2)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n + n2; i += stride)
        if (i < n) p[i] = 0u;
        else p2[i - n] = 0u;
}

hipError_t launch_clear2_u32(uint32_t* p, int64_t n, uint32_t* p2, int64_t n2, hipStream_t s)
{
    if (n + n2 <= 0) return hipSuccess;
    const int64_t blocks = min((n + n2 + 255) / 256, (int64_t)2048);
    hipLaunchKernelGGL(k_clear2_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, p2, n2);
    return hipGetLastError();
}

__global__ void k_advance_u64(uint64_t* counter)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) counter[0] += 1;
}

hipError_t launch_advance_u64(uint64_t* counter, hipStream_t s)
{
    hipLaunchKernelGGL(k_advance_u64, dim3(1), dim3(64), 0, s, counter);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// absmax of fp32 tensors (HBM-bound: 4 bytes read per element).  blockIdx.y selects the tensor (x + z*stride).  At most
// one workgroup per compute unit and tensor, each leaving its own candidate: no word to clear first and no atomics.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t absbits4(const float4 v)
{
    const uint32_t a = max(__float_as_uint(v.x) & 0x7FFFFFFFu, __float_as_uint(v.y) & 0x7FFFFFFFu);
    const uint32_t b = max(__float_as_uint(v.z) & 0x7FFFFFFFu, __float_as_uint(v.w) & 0x7FFFFFFFu);
    return max(a, b);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ldf4(const float4* p)   // streaming hint: the tensor is larger than the caches
{
    const f32x4 v = __builtin_nontemporal_load((const f32x4*)p);
    return make_float4(v.x, v.y, v.z, v.w);
}

constexpr int ABS_THREADS = 512;
__global__ __launch_bounds__(ABS_THREADS) void k_absmax_f32(const float* __restrict__ x0, int64_t st_x, int64_t n,
                                                            uint32_t* __restrict__ part, uint32_t* __restrict__ clear,
                                                            int64_t clear_n)
{
    for (int64_t i = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * ABS_THREADS + threadIdx.x; i < clear_n;
         i += (int64_t)gridDim.x * gridDim.y * ABS_THREADS)
        clear[i] = 0u;
    const float* __restrict__ x = x0 + (int64_t)blockIdx.y * st_x;
    // scalar head until 16-byte alignment, float4 body, scalar tail
    const uintptr_t addr = (uintptr_t)x;
    int64_t head = (int64_t)(((16 - (addr & 15)) & 15) >> 2);
    if (head > n) head = n;
    const int64_t nvec = (n - head) >> 2;
    const float4* __restrict__ xv = (const float4*)(x + head);
    const int64_t gtid = (int64_t)blockIdx.x * ABS_THREADS + threadIdx.x;
    uint32_t m = 0;
    // A workgroup walks contiguous spans, two of them per trip: eight 16-byte loads per thread in flight.  With four, the 256
    // workgroups of a large tensor ask for 32 KB per compute unit and do not fill HBM (ff_quantize of 16384 x 4096: 133 us,
    // with eight 102).
    constexpr int64_t SPAN = 4 * ABS_THREADS;
    const int64_t step = (int64_t)gridDim.x * SPAN;
    for (int64_t b = (int64_t)blockIdx.x * SPAN; b < nvec; b += 2 * step) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = b + (u >> 2) * step + (u & 3) * ABS_THREADS + threadIdx.x;
            v[u] = i < nvec ? ldf4(xv + i) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) m = max(m, absbits4(v[u]));
    }
    if (gtid < head) m = max(m, __float_as_uint(x[gtid]) & 0x7FFFFFFFu);
    const int64_t tail0 = head + (nvec << 2);
    if (tail0 + gtid < n) m = max(m, __float_as_uint(x[tail0 + gtid]) & 0x7FFFFFFFu);
    block_store_max_bits<ABS_THREADS>(m, part + blockIdx.y * ABSMAX_MAX_BLOCKS + blockIdx.x);
}

int absmax_blocks(int64_t n)
{
    const int64_t blocks = (n + ABS_THREADS * 16 - 1) / (ABS_THREADS * 16);
    return (int)max((int64_t)1, min((int64_t)ABSMAX_MAX_BLOCKS, blocks));
}

hipError_t launch_absmax(const float* x, int64_t st_x, int nb, int64_t n, uint32_t* part, hipStream_t s, uint32_t* clear,
                         int64_t clear_n)
{
    if (n <= 0) return launch_fill_u32(clear, clear_n, 0u, s);
    hipLaunchKernelGGL(k_absmax_f32, dim3((unsigned)absmax_blocks(n), (unsigned)nb), dim3(ABS_THREADS), 0, s, x, st_x, n, part,
                       clear, clear_n);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// quantiser
// ------------------------------------------------------------------------------------------------
// 16-byte load of data that is not read again soon (source tensors of the quantisers): a streaming hint keeps it
// from displacing what the next kernels will read
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_stream16(const void* p)
{
    const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)v, d), hi = (unsigned)__shfl_xor((int)(unsigned)(v >> 32), d);
        v += ((unsigned long long)hi << 32) | lo;
    }
    return v;
}

constexpr int QT_THREADS = 256;
// Tile of one workgroup: CB column blocks of four columns, U x (256 / CB) row blocks of four rows: 128 x 64 elements
// for CB = 16, 256 x 32 for CB = 8 (matrices of at most 32 columns: no idle column lanes, and with a row pitch of
// 32 columns or fewer the tile is one contiguous span of memory), both for U = 2.
template <int CB, int U> struct QTile {
    static constexpr int COLS = 4 * CB;
    static constexpr int RH = 4 * (QT_THREADS / CB);   // rows of one part of the tile (u < U)
    static constexpr int ROWS = U * RH;
    static constexpr int LDW = ROWS / 4 + 1;           // words per column in the transposed LDS tile (+1: bank spread)
    static constexpr int CHUNKS = ROWS / 16;           // 16-byte pieces of one transposed column
};

// Maximum over the workgroup, in every thread.  The barrier is a bare one behind the LDS write: __syncthreads() would wait for
// the loads of the source tensor, which are in flight across it.
__device__ __forceinline__ uint32_t workgroup_max(uint32_t v)
{
    __shared__ uint32_t red[QT_THREADS / 64];
    v = wave_max_u32(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    return max(max(red[0], red[1]), max(red[2], red[3]));
}
// ... of the n candidates a producer left, one per workgroup; four loads per thread in flight
__device__ __forceinline__ uint32_t max_of_candidates(const uint32_t* __restrict__ c, int n)
{
    uint32_t m = 0;
    for (int i0 = threadIdx.x; i0 < n; i0 += 4 * QT_THREADS) {
        uint32_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = c[i0 + e * QT_THREADS < n ? i0 + e * QT_THREADS : i0];
        m = max(m, max(max(v[0], v[1]), max(v[2], v[3])));
    }
    return workgroup_max(m);
}

// Each thread owns U 4x4 element blocks (rows 4*rb+j, cols 4*cb+c).  Codes are packed four columns
// to a word for q, byte-transposed in registers for q_t and regrouped through LDS so that q_t is
// written in 16-byte pieces.  All 4 U 16-byte loads of a thread are issued before any arithmetic.
// FORM 0: element loads (an fp32 source whose columns or base are not 16-byte friendly).  1: 16-byte loads (always legal
// for the int32 sources).  2: 16-byte loads and cols % 4 == 0, so that four neighbours share a hash head (sr_head4).
// Tensors have fewer than 2^32 elements (checked by the entry points), so the low word of the element index is the
// whole index.
// What bounds it: for tensors of tens of megabytes HBM, below that the vector ALUs and, for a few tiles per compute unit, the
// chain of a wavefront.  Hence: whole tiles take a body without bounds checks, row pointers advance by
// additions, and the sample of a row comes from one 32-bit division per four rows (local gradient of 2 x 8192 x 4096:
// 71 -> 64 us, 5.2 TB/s).  The loads of the tile go out first, those of the rows' factors and (RANGE_FIRST apart) of the range behind
// them, so that they are all in flight together; the rounding is done in fixed point where that is exact (device_math.hpp).  Local gradient of
// 2 x 1024 x 2000 10.6 -> 8.5 us, normalised hand-off 14.5 -> 12.4, requantised weights 7.1 -> 6.3; gradients of a
// MobileNet-shaped step 90 -> 76 us on average.
template <int SRC, bool STOCH, int FORM, int CB, int U, bool WHOLE>
__device__ __forceinline__ void quantize_tile(const QuantArgs& a, uint32_t* tileT, int bx, int by)
{
    constexpr int QT_ROWS = QTile<CB, U>::ROWS, QT_COLS = QTile<CB, U>::COLS, QT_LDW = QTile<CB, U>::LDW, QT_RH = QTile<CB, U>::RH;
    constexpr bool FX = SRC == QSRC_F32_FX, PLAIN = SRC == QSRC_F32 || FX;
    constexpr bool F32SRC = PLAIN || SRC == QSRC_F32_GRAD;   // the source is an fp32 tensor
    constexpr bool GRAD = SRC == QSRC_GRAD || SRC == QSRC_F32_GRAD, norm = SRC == QSRC_HANDOFF_NORM;
    const int z = blockIdx.z;
    const float* __restrict__ per_sample = a.per_sample ? a.per_sample + z * a.st_per_sample : nullptr;
    int8_t* __restrict__ q = a.q ? a.q + z * a.st_q : nullptr;
    int8_t* __restrict__ q_t = a.q_t ? a.q_t + z * a.st_qt : nullptr;

    // ---- range.  A vanishing one (absmax < 2^-100, all-zero tensor included) quantises to zero codes with scale 1
    uint32_t amax_word;
    auto range = [&] {
        amax_word = a.amax_bits ? a.amax_bits[z * a.st_amax] : 0u;
        if (a.amax_n > 1) amax_word = max_of_candidates(a.amax_bits + z * a.st_amax, a.amax_n);   // (uniform) one per workgroup of the producer
    };
    // Stochastic rounding of an fp32 tensor forms it before the tile's loads go out, every other form behind them: layer inputs
    // of 256 x 16 x 16 x 128 10.0 us behind and 9.4 first, of 154 x 28 x 28 x 120 21.3 and 19.6.
    constexpr bool RANGE_FIRST = SRC == QSRC_F32 && STOCH;
    if constexpr (RANGE_FIRST) range();

    const int64_t r0 = (int64_t)by * QT_ROWS;
    const int64_t c0 = (int64_t)bx * QT_COLS;
    const int t = threadIdx.x;
    const int cb = t & (CB - 1), rg = t / CB;
    const int64_t col = c0 + 4 * cb;
    const int64_t rowb = r0 + 4 * rg;
    const bool col_in = WHOLE || col < a.cols;
    auto row_in = [&](int dr) { return WHOLE || rowb + dr < a.rows; };

    // ---- loads: U blocks x 4 rows x 16 bytes, raw bits.  Row (u, j) of this thread is rowb + QT_RH*u + j.
    const int64_t ld = F32SRC ? a.cols : a.ldacc;
    const uint32_t* __restrict__ src =
        (F32SRC ? (const uint32_t*)(a.x + z * a.st_x) : (const uint32_t*)(a.acc + z * a.st_acc)) + rowb * ld + col;
    uint32_t raw[U][4][4];
    const bool ragged = FORM == 1 && (a.cols & 3) != 0;   // the int32 sources' pad columns hold junk: mask them at load
    // A tile that reaches beyond the matrix loads from its last row and first columns instead and drops what it got: with a
    // branch around every load each would wait for the one before (hand-off of 35322 x 224, every fourth tile of a row half
    // outside: 18.0 us with branches, 14.0 this way).
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t* __restrict__ ps = src + (u ? (int64_t)QT_RH * ld : 0);
        if (FORM != 0 && !WHOLE) ps -= (col_in ? 0 : col) + max((int64_t)0, rowb + QT_RH * u - (a.rows - 1)) * ld;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;
            const bool in = row_in(QT_RH * u + j) && col_in;
            if (FORM != 0) {
                const uint4 f = ld_stream16(ps);
                w0 = in ? f.x : 0u;
                w1 = in && !(ragged && col + 1 >= a.cols) ? f.y : 0u;
                w2 = in && !(ragged && col + 2 >= a.cols) ? f.z : 0u;
                w3 = in && !(ragged && col + 3 >= a.cols) ? f.w : 0u;
            } else if (in) {
                w0 = ps[0];
                if (col + 1 < a.cols) w1 = ps[1];
                if (col + 2 < a.cols) w2 = ps[2];
                if (col + 3 < a.cols) w3 = ps[3];
            }
            raw[u][j][0] = w0; raw[u][j][1] = w1; raw[u][j][2] = w2; raw[u][j][3] = w3;
            ps += FORM == 0 || row_in(QT_RH * u + j + 1) ? ld : 0;
        }
    }
    // ---- what the rows' factors are made of: one load per row, all of them in flight
    float rowf[U][4];
    unsigned long long rows[U][4];
    if (GRAD || norm) {
        const uint32_t rps = (uint32_t)a.rows_per_sample, last = (uint32_t)a.rows - 1u;
        uint32_t smp[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t rfirst = WHOLE ? (uint32_t)rowb + QT_RH * u : min((uint32_t)rowb + QT_RH * u, last);
            smp[u][0] = rfirst;
            uint32_t rem = 0;
            if (rps != 1) {
                smp[u][0] = rfirst / rps;
                rem = rfirst - smp[u][0] * rps;
            }
#pragma unroll
            for (int j = 1; j < 4; ++j) {
                smp[u][j] = smp[u][j - 1];
                if (row_in(QT_RH * u + j) && ++rem >= rps) { rem = 0; ++smp[u][j]; }
            }
        }
        if (norm && a.gsum) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) rows[u][j] = a.gsum[z * a.st_b + smp[u][j]];
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) rowf[u][j] = per_sample[smp[u][j]];
        }
    }

    if constexpr (!RANGE_FIRST) range();
    float s_y = 1.0f;
    if (!F32SRC) s_y = a.s_a[z * a.st_s_a] * a.s_w[z * a.st_s_w];
    const double s_yd = (double)s_y, pow2r = (double)(1ull << a.rshift);
    if ((SRC == QSRC_HANDOFF || norm) && a.vmax) {   // (uniform) straight from the contraction's per-sample maxima (and sums)
        const int32_t* vm = a.vmax + z * a.st_b;
        const unsigned long long* gs = a.gsum + z * a.st_b;
        // (four samples at a time, all loads before the arithmetic; beyond the batch: a sample of this thread's once more)
        uint32_t mm = 0;
        for (int i0 = threadIdx.x; i0 < a.B; i0 += 4 * QT_THREADS) {
            int i[4];
            int32_t v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                i[e] = i0 + e * QT_THREADS < a.B ? i0 + e * QT_THREADS : i0;
                v[e] = vm[i[e]];
            }
            if (norm) {
                unsigned long long g[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = gs[i[e]];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float nrm = sqrtf(goodness_value(g[e], pow2r, s_yd));
                    mm = max(mm, __float_as_uint(nrm > 0.0f ? ((float)v[e] * s_y) / nrm : 0.0f));
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) mm = max(mm, (uint32_t)v[e]);
            }
        }
        mm = workgroup_max(mm);
        amax_word = norm ? mm : __float_as_uint((float)(int)mm * s_y);
    }
    if (SRC == QSRC_GRAD && a.vmax) {   // (uniform) the absmax of the gradient, from the per-sample factors and maxima
        const int32_t* vm = a.vmax + z * a.st_b;
        uint32_t mm = 0;
        for (int i0 = threadIdx.x; i0 < a.B; i0 += 4 * QT_THREADS) {
            int32_t v[4];
            float ct[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = i0 + e * QT_THREADS < a.B ? i0 + e * QT_THREADS : i0;
                v[e] = vm[i];
                ct[e] = per_sample[i];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) mm = max(mm, __float_as_uint(fabsf(2.0f * ct[e]) * ((float)v[e] * s_y)));
        }
        amax_word = workgroup_max(mm);
    }
    // ---- per-row factor (local gradients: 2*coeff; normalised hand-off: sqrt(goodness) and its reciprocal)
    if (GRAD || norm) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (norm && a.gsum) rowf[u][j] = goodness_value(rows[u][j], pow2r, s_yd);
                rowf[u][j] = !row_in(QT_RH * u + j) ? 0.0f : (GRAD ? 2.0f * rowf[u][j] : sqrtf(rowf[u][j]));
            }
    }

    const float amax = __uint_as_float(amax_word);
    const bool live = amax >= 0x1p-100f;
    const float inv = live ? 127.0f / amax : 0.0f;
    if (blockIdx.x == 0 && blockIdx.y == 0 && t == 0) a.scale[z * a.st_scale] = live ? amax / 127.0f : 1.0f;
    const float floor_y = a.relu ? 0.0f : -__builtin_inff();
    SrKey key = z ? a.key2 : a.key;
    if (a.step_dev) key = make_sr_key(a.seed, stream_tag_of(a.step_dev[0], a.tag_layer, (uint32_t)z, a.tag_kind));
    // (the smallest nonzero activity is s_y, the largest 2^31 s_y: with these bounds every quotient and remainder is normal)
    const bool plain_range = s_y > 0x1p-40f && s_y < 0x1p40f;

    // fixed-point rounding where no t is a NaN and its sign is known per row (or taken from t): a finite range, of activities that
    // have not overflowed themselves.  A finite range makes the factors and everything that counts for it finite.  Negative
    // activities do not count: times a row's factor, over a small norm or times inv they may become infinite, but not NaN (inv is neither
    // zero nor infinite), and the bound on their side is zero.
    // (Half-size tiles of an fp32 tensor, which has no sign known beforehand, in floating point: 1000 x 784 4.4 us, 4.7 with the fixed form.)
    constexpr bool MAY_FIX = STOCH && !(SRC == QSRC_F32 && U == 1);
    const bool fixed = MAY_FIX && live && amax < __builtin_inff() && (PLAIN || a.relu) && (F32SRC || s_y < 0x1p80f);

    // ---- quantise
    const uint32_t idx0 = (uint32_t)rowb * (uint32_t)a.cols + (uint32_t)col;   // element index of (row rowb, col)
    int8_t* __restrict__ pq0 = q ? q + rowb * a.ldq + col : nullptr;
    auto codes = [&](auto form) {
    constexpr bool FIXED = decltype(form)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint32_t rowpack[4];
        uint32_t idx = idx0 + (uint32_t)(QT_RH * u) * (uint32_t)a.cols;
        int8_t* __restrict__ pq = pq0 + (u ? (int64_t)QT_RH * a.ldq : 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t w[4];
            if (STOCH) {
                if (FORM == 2) {
                    sr_head4(idx ^ key.k0, w);
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) w[c] = sr_head((idx + (uint32_t)c) ^ key.k0);
                }
            }
            float v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                v[c] = F32SRC ? __uint_as_float(raw[u][j][c]) : (float)(int)raw[u][j][c];
                if (!F32SRC) v[c] = v[c] * s_y;
                if (!F32SRC && !FIXED) v[c] = fmaxf(v[c], floor_y);   // (the fixed-point rounding rectifies with its bounds)
                if (GRAD) v[c] = rowf[u][j] * v[c];
            }
            if (norm) {
                const float d = rowf[u][j];
                if (plain_range && d > 0x1p-40f && d < 0x1p40f && a.relu) {
                    const float y = 1.0f / d;
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] = div_by_reciprocal(v[c], d, y);
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] = d > 0.0f ? v[c] / d : 0.0f;
                }
            }
            // elements outside the tensor were loaded as zero and a dead range has inv == 0: in both
            // cases t == 0, so the code is 0 in either rounding mode without any masking
            if constexpr (FIXED) {
                uint32_t top[4];
                // a rectified source: t has the sign of the row's factor, or of nothing at all
                const bool down = GRAD && rowf[u][j] < 0.0f;
                const float one = down ? 1.0f : 0.0f;
                const float lo = PLAIN || !down ? -SR_MOST : 0.0f, hi = PLAIN || down ? SR_MOST : 0.0f;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float t = v[c] * inv;
                    const float scaled = PLAIN ? sr_scale(t, sr_one_if_negative(t)) : (GRAD ? sr_scale(t, one) : t * -0x1p24f);
                    top[c] = sr_top(scaled, lo, hi, w[c]);
                }
                rowpack[j] = sr_pack(top[0], top[1], top[2], top[3]);
            } else {
                int code[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) code[c] = quant_code_of_word<STOCH>(v[c], inv, STOCH ? w[c] ^ (w[c] >> 16) : 0u);
                const uint32_t lo = __builtin_amdgcn_perm((uint32_t)code[1], (uint32_t)code[0], 0x0C0C0400u);
                const uint32_t hi = __builtin_amdgcn_perm((uint32_t)code[3], (uint32_t)code[2], 0x04000C0Cu);
                rowpack[j] = lo | hi;
            }
            if (q && row_in(QT_RH * u + j) && (WHOLE || col < a.ldq)) *(uint32_t*)pq = rowpack[j];
            idx += (uint32_t)a.cols;
            pq += a.ldq;
        }
        if (q_t) {
            // 4x4 byte transpose: column word c = byte c of rowpack[0..3]
            const int rb = rg + (QT_THREADS / CB) * u;
            const uint32_t t0 = __builtin_amdgcn_perm(rowpack[1], rowpack[0], 0x05010400u);
            const uint32_t t1 = __builtin_amdgcn_perm(rowpack[1], rowpack[0], 0x07030602u);
            const uint32_t t2 = __builtin_amdgcn_perm(rowpack[3], rowpack[2], 0x05010400u);
            const uint32_t t3 = __builtin_amdgcn_perm(rowpack[3], rowpack[2], 0x07030602u);
            tileT[(4 * cb + 0) * QT_LDW + rb] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
            tileT[(4 * cb + 1) * QT_LDW + rb] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
            tileT[(4 * cb + 2) * QT_LDW + rb] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
            tileT[(4 * cb + 3) * QT_LDW + rb] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
        }
    }
    };
    if constexpr (MAY_FIX) {
        if (fixed) codes(std::true_type{});   // (uniform)
        else codes(std::false_type{});
    } else {
        codes(std::false_type{});
    }
    if constexpr (FX) {
        // The goodness sums of the tensor at hand (the output of a residual block), in the fixed point of k_goodness_fx: per element
        // floor(r r 2^40), r = y / amax.  Products and sums of a thread are exact in fp64 (24-bit factors, at most 32 terms).
        const float fx_inv = live ? 1.0f / amax : 0.0f;
        const uint32_t rps = (uint32_t)a.rows_per_sample, last = (uint32_t)a.rows - 1u;
        unsigned long long* const gs = a.fx_gsum + z * a.st_b;
        if (blockIdx.x == 0 && blockIdx.y == 0 && t == 0) a.fx_amax[z] = amax_word;
        double sum[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sum[u][j] = 0.0;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double r = (double)(__uint_as_float(raw[u][j][c]) * fx_inv);
                    sum[u][j] += __builtin_trunc(r * r * 0x1p40);
                }
            }
        // (a tile may begin beyond the tensor, where the pitch of q_t does: nothing but zeros)
        const uint32_t s0 = min((uint32_t)r0, last) / rps, s1 = min((uint32_t)r0 + QT_ROWS - 1u, last) / rps;
        if (s0 == s1) {   // (uniform) one atomic per tile
            double w = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) w += (sum[u][0] + sum[u][1]) + (sum[u][2] + sum[u][3]);
            const unsigned long long part = wave_sum_u64((unsigned long long)w);
            __shared__ unsigned long long reds[QT_THREADS / 64];
            if ((t & 63) == 0) reds[t >> 6] = part;
            __syncthreads();
            if (t == 0) atomicAdd(gs + s0, (reds[0] + reds[1]) + (reds[2] + reds[3]));
        } else {
            // The CB lanes of a row, or of four rows of one sample, meet and add to their sample's word in LDS; one global atomic per
            // sample of the tile.  Per row they meet in a few cache lines at 2 to 4 ns each: 256 channels on 7x7 maps of 38 images
            // (two passes) 35.8 us, 5.6 this way.
            __shared__ unsigned long long part[QT_ROWS];
            for (int i = t; i < QT_ROWS; i += QT_THREADS) part[i] = 0;
            __syncthreads();
            const bool fours = (rps & 3u) == 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (fours) sum[u][0] = (sum[u][0] + sum[u][1]) + (sum[u][2] + sum[u][3]);
                for (int j = 0; j < (fours ? 1 : 4); ++j) {
                    unsigned long long v = (unsigned long long)(j == 0 ? sum[u][0] : j == 1 ? sum[u][1] : j == 2 ? sum[u][2] : sum[u][3]);
#pragma unroll
                    for (int d = 1; d < CB; d <<= 1) {
                        const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)v, d), hi = (unsigned)__shfl_xor((int)(unsigned)(v >> 32), d);
                        v += ((unsigned long long)hi << 32) | lo;
                    }
                    if (cb == 0 && v) atomicAdd(part + (min((uint32_t)rowb + QT_RH * u + j, last) / rps - s0), v);
                }
            }
            __syncthreads();
            for (uint32_t i = t; i <= s1 - s0; i += QT_THREADS)
                if (part[i]) atomicAdd(gs + s0 + i, part[i]);
        }
    }
    if (q_t) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = t + QT_THREADS * u;
            const int cl = e / QTile<CB, U>::CHUNKS, ch = e % QTile<CB, U>::CHUNKS;
            const int64_t oc = c0 + cl;
            const int64_t orow = r0 + 16 * ch;
            if ((WHOLE || oc < a.cols) && orow < a.ldqt) {
                u32x4 o;
                o.x = tileT[cl * QT_LDW + 4 * ch + 0];
                o.y = tileT[cl * QT_LDW + 4 * ch + 1];
                o.z = tileT[cl * QT_LDW + 4 * ch + 2];
                o.w = tileT[cl * QT_LDW + 4 * ch + 3];
                // the transposed copy of a layer input is read by the weight-gradient contraction much later
                // (streaming store); that of a local gradient right away
                if (a.qt_streaming) __builtin_nontemporal_store(o, (u32x4*)(q_t + oc * a.ldqt + orow));
                else *(u32x4*)(q_t + oc * a.ldqt + orow) = o;
            }
        }
    }
}

template <int SRC, bool STOCH, int FORM, int CB, int U>
__global__ __launch_bounds__(QT_THREADS) void k_quantize(QuantArgs a)
{
    __shared__ uint32_t tileT[QTile<CB, U>::COLS * QTile<CB, U>::LDW];
    int bx = blockIdx.x, by = blockIdx.y;
    if (U == 2 && a.row_per_xcd) {   // (see launch_quantize_tiles; the last rows, fewer than eight, stay as they are)
        const uint32_t id = blockIdx.y * gridDim.x + blockIdx.x;
        if (id < (gridDim.y & ~7u) * gridDim.x) {
            by = (int)((id >> 3) / gridDim.x * 8 + (id & 7));
            bx = (int)((id >> 3) % gridDim.x);
        }
    }
    const bool whole = (int64_t)(by + 1) * QTile<CB, U>::ROWS <= a.rows && (int64_t)(bx + 1) * QTile<CB, U>::COLS <= a.cols;
    if (whole) quantize_tile<SRC, STOCH, FORM, CB, U, true>(a, tileT, bx, by);
    else quantize_tile<SRC, STOCH, FORM, CB, U, false>(a, tileT, bx, by);
}

// fp32 tensors of at most four columns, row-major codes only (the pixels of a first layer: one or three channels, 16 bytes
// of codes per pixel): a thread takes a row.  In the tiles above fifteen of sixteen lanes would have nothing to do
// (3 channels, 32x32 maps, 512 images: 25 us there, 7 us here).
template <bool STOCH>
__global__ __launch_bounds__(QT_THREADS) void k_quantize_pixels(QuantArgs a)
{
    const int z = blockIdx.y;
    uint32_t amax_word = a.amax_bits[z * a.st_amax];
    if (a.amax_n > 1) amax_word = max_of_candidates(a.amax_bits + z * a.st_amax, a.amax_n);   // (uniform) one per workgroup of the producer
    const float amax = __uint_as_float(amax_word);
    const bool live = amax >= 0x1p-100f;
    const float inv = live ? 127.0f / amax : 0.0f;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.scale[z * a.st_scale] = live ? amax / 127.0f : 1.0f;
    SrKey key = z ? a.key2 : a.key;
    if (a.step_dev) key = make_sr_key(a.seed, stream_tag_of(a.step_dev[0], a.tag_layer, (uint32_t)z, a.tag_kind));
    const int cols = (int)a.cols;
    for (int64_t row = (int64_t)blockIdx.x * QT_THREADS + threadIdx.x; row < a.rows; row += (int64_t)gridDim.x * QT_THREADS) {
        const float* px = a.x + z * a.st_x + row * cols;
        const uint32_t idx = (uint32_t)row * (uint32_t)cols;
        float v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = c < cols ? px[c] : 0.0f;
        uint32_t pack = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c < cols) pack |= ((uint32_t)quant_code<STOCH>(v[c], inv, (idx + (uint32_t)c) ^ key.k0) & 0xFFu) << (8 * c);
        *(u32x4*)(a.q + z * a.st_q + row * a.ldq) = (u32x4){pack, 0u, 0u, 0u};   // (the row pitch of up to four columns is 16)
    }
}

template <int SRC, bool STOCH, int FORM, int CB, int U>
static void launch_quantize_tiles(QuantArgs a, int64_t span, hipStream_t s)
{
    // Rows of the source, or of the codes, that do not start on 128-byte lines: two neighbouring tiles of a row of tiles share
    // a line of every row.  Workgroups go to the eight XCDs in turn, so the line would be fetched into, or written back from,
    // two L2s; with a row of tiles on one XCD it is one.  Local gradient of 65536 x 1000: backward 132 -> 114 us, x 500:
    // 88 -> 79, 40000 x 2000: 142 -> 122; hand-off of 35322 x 224 with its transposed copy 14.0 -> 11.5, of 16384 x 1000
    // 25.5 -> 20.5.  Rows that start on lines keep the plain order (a normalised hand-off of 8192 x 4096: 36 us, 40 this way).
    constexpr bool F32SRC = SRC == QSRC_F32 || SRC == QSRC_F32_GRAD || SRC == QSRC_F32_FX;
    a.row_per_xcd = (((F32SRC ? a.cols : a.ldacc) & 31) != 0 || (a.q && (a.ldq & 127) != 0)) && span > QTile<CB, U>::COLS;
    // (row tiles up to the row pitch of q_t, for the same reason)
    const int64_t rspan = a.q_t && a.ldqt > a.rows ? a.ldqt : a.rows;
    const dim3 grid((unsigned)((span + QTile<CB, U>::COLS - 1) / QTile<CB, U>::COLS),
                    (unsigned)((rspan + QTile<CB, U>::ROWS - 1) / QTile<CB, U>::ROWS), (unsigned)a.nb);
    hipLaunchKernelGGL((k_quantize<SRC, STOCH, FORM, CB, U>), grid, dim3(QT_THREADS), 0, s, a);
}

template <int SRC, bool STOCH>
static void launch_quantize_t(const QuantArgs& a, hipStream_t s)
{
    constexpr bool F32SRC = SRC == QSRC_F32 || SRC == QSRC_F32_GRAD || SRC == QSRC_F32_FX;
    constexpr int GENERAL = F32SRC ? 0 : 1;
    if (SRC == QSRC_F32 && a.cols <= 4 && a.q && !a.q_t) {
        const int64_t blocks = min((a.rows + QT_THREADS - 1) / QT_THREADS, (int64_t)8 * num_cus());
        hipLaunchKernelGGL((k_quantize_pixels<STOCH>), dim3((unsigned)blocks, (unsigned)a.nb), dim3(QT_THREADS), 0, s, a);
        return;
    }
    const bool cols4 = (a.cols & 3) == 0;
    const bool vec = !F32SRC || (cols4 && (((uintptr_t)a.x) & 15) == 0 && ((a.st_x & 3) == 0 || a.nb == 1));
    const bool narrow = a.cols <= QTile<8, 2>::COLS && vec;
    // (column tiles up to the row pitch of q, so that its pad bytes are written too: zeros)
    const int64_t span = a.q && a.ldq > a.cols ? a.ldq : a.cols;
    // Tensors that would give a compute unit fewer than four tiles of two blocks per thread are bound by the latency of one
    // wavefront's chain (loads, hash, stores), not by HBM: half the tile, twice the wavefronts (steps of 784-2000^4 at
    // 1024 samples 302 -> 290 us, 1000-1500^2-1001 with the chain 284 -> 267 us).  At five and more the whole tile is better, whose
    // transposed stores are whole lines: hand-off with the transposed copy, halves against whole tiles, 65536 x 128
    // 13.0 -> 11.0 us, 16384 x 500 13.5 -> 11.0, 8000 x 1500 19.3 -> 15.6; at 860 tiles (5493 x 1232) 11.7 and 10.7 with, 8.9
    // and 9.1 without the copy.
    constexpr int64_t Q_FEW = 4;
    const int64_t tiles = narrow ? (a.rows + QTile<8, 2>::ROWS - 1) / QTile<8, 2>::ROWS
                                 : ((span + QTile<16, 2>::COLS - 1) / QTile<16, 2>::COLS) * ((a.rows + QTile<16, 2>::ROWS - 1) / QTile<16, 2>::ROWS);
    const bool few = tiles * a.nb < Q_FEW * num_cus() && (a.rows + 127) / QTile<16, 1>::ROWS < 65535;   // (grid.y)
    if (narrow) {
        if (cols4 && few) launch_quantize_tiles<SRC, STOCH, 2, 8, 1>(a, QTile<8, 1>::COLS, s);
        else if (cols4) launch_quantize_tiles<SRC, STOCH, 2, 8, 2>(a, QTile<8, 2>::COLS, s);
        else if constexpr (!F32SRC) launch_quantize_tiles<SRC, STOCH, 1, 8, 2>(a, QTile<8, 2>::COLS, s);
    } else if (vec && cols4) {
        if (few) launch_quantize_tiles<SRC, STOCH, 2, 16, 1>(a, span, s);
        else launch_quantize_tiles<SRC, STOCH, 2, 16, 2>(a, span, s);
    } else if constexpr (SRC != QSRC_F32_FX) {
        if (few) launch_quantize_tiles<SRC, STOCH, GENERAL, 16, 1>(a, span, s);
        else launch_quantize_tiles<SRC, STOCH, GENERAL, 16, 2>(a, span, s);
    }
}

hipError_t launch_quantize(int src, const QuantArgs& a, hipStream_t s)
{
    if (a.rows <= 0 || a.cols <= 0) return hipSuccess;
    const bool st = a.round_mode == FF_ROUND_STOCHASTIC;
    switch (src) {
        case QSRC_F32_FX:   // (block outputs are 16-byte aligned rows of a multiple of four columns)
            if ((a.cols & 3) != 0 || (((uintptr_t)a.x) & 15) != 0 || (a.st_x & 3) != 0 || !st || !a.fx_gsum || !a.fx_amax || a.rows_per_sample < 1)
                return hipErrorInvalidValue;
            launch_quantize_t<QSRC_F32_FX, true>(a, s);
            break;
        case QSRC_F32:
            if (st) launch_quantize_t<QSRC_F32, true>(a, s);
            else launch_quantize_t<QSRC_F32, false>(a, s);
            break;
        case QSRC_HANDOFF:
            if (a.l2norm && st) launch_quantize_t<QSRC_HANDOFF_NORM, true>(a, s);
            else if (a.l2norm) launch_quantize_t<QSRC_HANDOFF_NORM, false>(a, s);
            else if (st) launch_quantize_t<QSRC_HANDOFF, true>(a, s);
            else launch_quantize_t<QSRC_HANDOFF, false>(a, s);
            break;
        case QSRC_F32_GRAD:
            if (st) launch_quantize_t<QSRC_F32_GRAD, true>(a, s);
            else launch_quantize_t<QSRC_F32_GRAD, false>(a, s);
            break;
        default:
            if (st) launch_quantize_t<QSRC_GRAD, true>(a, s);
            else launch_quantize_t<QSRC_GRAD, false>(a, s);
            break;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// goodness, loss, dL/dG, absmax of the hand-off tensor: one workgroup per pass, fixed reduction order
// ------------------------------------------------------------------------------------------------
constexpr int GL_THREADS = 1024;

__global__ __launch_bounds__(GL_THREADS) void k_goodness_loss(GoodnessArgs a)
{
    const int z = blockIdx.x;
    const unsigned long long* gsum = a.gsum + z * a.st_b;
    const int32_t* vmax = a.vmax + z * a.st_b;
    float* goodness = a.goodness + z * a.st_b;
    float* coeff = a.coeff + z * a.st_b;
    const int sign = z ? -a.pass_sign : a.pass_sign;
    const bool fx = a.fx_amax_bits != nullptr;
    const float s_y = fx ? 1.0f : a.s_a[z * a.st_scalar] * a.s_w[0];
    const float fx_amax = fx ? __uint_as_float(a.fx_amax_bits[z * a.st_scalar]) : 0.0f;
    const double s_yd = fx ? (double)fx_amax : (double)s_y;
    const double pow2r = fx ? 0x1p-40 : (double)(1ull << a.rshift);

    double lsum = 0.0;
    uint32_t amax_bits = 0;
    const int wg = blockIdx.y, nwg = gridDim.y;
    for (int64_t b = (int64_t)wg * GL_THREADS + threadIdx.x; b < a.B; b += (int64_t)nwg * GL_THREADS) {
        const float G = (fx && fx_amax < 0x1p-100f) ? 0.0f : goodness_value(gsum[b], pow2r, s_yd);
        goodness[b] = G;
        float xs;
        coeff[b] = loss_derivative(G - a.theta, sign, xs);
        lsum += (double)loss_term(xs);   // fp32 terms, summed in fp64
        if (a.next_amax_bits) {
            float ymax = (float)vmax[b] * s_y;
            if (a.l2norm) {
                const float nrm = sqrtf(G);
                ymax = nrm > 0.0f ? ymax / nrm : 0.0f;
            }
            amax_bits = max(amax_bits, __float_as_uint(ymax));
        }
    }
    __shared__ double red[GL_THREADS];
    __shared__ uint32_t redm[GL_THREADS];
    red[threadIdx.x] = lsum;
    redm[threadIdx.x] = amax_bits;
    __syncthreads();
    for (int s = GL_THREADS / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            red[threadIdx.x] += red[threadIdx.x + s];
            redm[threadIdx.x] = max(redm[threadIdx.x], redm[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (nwg == 1) {
            a.loss_mean[z * a.st_scalar] = a.B > 0 ? (float)(red[0] / (double)a.B) : 0.0f;
            if (a.next_amax_bits) a.next_amax_bits[z * a.st_scalar] = redm[0];
        } else {
            if (a.next_amax_bits && redm[0]) atomicMax(a.next_amax_bits + z * a.st_scalar, redm[0]);
            unsigned long long* part = a.loss_part + z * GL_MAX_WG;
            __hip_atomic_store(part + wg, (unsigned long long)__double_as_longlong(red[0]), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __threadfence();
            if (atomicAdd(a.wg_counter + z, 1u) == (unsigned)(nwg - 1)) {
                // last workgroup of this pass: every partial sum has been published; add them in index order
                __threadfence();
                double t = 0.0;
                for (int i = 0; i < nwg; ++i)
                    t += __longlong_as_double((long long)__hip_atomic_load(part + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                a.loss_mean[z * a.st_scalar] = (float)(t / (double)a.B);
                __hip_atomic_store(a.wg_counter + z, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

hipError_t launch_goodness_loss(const GoodnessArgs& a, hipStream_t s)
{
    // one workgroup of 1024 threads per pass, or (large batches, scratch given) one per 1024 samples
    int nwg = 1;
    if (a.loss_part && a.wg_counter && a.B >= 2 * GL_THREADS) nwg = (int)min((int64_t)GL_MAX_WG, (a.B + GL_THREADS - 1) / GL_THREADS);
    hipLaunchKernelGGL(k_goodness_loss, dim3((unsigned)a.nb, (unsigned)nwg), dim3(GL_THREADS), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// residual layers: block output y = act(fp32(acc) * s_y + skip), one rounding per operation, stored as
// fp32; max|y| per sample and over the pass (bit patterns, atomic max).  A thread owns four columns.
// ------------------------------------------------------------------------------------------------
// Work split of the two residual kernels: blockIdx.y = sample, blockIdx.x = a contiguous share of the sample's
// terms (RES_VPT four-element vectors per thread), blockIdx.z = pass.  A workgroup therefore reduces for ONE
// sample and issues one atomic.
constexpr int RES_VPT = 4;

template <typename T, typename F>
__device__ __forceinline__ T block_reduce_256(T v, F op, T* red)
{
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return op(op(red[0], red[1]), op(red[2], red[3]));
}

__global__ __launch_bounds__(256) void k_residual_act(ResidualArgs a)
{
    const int z = blockIdx.z;
    const int64_t smp = blockIdx.y;
    const int N = (int)a.N;
    const int tv = a.rows_per_sample * (N >> 2);   // vectors per sample
    const float s_y = a.s_a[z * a.st_s_a] * a.s_w[0];
    const float s_u = a.skip == FF_SKIP_IDENTITY ? a.s_x[z * a.st_s_x] : a.s_ap[z * a.st_s_ap] * a.s_wp[0];
    const int64_t row0 = smp * a.rows_per_sample;
    uint32_t m = 0;
#pragma unroll
    for (int it = 0; it < RES_VPT; ++it) {
        const int v = ((int)blockIdx.x * RES_VPT + it) * 256 + (int)threadIdx.x;
        if (v >= tv) break;
        const int e = v * 4;
        const int r = e / N, col = e - r * N;
        const int64_t row = row0 + r;
        // the accumulators of a residual layer are not read again (everything downstream uses y): streaming hint
        const uint4 cw = ld_stream16(a.acc + z * a.st_acc + row * a.ldacc + col);
        const int4 c = make_int4((int)cw.x, (int)cw.y, (int)cw.z, (int)cw.w);
        float u[4];
        if (a.skip == FF_SKIP_IDENTITY) {
            const uint32_t xw = *(const uint32_t*)(a.xq + z * a.st_xq + row * a.ldx + col);
#pragma unroll
            for (int q = 0; q < 4; ++q) u[q] = (float)(int)(int8_t)(xw >> (8 * q)) * s_u;
        } else {
            const int4 cp = *(const int4*)(a.accp + z * a.st_accp + row * a.ldaccp + col);
            u[0] = (float)cp.x * s_u; u[1] = (float)cp.y * s_u; u[2] = (float)cp.z * s_u; u[3] = (float)cp.w * s_u;
        }
        const int cc[4] = {c.x, c.y, c.z, c.w};
        float yv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float t = (float)cc[q] * s_y;
            float w = t + u[q];
            if (a.relu) w = fmaxf(w, 0.0f);
            yv[q] = w;
            m = max(m, __float_as_uint(fabsf(w)));
        }
        *(float4*)(a.y + z * a.st_y + row * N + col) = make_float4(yv[0], yv[1], yv[2], yv[3]);
    }
    __shared__ uint32_t red[4];
    const uint32_t bm = block_reduce_256(wave_max_u32(m), [](uint32_t x, uint32_t y) { return max(x, y); }, red);
    if (threadIdx.x == 0 && bm) atomicMax(a.ymax_bits + z * a.st_b + smp, bm);
}

hipError_t launch_residual_act(const ResidualArgs& a, hipStream_t s)
{
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    const int64_t tv = (int64_t)a.rows_per_sample * (a.N >> 2);
    const int64_t B = a.M / a.rows_per_sample;
    const unsigned bx = (unsigned)((tv + 256 * RES_VPT - 1) / (256 * RES_VPT));
    if (B > 65535 || tv > (int64_t(1) << 28)) return hipErrorInvalidValue;   // grid y limit; 32-bit in-sample offsets
    hipLaunchKernelGGL(k_residual_act, dim3(bx, (unsigned)B, (unsigned)a.nb), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Fixed-point goodness sums of an fp32 activity tensor: per element floor(r * r * 2^40), r = y * (1 / amax) in
// fp32, the product in fp64 (exact); unsigned 64-bit integer sums per sample (order-free).  amax is the maximum
// of the per-sample maxima, recomputed by every workgroup; workgroup (0, 0) of a pass also stores it to the slot
// the quantisers of the next layers read.
__global__ __launch_bounds__(256) void k_goodness_fx(GoodnessFxArgs a)
{
    const int z = blockIdx.z;
    const int64_t smp = blockIdx.y;
    const int64_t B = gridDim.y;
    __shared__ uint32_t redm[4];
    __shared__ unsigned long long reds[4];
    uint32_t mb = 0;
    for (int64_t b = threadIdx.x; b < B; b += 256) mb = max(mb, a.ymax_bits[z * a.st_b + b]);
    mb = block_reduce_256(wave_max_u32(mb), [](uint32_t x, uint32_t y) { return max(x, y); }, redm);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) a.amax_bits[z * a.st_amax] = mb;
    const float amax = __uint_as_float(mb);
    const float inv = amax >= 0x1p-100f ? 1.0f / amax : 0.0f;
    const int64_t tv = (int64_t)a.rows_per_sample * (a.N >> 2);
    const float* ys = a.y + z * a.st_y + smp * tv * 4;
    unsigned long long q = 0;
#pragma unroll
    for (int it = 0; it < RES_VPT; ++it) {
        const int64_t v = ((int64_t)blockIdx.x * RES_VPT + it) * 256 + threadIdx.x;
        if (v >= tv) break;
        const float4 w = *(const float4*)(ys + v * 4);
        const float ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float r = ww[e] * inv;
            q += (unsigned long long)((double)r * (double)r * 0x1p40);
        }
    }
    const unsigned long long t =
        block_reduce_256(wave_sum_u64(q), [](unsigned long long x, unsigned long long y) { return x + y; }, reds);
    if (threadIdx.x == 0 && t) atomicAdd(a.gsum + z * a.st_b + smp, t);
}

hipError_t launch_goodness_fx(const GoodnessFxArgs& a, hipStream_t s)
{
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    const int64_t tv = (int64_t)a.rows_per_sample * (a.N >> 2);
    const int64_t B = a.M / a.rows_per_sample;
    const unsigned bx = (unsigned)((tv + 256 * RES_VPT - 1) / (256 * RES_VPT));
    if (B > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_goodness_fx, dim3(bx, (unsigned)B, (unsigned)a.nb), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// look-ahead (Eq. (3)/(4)): per sample, walk the layers from the last to the first
// ------------------------------------------------------------------------------------------------
struct LookaheadKArgs {
    LookaheadArgs a;
    const float* s_w[32];
};

__global__ __launch_bounds__(256) void k_lookahead(LookaheadKArgs ka)
{
    const LookaheadArgs& a = ka.a;
    const int p = blockIdx.y;
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool live = b < a.B;
    float S = 0.0f;
    for (int i = a.k - 1; i >= 0; --i) {
        const int64_t off = i * a.st_layer + p * a.st_pass + (live ? b : 0);
        const float c = live ? a.coeff[off] : 0.0f;
        const float ct = __builtin_fmaf(a.lambda, S, c);
        S = S + c;
        if (live) a.coeff_total[off] = ct;
        if (a.vmax) {
            uint32_t bits = 0;
            if (live) {
                float ymax;
                if ((a.fx_mask >> i) & 1u) {
                    ymax = __uint_as_float((uint32_t)a.vmax[off]);
                } else {
                    const float s_y = a.s_a[i * a.np + p] * ka.s_w[i][0];
                    ymax = (float)a.vmax[off] * s_y;
                }
                bits = __float_as_uint(fabsf(2.0f * ct) * ymax);
            }
            bits = wave_max_u32(bits);
            if ((threadIdx.x & 63) == 0 && bits) atomicMax(a.g_amax_bits + i * a.np + p, bits);
        }
    }
}

hipError_t launch_lookahead_impl(const LookaheadArgs& a, const float* const* s_w_host, hipStream_t s)
{
    LookaheadKArgs ka;
    ka.a = a;
    for (int i = 0; i < 32; ++i) ka.s_w[i] = (s_w_host && i < a.k) ? s_w_host[i] : nullptr;
    hipLaunchKernelGGL(k_lookahead, dim3((unsigned)((a.B + 255) / 256), (unsigned)a.np), dim3(256), 0, s, ka);
    return hipGetLastError();
}

hipError_t launch_lookahead(const LookaheadArgs& a, hipStream_t s)
{
    // a.s_w is a HOST array of device pointers here; they travel in the kernel argument block
    return launch_lookahead_impl(a, a.s_w, s);
}

__global__ __launch_bounds__(1024) void k_grad_amax(const float* __restrict__ ct0, const int32_t* __restrict__ vmax0,
                                                    const float* __restrict__ s_a, const float* __restrict__ s_w,
                                                    int64_t B, uint32_t* __restrict__ slot)
{
    const int z = blockIdx.x;
    const float* ct = ct0 + z * B;
    const int32_t* vmax = vmax0 + z * B;
    const float s_y = s_a[z] * s_w[0];
    uint32_t bits = 0;
    for (int64_t b = threadIdx.x; b < B; b += 1024) {
        const float ymax = (float)vmax[b] * s_y;
        bits = max(bits, __float_as_uint(fabsf(2.0f * ct[b]) * ymax));
    }
    block_store_max_bits<1024>(bits, slot + z);
}

hipError_t launch_grad_amax(const float* ct, const int32_t* vmax, const float* s_a, const float* s_w, int64_t B, int nb,
                            uint32_t* slot, hipStream_t s)
{
    hipLaunchKernelGGL(k_grad_amax, dim3((unsigned)nb), dim3(1024), 0, s, ct, vmax, s_a, s_w, B, slot);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Goodness, loss, dL/dG, look-ahead and the absmax of the local gradients of ALL layers at once.  Nothing in the forward
// pass needs a goodness before the look-ahead (the hand-off quantiser takes its range from the contraction's own
// per-sample maxima), so the per-layer launches -- 4 to 6 us each between two contractions -- are folded into this one.
// Workgroups 0 .. tiles-1 of a pass: 64 samples each, one wavefront per layer (16 layers at a time): every (layer, sample)
// is worked out side by side, the coefficients meet in LDS and every thread forms its own suffix sum.  The workgroups
// after them: the loss of one layer each, in a fixed order.
// ------------------------------------------------------------------------------------------------
// The range of one layer's output for the hand-off of a larger batch: one workgroup per pass.  Bound by its latency (two
// dependent loads, a square root, a reduction): a batch of 12288 is 12 samples per thread, too few to split further.
__global__ __launch_bounds__(1024) void k_handoff_range(RangeArgs a)
{
    const int z = blockIdx.x;
    const float s_y = a.s_a[z] * a.s_w[0];
    const double s_yd = (double)s_y, pow2r = (double)(1ull << a.rshift);
    uint32_t m = 0;
    for (int64_t b = threadIdx.x; b < a.B; b += 1024) {
        float y = (float)a.vmax[z * a.B + b] * s_y;
        if (a.l2norm) {
            const float nrm = sqrtf(goodness_value(a.gsum[z * a.B + b], pow2r, s_yd));
            y = nrm > 0.0f ? y / nrm : 0.0f;
        }
        m = max(m, __float_as_uint(y));
    }
    block_store_max_bits<1024>(m, a.out + z);
}

hipError_t launch_handoff_range(const RangeArgs& a, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_handoff_range, dim3(2), dim3(1024), 0, s, a);
    return hipGetLastError();
}

constexpr int GA_WAVES = 16, GA_THREADS = 64 * GA_WAVES;

__device__ __forceinline__ float goodness_of(const GoodnessAllArgs& a, const GoodnessLayer& L, int i, int p, int64_t b, float& s_y)
{
    const int64_t o = ((int64_t)i * 2 + p) * a.B + b;
    if (L.fx) {
        const float amax = __uint_as_float(a.out_amax[2 * (i + 1) + p]);
        s_y = 1.0f;
        return amax < 0x1p-100f ? 0.0f : goodness_value(a.gsum[o], 0x1p-40, (double)amax);
    }
    s_y = a.s_a[2 * i + p] * L.s_w[0];
    return goodness_value(a.gsum[o], (double)(1ull << L.rshift), (double)s_y);
}

__global__ __launch_bounds__(GA_THREADS) void k_goodness_all(GoodnessAllArgs a)
{
    __shared__ float sc[32][64];
    __shared__ double red[GA_THREADS];
    const int p = blockIdx.y, tiles = (int)((a.B + 63) >> 6);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int sign = p ? -1 : 1;
    if ((int)blockIdx.x >= tiles) {   // the loss of one layer
        const int i = (int)blockIdx.x - tiles;
        const GoodnessLayer& L = a.L[i];
        if (L.projection) {
            if (threadIdx.x == 0) a.loss[2 * i + p] = 0.0f;
            return;
        }
        double lsum = 0.0;
        for (int64_t b = threadIdx.x; b < a.B; b += GA_THREADS) {
            float s_y, xs;
            const float G = goodness_of(a, L, i, p, b, s_y);
            (void)loss_derivative(G - L.theta, sign, xs);
            lsum += (double)loss_term(xs);
        }
        red[threadIdx.x] = lsum;
        __syncthreads();
        for (int s = GA_THREADS / 2; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
            __syncthreads();
        }
        if (threadIdx.x == 0) a.loss[2 * i + p] = (float)(red[0] / (double)a.B);
        return;
    }
    const int64_t b = (int64_t)blockIdx.x * 64 + lane;
    const bool in = b < a.B;
    float ym[2];   // largest activity of the thread's (up to two) layers
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int i = r * GA_WAVES + wv;
        ym[r] = 0.0f;
        if (i >= a.k) continue;
        const GoodnessLayer& L = a.L[i];
        float c = 0.0f;
        if (in) {
            const int64_t o = ((int64_t)i * 2 + p) * a.B + b;
            float G = 0.0f;
            if (!L.projection) {   // (a projection has no activity of its own: zero goodness, nothing enters the sums)
                float s_y, xs;
                G = goodness_of(a, L, i, p, b, s_y);
                c = loss_derivative(G - L.theta, sign, xs);
                ym[r] = L.fx ? __uint_as_float((uint32_t)a.vmax[o]) : (float)a.vmax[o] * s_y;
            }
            a.goodness[o] = G;
            a.coeff[o] = c;
        }
        sc[i][lane] = c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int i = r * GA_WAVES + wv;
        if (i >= a.k) continue;
        float S = 0.0f;
        for (int j = a.k - 1; j > i; --j) S = S + sc[j][lane];
        const float ct = __builtin_fmaf(a.lambda, S, sc[i][lane]);
        if (in) a.coeff_total[((int64_t)i * 2 + p) * a.B + b] = ct;
        const uint32_t bits = wave_max_u32(__float_as_uint(fabsf(2.0f * ct) * ym[r]));
        if (lane == 0 && bits) atomicMax(a.g_amax_bits + 2 * i + p, bits);
    }
}

hipError_t launch_goodness_all(const GoodnessAllArgs& a, hipStream_t s)
{
    if (a.k < 1 || a.k > 32 || a.B < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_goodness_all, dim3((unsigned)((a.B + 63) / 64 + a.k), 2), dim3(GA_THREADS), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Exact-derivative look-ahead: the two gradients of a dense layer (see ChainArgs).  A thread owns four
// consecutive columns of one row per trip; HBM-bound (two int32 tensors read, two fp32 tensors written).  At most 1024
// workgroups per pass, each leaving one candidate for the absmax of either tensor: with one workgroup per 1024 elements
// the thousands of atomics on two words were most of a launch (2 x 1500 x 1500: 72 us, now 13).
// ------------------------------------------------------------------------------------------------
template <bool VEC>
__global__ __launch_bounds__(256) void k_chain_combine(ChainArgs a)
{
    const int z = blockIdx.y;
    const uint32_t ngroups = (uint32_t)((a.N + 3) >> 2);
    const int64_t total = a.M * ngroups;
    const float s_y = a.s_a[z * a.st_s_a] * a.s_w[0];
    const float s_e = a.e_acc ? a.s_h[z * a.st_s_h] * a.s_w_up[0] : 0.0f;
    uint32_t mh = 0, mg = 0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const uint32_t m = (uint32_t)e / ngroups;   // fewer than 2^32 elements
        const int64_t j0 = (int64_t)((uint32_t)e - m * ngroups) << 2;
        const float d = 2.0f * a.coeff[z * a.st_coeff + m];
        const uint4 av = ld_stream16(a.acc + z * a.st_acc + m * a.ldacc + j0);
        uint4 ev = make_uint4(0u, 0u, 0u, 0u);
        if (a.e_acc) ev = ld_stream16(a.e_acc + z * a.st_e + m * a.lde + j0);
        const int ai[4] = {(int)av.x, (int)av.y, (int)av.z, (int)av.w};
        const int ei[4] = {(int)ev.x, (int)ev.y, (int)ev.z, (int)ev.w};
        float hv[4], gv[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float y = (float)ai[c] * s_y;
            if (a.relu && y < 0.0f) y = 0.0f;
            const float t = d * y;
            const float E = a.e_acc ? (float)ei[c] * s_e : 0.0f;
            const bool live = (!a.relu || ai[c] > 0) && j0 + c < a.N;
            hv[c] = live ? t + E : 0.0f;
            gv[c] = live ? __builtin_fmaf(a.lambda, E, t) : 0.0f;
            mh = max(mh, __float_as_uint(hv[c]) & 0x7FFFFFFFu);
            mg = max(mg, __float_as_uint(gv[c]) & 0x7FFFFFFFu);
        }
        float* gp = a.g + z * a.st_out + m * a.N + j0;
        float* hp = a.h ? a.h + z * a.st_out + m * a.N + j0 : nullptr;
        if (VEC) {
            *(float4*)gp = make_float4(gv[0], gv[1], gv[2], gv[3]);
            if (hp) *(float4*)hp = make_float4(hv[0], hv[1], hv[2], hv[3]);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (j0 + c < a.N) {
                    gp[c] = gv[c];
                    if (hp) hp[c] = hv[c];
                }
        }
    }
    if (a.amax_atomic) block_atomic_max_bits<256>(mg, a.g_amax_bits + z);
    else block_store_max_bits<256>(mg, a.g_amax_bits + z * CHAIN_MAX_BLOCKS + blockIdx.x);
    if (a.h) {
        __syncthreads();   // the reduction buffer of the first call is read by thread 0 until here
        if (a.amax_atomic) block_atomic_max_bits<256>(mh, a.h_amax_bits + z);
        else block_store_max_bits<256>(mh, a.h_amax_bits + z * CHAIN_MAX_BLOCKS + blockIdx.x);
    }
}

int chain_blocks(int64_t M, int64_t N)
{
    const int64_t total = M * ((N + 3) >> 2);
    return (int)max((int64_t)1, min((int64_t)CHAIN_MAX_BLOCKS, (total + 255) / 256));
}

hipError_t launch_chain_combine(const ChainArgs& a, hipStream_t s)
{
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    const dim3 grid((unsigned)chain_blocks(a.M, a.N), (unsigned)a.nb);
    const bool vec = (a.N & 3) == 0 && ((((uintptr_t)a.g) & 15) == 0) && (!a.h || (((uintptr_t)a.h) & 15) == 0) &&
                     (a.st_out & 3) == 0;
    if (vec) hipLaunchKernelGGL(k_chain_combine<true>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_chain_combine<false>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

// Transposed copy of an int8 matrix (the weights of a layer, for the gradient handed down the chain): 128 x 64 bytes per
// workgroup, 4 x 4 byte transposes in registers, regrouped through LDS into 16-byte stores.
__global__ __launch_bounds__(QT_THREADS) void k_transpose_i8(const int8_t* __restrict__ q, int8_t* __restrict__ q_t, int64_t N,
                                                             int64_t K, int64_t ldq, int64_t ldqt,
                                                             const float* __restrict__ s_in, float* __restrict__ s_out)
{
    constexpr int LDW = QTile<16, 2>::LDW, RH = QTile<16, 2>::RH, CHUNKS = QTile<16, 2>::CHUNKS;
    __shared__ uint32_t tileT[QTile<16, 2>::COLS * LDW];
    const int t = threadIdx.x, cb = t & 15, rg = t >> 4;
    const int64_t r0 = (int64_t)blockIdx.y * QTile<16, 2>::ROWS, c0 = (int64_t)blockIdx.x * QTile<16, 2>::COLS;
    if (blockIdx.x == 0 && blockIdx.y == 0 && t == 0) s_out[0] = s_in[0];
    const int64_t col = c0 + 4 * cb;
    uint32_t w[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t row = r0 + 4 * rg + RH * u + j;
            w[u][j] = row < N && col < ldq ? *(const uint32_t*)(q + row * ldq + col) : 0u;
        }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int rb = rg + 16 * u;
        const uint32_t t0 = __builtin_amdgcn_perm(w[u][1], w[u][0], 0x05010400u), t1 = __builtin_amdgcn_perm(w[u][1], w[u][0], 0x07030602u);
        const uint32_t t2 = __builtin_amdgcn_perm(w[u][3], w[u][2], 0x05010400u), t3 = __builtin_amdgcn_perm(w[u][3], w[u][2], 0x07030602u);
        tileT[(4 * cb + 0) * LDW + rb] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
        tileT[(4 * cb + 1) * LDW + rb] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
        tileT[(4 * cb + 2) * LDW + rb] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
        tileT[(4 * cb + 3) * LDW + rb] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int e = t + QT_THREADS * u;
        const int cl = e / CHUNKS, ch = e % CHUNKS;
        const int64_t oc = c0 + cl, orow = r0 + 16 * ch;
        if (oc < K && orow < ldqt) {
            const uint32_t* p = tileT + cl * LDW + 4 * ch;
            *(u32x4*)(q_t + oc * ldqt + orow) = (u32x4){p[0], p[1], p[2], p[3]};
        }
    }
}

hipError_t launch_transpose_i8(const int8_t* q, int8_t* q_t, int64_t N, int64_t K, const float* s_in, float* s_out, hipStream_t s)
{
    if (N <= 0 || K <= 0) return hipSuccess;
    const dim3 grid((unsigned)((K + QTile<16, 2>::COLS - 1) / QTile<16, 2>::COLS), (unsigned)((N + QTile<16, 2>::ROWS - 1) / QTile<16, 2>::ROWS));
    hipLaunchKernelGGL(k_transpose_i8, grid, dim3(QT_THREADS), 0, s, q, q_t, N, K, pitch8(K), pitch8(N), s_in, s_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// weight update (HBM-bound: 4 B x (1 + n_terms x splits) read + 4 B written per weight) with fused absmax.  The matrix is
// walked as a flat sequence of four-column groups.  A split weight gradient is summed here, while its partial results are
// still in the caches, instead of by a kernel of its own that writes the sum for this one to read.
// k_update: a thread owns groups; G of them, 256 apart, per trip, all loads before the arithmetic.
// k_update_wide: many splits of a small output (a thread that walked them alone would issue one load after the other): sixteen
// lanes share the splits of a group and meet in LDS.
// ------------------------------------------------------------------------------------------------
struct UpdateScale {
    float sc[4], lr_eff;
};
__device__ __forceinline__ UpdateScale update_scale(const UpdateArgs& a)
{
    UpdateScale u;
#pragma unroll
    for (int j = 0; j < 4; ++j) u.sc[j] = j < a.n_terms ? a.s_g[j][0] * a.s_a[j][0] : 0.0f;
    u.lr_eff = a.lr / (float)a.total_samples;
    return u;
}
__device__ __forceinline__ float update_weight(const UpdateArgs& a, const UpdateScale& u, float w, int d0, int d1, int d2, int d3)
{
    float gr = (float)d0 * u.sc[0];
    if (1 < a.n_terms) gr = __builtin_fmaf((float)d1, u.sc[1], gr);
    if (2 < a.n_terms) gr = __builtin_fmaf((float)d2, u.sc[2], gr);
    if (3 < a.n_terms) gr = __builtin_fmaf((float)d3, u.sc[3], gr);
    return __builtin_fmaf(-u.lr_eff, gr, w);
}
// weights of one group: where they start, how many there are (four except at the end of a row that is no multiple of 4)
template <bool VEC>
__device__ __forceinline__ int update_group(const UpdateArgs& a, int64_t e, int64_t& at_w, int64_t& at_d)
{
    if (VEC) {   // rows of w and of the accumulators are contiguous: K % 4 == 0
        at_w = at_d = 4 * e;
        return 4;
    }
    const uint32_t kg = (uint32_t)((a.K + 3) >> 2);
    const uint32_t n = (uint32_t)e / kg;   // (an [N, K] tensor has fewer than 2^32 elements)
    const int64_t k = (int64_t)((uint32_t)e - n * kg) << 2;
    at_w = n * a.K + k;
    at_d = n * a.lddw + k;
    return (int)min((int64_t)4, a.K - k);
}

template <bool VEC, int G>
__global__ __launch_bounds__(256) void k_update(UpdateArgs a)
{
    constexpr int UNROLL = 4 / G;   // four loads in flight either way
    const UpdateScale us = update_scale(a);
    const int64_t total = a.N * ((a.K + 3) >> 2);
    uint32_t m = 0;
    for (int64_t e0 = (int64_t)blockIdx.x * 256 * G; e0 < total; e0 += (int64_t)gridDim.x * 256 * G) {
        float w[G][4];
        int4 d[G][4];
        int64_t at_w[G], at_d[G];
        int cnt[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int64_t e = e0 + g * 256 + threadIdx.x;
            cnt[g] = 0;
            at_w[g] = at_d[g] = 0;
            if (e < total) cnt[g] = update_group<VEC>(a, e, at_w[g], at_d[g]);
            if (VEC) {
                float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
                if (cnt[g]) f = *(const float4*)(a.w + at_w[g]);
                w[g][0] = f.x; w[g][1] = f.y; w[g][2] = f.z; w[g][3] = f.w;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) w[g][c] = c < cnt[g] ? a.w[at_w[g] + c] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                d[g][j] = make_int4(0, 0, 0, 0);
                if (j < a.n_terms && cnt[g]) {   // last use of the accumulators: streaming hint
                    const uint4 v = ld_stream16(a.dw[j] + at_d[g]);
                    d[g][j] = make_int4((int)v.x, (int)v.y, (int)v.z, (int)v.w);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j >= a.n_terms) break;
#pragma unroll UNROLL
            for (int sp = 1; sp < a.splits[j]; ++sp) {
                const int32_t* __restrict__ part = a.dw[j] + sp * a.st_split;
#pragma unroll
                for (int g = 0; g < G; ++g)
                    if (cnt[g]) {
                        const int4 v = *(const int4*)(part + at_d[g]);
                        d[g][j].x += v.x; d[g][j].y += v.y; d[g][j].z += v.z; d[g][j].w += v.w;
                    }
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            w[g][0] = update_weight(a, us, w[g][0], d[g][0].x, d[g][1].x, d[g][2].x, d[g][3].x);
            w[g][1] = update_weight(a, us, w[g][1], d[g][0].y, d[g][1].y, d[g][2].y, d[g][3].y);
            w[g][2] = update_weight(a, us, w[g][2], d[g][0].z, d[g][1].z, d[g][2].z, d[g][3].z);
            w[g][3] = update_weight(a, us, w[g][3], d[g][0].w, d[g][1].w, d[g][2].w, d[g][3].w);
            if (VEC) {
                if (cnt[g]) *(float4*)(a.w + at_w[g]) = make_float4(w[g][0], w[g][1], w[g][2], w[g][3]);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c < cnt[g]) {
                    if (!VEC) a.w[at_w[g] + c] = w[g][c];
                    m = max(m, __float_as_uint(w[g][c]) & 0x7FFFFFFFu);
                }
        }
    }
    block_store_max_bits<256>(m, a.block_max + blockIdx.x);
}

template <bool VEC>
__global__ __launch_bounds__(256) void k_update_wide(UpdateArgs a)
{
    __shared__ int4 red[4][16][16];
    const UpdateScale us = update_scale(a);
    const int64_t total = a.N * ((a.K + 3) >> 2);
    const int el = threadIdx.x & 15, sl = threadIdx.x >> 4;
    int most = 1;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j < a.n_terms) most = max(most, a.splits[j]);
    uint32_t m = 0;
    for (int64_t e0 = (int64_t)blockIdx.x * 16; e0 < total; e0 += (int64_t)gridDim.x * 16) {
        int64_t at_w = 0, at_d = 0;
        int cnt = 0;
        if (e0 + el < total) cnt = update_group<VEC>(a, e0 + el, at_w, at_d);
        // two splits of every term per trip, all eight loads in flight: a lane that loaded one split after the other waited for
        // each (launches of a MobileNet-shaped step 17.5 -> 7.9 us on average)
        int4 d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) d[j] = make_int4(0, 0, 0, 0);
        for (int sp = sl; sp < most; sp += 32) {
            int4 v[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    v[h][j] = make_int4(0, 0, 0, 0);
                    if (j < a.n_terms && cnt && sp + 16 * h < a.splits[j]) v[h][j] = *(const int4*)(a.dw[j] + (sp + 16 * h) * a.st_split + at_d);
                }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    d[j].x += v[h][j].x; d[j].y += v[h][j].y; d[j].z += v[h][j].z; d[j].w += v[h][j].w;
                }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < a.n_terms) red[j][sl][el] = d[j];
        __syncthreads();
        // four threads per group, one column each
        if (threadIdx.x < 64) {
            const int gel = threadIdx.x >> 2, c = threadIdx.x & 3;
            int64_t gw = 0, gd = 0;
            int gc = 0;
            if (e0 + gel < total) gc = update_group<VEC>(a, e0 + gel, gw, gd);
            if (c < gc) {
                int d[4] = {0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (j >= a.n_terms) break;
#pragma unroll
                    for (int r = 0; r < 16; ++r) d[j] += ((const int*)&red[j][r][gel])[c];
                }
                const float w = update_weight(a, us, a.w[gw + c], d[0], d[1], d[2], d[3]);
                a.w[gw + c] = w;
                m = max(m, __float_as_uint(w) & 0x7FFFFFFFu);
            }
        }
        __syncthreads();
    }
    block_store_max_bits<256>(m, a.block_max + blockIdx.x);
}

static int most_splits(const UpdateArgs& a)
{
    int most = 1;
    for (int j = 0; j < a.n_terms; ++j) most = max(most, a.splits[j]);
    return most;
}
// Sixteen lanes per group where a thread would have many splits to walk and there are too few groups to hide that.  A thread
// alone against sixteen lanes: 64 -> 64 channels (9 thousand groups, 64 splits) 32 -> 8 us, 256 x 256 (16 thousand, 16 to 32)
// 16 -> 7; past the line 700 x 700 (122 thousand, 16) 12.1 and 18.4, 500 x 500 (62 thousand, 8) 10.7 and 12.0.
static bool update_wide(const UpdateArgs& a)
{
    const int most = most_splits(a);
    return most >= 4 && a.N * ((a.K + 3) >> 2) <= (int64_t)most << 12;
}
// Groups of a thread per trip: four, or one where partial results are summed and four would leave the update with fewer than
// two workgroups per compute unit (590 thousand weights, 14 splits: 38 -> 16 us; 1000 x 1000, 8 splits: 28 -> 16).
static int update_groups(const UpdateArgs& a) { return most_splits(a) > 1 && a.N * ((a.K + 3) >> 2) <= (int64_t(1) << 19) ? 1 : 4; }

int update_blocks(const UpdateArgs& a)
{
    const int64_t total = a.N * ((a.K + 3) >> 2), per = update_wide(a) ? 16 : 256 * update_groups(a);
    return (int)max((int64_t)1, min((int64_t)a.max_blocks, (total + per - 1) / per));
}

hipError_t launch_update(const UpdateArgs& a, hipStream_t s)
{
    if (a.N <= 0 || a.K <= 0) return hipSuccess;
    const dim3 grid((unsigned)update_blocks(a));
    const bool vec = (a.K & 3) == 0 && ((((uintptr_t)a.w) & 15) == 0);
    if (update_wide(a)) {
        if (vec) hipLaunchKernelGGL(k_update_wide<true>, grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL(k_update_wide<false>, grid, dim3(256), 0, s, a);
    } else {
        const bool one = update_groups(a) == 1;
        if (vec && one) hipLaunchKernelGGL((k_update<true, 1>), grid, dim3(256), 0, s, a);
        else if (vec) hipLaunchKernelGGL((k_update<true, 4>), grid, dim3(256), 0, s, a);
        else if (one) hipLaunchKernelGGL((k_update<false, 1>), grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_update<false, 4>), grid, dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace ffi
