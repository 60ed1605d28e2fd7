// Device code that turns a 32x32 block of int32 accumulators, as v_mfma_i32_32x32x32_i8 leaves it, into int8 codes: the
// arithmetic of the quantiser (elementwise.hip, sources QSRC_HANDOFF and QSRC_GRAD, stochastic rounding) on values that never
// leave the registers.  Include it only in files compiled with -ffp-contract=off.
#pragma once

#include <type_traits>

#include "ff_internal.hpp"
#include "device_math.hpp"

namespace ffi {

// What every element of a pass shares.
struct CodeScale {
    float s_y, inv, floor_y;
    uint32_t key;
    bool fixed, live;   // fixed-point rounding applies: no NaN, infinite only where rectified away (see quantize_tile); the range does not vanish
    float amax;
};

// Maximum over a workgroup of `THREADS` threads, in every thread.
template <int THREADS>
__device__ __forceinline__ uint32_t block_max_u32(uint32_t v)
{
    __shared__ uint32_t red[THREADS / 64];
    v = wave_max_u32(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < THREADS / 64; ++i) v = max(v, red[i]);
    return v;
}

// Range, factors and random key of pass z.  Every thread of the workgroup calls it.
template <int THREADS>
__device__ __forceinline__ CodeScale code_scale(const QuantArgs& a, int z)
{
    CodeScale c;
    c.s_y = a.s_a[z * a.st_s_a] * a.s_w[z * a.st_s_w];
    uint32_t word;
    if (a.vmax) {   // (uniform) a hand-off that takes its range from the contraction's per-sample maxima
        const int32_t* vm = a.vmax + z * a.st_b;
        uint32_t mm = 0;
        for (int i = threadIdx.x; i < a.B; i += THREADS) mm = max(mm, (uint32_t)vm[i]);
        word = __float_as_uint((float)(int)block_max_u32<THREADS>(mm) * c.s_y);
    } else {
        word = a.amax_bits[z * a.st_amax];
    }
    c.amax = __uint_as_float(word);
    c.live = c.amax >= 0x1p-100f;
    c.inv = c.live ? 127.0f / c.amax : 0.0f;
    c.floor_y = a.relu ? 0.0f : -__builtin_inff();
    c.key = (z ? a.key2 : a.key).k0;
    if (a.step_dev) c.key = make_sr_key(a.seed, stream_tag_of(a.step_dev[0], a.tag_layer, (uint32_t)z, a.tag_kind)).k0;
    c.fixed = c.live && c.amax < __builtin_inff() && a.relu && c.s_y < 0x1p80f;
    return c;
}

// How a block is rounded: in floating point, or in fixed point with the sign of the row's factor (GRAD) known for the whole
// wavefront -- codes up from zero, or down -- or per lane.
enum CodeForm { CODE_FLOAT, CODE_UP, CODE_DOWN, CODE_LANE };

// Codes of four neighbouring columns of one row, packed; idx: element index of the first, a multiple of four.  rowf: the
// row's factor (GRAD).
template <bool GRAD, int FORM>
__device__ __forceinline__ uint32_t quad_codes(const CodeScale& s, int c0, int c1, int c2, int c3, uint32_t idx, float rowf)
{
    uint32_t w[4];
    sr_head4(idx ^ s.key, w);
    const int cc[4] = {c0, c1, c2, c3};
    if constexpr (FORM != CODE_FLOAT) {
        uint32_t top[4];
        const bool down = FORM == CODE_DOWN || (FORM == CODE_LANE && rowf < 0.0f);
        const float one = down ? 1.0f : 0.0f;
        const float lo = down ? 0.0f : -SR_MOST, hi = down ? SR_MOST : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float v = (float)cc[e] * s.s_y;
            if (GRAD) v = rowf * v;
            const float t = v * s.inv;
            top[e] = sr_top(FORM != CODE_UP ? sr_scale(t, one) : t * -0x1p24f, lo, hi, w[e]);
        }
        return sr_pack(top[0], top[1], top[2], top[3]);
    } else {
        uint32_t word = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float v = fmaxf((float)cc[e] * s.s_y, s.floor_y);
            if (GRAD) v = rowf * v;
            word |= ((uint32_t)quant_code_of_word<true>(v, s.inv, w[e] ^ (w[e] >> 16)) & 0xFFu) << (8 * e);
        }
        return word;
    }
}

__device__ __forceinline__ unsigned long long xor_lane_u64(unsigned long long v, int d)
{
    const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)v, d), hi = (unsigned)__shfl_xor((int)(unsigned)(v >> 32), d);
    return ((unsigned long long)hi << 32) | lo;
}

// Sum of squares and maximum of one block's activities, added to a lane's own.
__device__ __forceinline__ void goodness_terms(int relu, int rshift, const int* v, int n, unsigned long long& sq, int& vm)
{
    if (relu && rshift == 0) {
#pragma unroll
        for (int e = 0; e < n; ++e) {
            const unsigned y = (unsigned)max(v[e], 0);
            sq += (unsigned long long)y * y;
            vm = max(vm, (int)y);
        }
    } else {
#pragma unroll
        for (int e = 0; e < n; ++e) {
            const int y = relu ? max(v[e], 0) : v[e];
            const long long yl = (long long)y;
            sq += ((unsigned long long)(yl * yl)) >> rshift;
            vm = max(vm, y < 0 ? -y : y);
        }
    }
}
// A wavefront's sums into the words of one sample.
__device__ __forceinline__ void goodness_one(unsigned long long sq, int vm, unsigned long long* gsum, int32_t* vmax)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        sq += xor_lane_u64(sq, d);
        vm = max(vm, __shfl_xor(vm, d));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(gsum, sq);
        atomicMax(vmax, vm);
    }
}
// ... of rows i0 + (lane & 31) that belong to several samples: the rows of a sample are a run of lanes, one atomic per run.
// The two half-waves hold the two halves of a row's columns.
__device__ __forceinline__ void goodness_runs(unsigned long long sq, int vm, int i0, int I, uint32_t rps,
                                              unsigned long long* gsum, int32_t* vmax)
{
    const int lane = threadIdx.x & 63, lr = lane & 31;
    sq += xor_lane_u64(sq, 32);
    vm = max(vm, __shfl_xor(vm, 32));
    const int i = i0 + lr, smp = (int)((uint32_t)i / rps);
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
        const unsigned lo = (unsigned)__shfl_down((int)(unsigned)sq, d, 32);
        const unsigned hi = (unsigned)__shfl_down((int)(unsigned)(sq >> 32), d, 32);
        const int ov = __shfl_down(vm, d, 32), os = __shfl_down(smp, d, 32);
        if (lr + d < 32 && os == smp) {
            sq += ((unsigned long long)hi << 32) | lo;
            vm = max(vm, ov);
        }
    }
    const int before = __shfl_up(smp, 1, 32);
    if (lane < 32 && i < I && (lr == 0 || before != smp)) {
        atomicAdd(gsum + smp, sq);
        atomicMax(vmax + smp, vm);
    }
}
// Sample of the rows r0 .. r0 + n - 1 (r0 < I; those beyond I do not count), or -1 if they belong to several.
__device__ __forceinline__ int one_sample_of(int r0, int n, int I, uint32_t rps)
{
    const uint32_t a = (uint32_t)r0 / rps, b = (uint32_t)min(r0 + n - 1, I - 1) / rps;
    return a == b ? (int)a : -1;
}

// Block output of a residual layer from four accumulators of a row: y = act(fp32(acc) * s_y + u), one rounding per operation,
// u the block input's codes or the projection's accumulators at the same place.
struct ResidualScale {
    float s_y, s_u;
};
__device__ __forceinline__ ResidualScale residual_scale(const ResidualArgs& a, int z)
{
    return {a.s_a[z * a.st_s_a] * a.s_w[0],
            a.skip == FF_SKIP_IDENTITY ? a.s_x[z * a.st_s_x] : a.s_ap[z * a.st_s_ap] * a.s_wp[0]};
}
__device__ __forceinline__ float4 residual_value(const ResidualScale& s, int relu, const int c[4], const int4 skip, uint32_t& m)
{
    const int u[4] = {skip.x, skip.y, skip.z, skip.w};
    float y[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float t = (float)c[q] * s.s_y;
        y[q] = t + (float)u[q] * s.s_u;
    }
    if (relu) {   // (bits of values that are not negative, or of -0, compared as signed integers: no magnitudes to take)
        int b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            y[q] = fmaxf(y[q], 0.0f);
            b[q] = __float_as_int(y[q]);
        }
        m = (uint32_t)max(max(max((int)m, b[0]), b[1]), max(b[2], b[3]));
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) m = max(m, __float_as_uint(fabsf(y[q])));
    }
    return make_float4(y[0], y[1], y[2], y[3]);
}
// Rows row0 + rl + r RPI, r < NR, of a wavefront's output, LPR lanes of four columns to a row.  skip: what residual_load loads for them (codes of the
// block input as they lie, one word, or the projection's accumulators).
template <bool CODES> using ResidualSkip = std::conditional_t<CODES, uint32_t, int4>;
template <bool CODES, int LPR, int NR>
__device__ __forceinline__ void residual_load(const ResidualArgs& a, int z, int row0, int col, bool in, ResidualSkip<CODES> (&u)[NR])
{
    constexpr int RPI = 64 / LPR;
    const int rl = (int)(threadIdx.x & 63) / LPR;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int64_t row = row0 + r * RPI + rl;
        u[r] = {};
        if (in && row < a.M) {
            if constexpr (CODES) u[r] = *(const uint32_t*)(a.xq + z * a.st_xq + row * a.ldx + col);
            else u[r] = *(const int4*)(a.accp + z * a.st_accp + row * a.ldaccp + col);
        }
    }
}
// A lane's largest magnitudes of a wavefront's rows, which belong to one sample or to two (samples have RESIDUAL_MIN_ROWS rows at least): of `sample`, and
// of the one after it, whose rows start at `next`.
struct ResidualMax {
    uint32_t m[2], sample;
    int next;
};
__device__ __forceinline__ ResidualMax residual_max_of(const ResidualArgs& a, int row0)
{
    const uint32_t rps = (uint32_t)a.rows_per_sample, sample = (uint32_t)row0 / rps;
    return {{0, 0}, sample, (int)((sample + 1) * rps)};
}
// value(r) gives the accumulators, `in` says whether the lane has columns at all.  Stores y and takes its largest magnitudes into x.
template <bool CODES, int LPR, int NR, typename F>
__device__ __forceinline__ void residual_rows(const ResidualArgs& a, const ResidualScale& s, int z, int row0, int col, bool in, const ResidualSkip<CODES> (&u)[NR], ResidualMax& x, F value)
{
    constexpr int RPI = 64 / LPR;
    const int rl = (int)(threadIdx.x & 63) / LPR;
    const int M = (int)a.M;
    if (row0 >= M) return;   // (uniform)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int row = row0 + r * RPI + rl;
        int c[4];
        value(r, c);
        uint32_t mr = 0;
        int4 skip;
        if constexpr (CODES) skip = make_int4((int8_t)u[r], (int8_t)(u[r] >> 8), (int8_t)(u[r] >> 16), (int8_t)(u[r] >> 24));
        else skip = u[r];
        const float4 y = residual_value(s, a.relu, c, skip, mr);
        if (in && row < M) *(float4*)(a.y + z * a.st_y + (int64_t)row * a.N + col) = y;
        else mr = 0;
        x.m[0] = max(x.m[0], row < x.next ? mr : 0u);
        x.m[1] = max(x.m[1], row < x.next ? 0u : mr);
    }
}
// One atomic per sample for all ROWS rows of a wavefront from row0 on.  All atomics of a launch meet in a few cache lines, where they take 2 to 4 ns
// each: with one per slice of 8 rows, the forward contractions of a step with a 24-128 projection block on 16 images of 28x28 took
// 119 us, 85 this way; with one per row of a slice, 128 channels on 14x14 maps of 38 images (two passes) 29 instead of 17.
template <int ROWS>
__device__ __forceinline__ void residual_max_store(const ResidualArgs& a, int z, int row0, ResidualMax& x)
{
    static_assert(ROWS <= RESIDUAL_MIN_ROWS, "more than two samples");
    if (row0 >= (int)a.M) return;   // (uniform)
    uint32_t* const ymax = a.ymax_bits + z * a.st_b + x.sample;
    const int lane = threadIdx.x & 63;
    x.m[0] = wave_max_u32(x.m[0]);
    if (lane == 0 && x.m[0]) atomicMax(ymax, x.m[0]);
    if (x.next < min(row0 + ROWS, (int)a.M)) {   // (uniform)
        x.m[1] = wave_max_u32(x.m[1]);
        if (lane == 0 && x.m[1]) atomicMax(ymax + 1, x.m[1]);
    }
}

// A block's words: lane (lr = lane & 31, lh = lane >> 5) holds for its row the words g = 0 .. 3 of columns 8 g + 4 lh .. + 3.
// Row-major: afterwards lane lh holds columns 16 lh .. + 15 of its row, 16 bytes in order.
__device__ __forceinline__ uint4 words_row_major(const uint32_t w[4])
{
    const auto p = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
    const auto q = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
    return make_uint4(p[0], p[1], q[0], q[1]);
}
// Transposed: four neighbouring lanes 4 a + e exchange bytes; afterwards lane e holds, for column 8 g + 4 lh + e, the codes
// of the four rows of lanes 4 a .. 4 a + 3.
__device__ __forceinline__ uint32_t word_transposed(uint32_t w)
{
    const uint32_t lane = threadIdx.x;
    const uint32_t y = dpp_u32<0xB1>(w);   // quad_perm [1,0,3,2]
    const uint32_t r = __builtin_amdgcn_perm(y, w, lane & 1 ? 0x03070105u : 0x06020400u);
    const uint32_t x = dpp_u32<0x4E>(r);   // quad_perm [2,3,0,1]
    return __builtin_amdgcn_perm(x, r, lane & 2 ? 0x03020706u : 0x05040100u);
}

}  // namespace ffi
