// Contraction of short rows whose result is not stored: the accumulators of a 1x1 convolution (or of a first layer's patch
// matrix) with a reduction of up to 128 bytes are worked out again by each pass that needs them -- the goodness sums, the codes
// handed to the next layer, the codes of the local gradient -- instead of being written once as int32 and read twice.  12 bytes
// of traffic per output become the reduction's own row once per pass (24 channels -> 144: 0.2 bytes an output) and the
// multiplies are a handful.
//
// A wavefront takes 128 rows x 32 columns at a time.  Both operands go from global memory into the MFMA registers as they
// lie (a lane's 16 bytes are one chunk of one row; consecutive rows are consecutive memory), without LDS and barriers; the
// codes leave the registers through lane exchanges (codes.hpp).  For the transposed codes lane 4 a + e of block t stands for
// row 16 a + 4 t + e, so that after the exchange a lane holds 16 consecutive rows of a column: eight lanes store a whole
// 128-byte line.  Bound by the vector ALUs (hash, scaling, rounding: about 100 clocks per 64 codes), not by memory.
//
// 24 -> 144 channels, two passes of 256 images of 32x32: contraction with stores, hand-off and local gradient 97 + 80 + 95 us,
// goodness, hand-off and local gradient here 16 + 44 + 51; 3 -> 64 (patches of 27 bytes) 42 + 32 + 37 and 13 + 22 + 24.  A MobileNet-shaped
// step 2218 -> 1635 us, 3-64-128-256 at 32x32 946 -> 904, 1-32-48-96 at 28x28 195 -> 186.  The goodness sums take one reduction
// and two atomics per run of a wavefront's items in one sample (31 us with one per item).
#include "codes.hpp"

namespace ffi {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int ROWS_THREADS = 256, ROWS_WAVES = ROWS_THREADS / 64;
constexpr int UNIT = 128;   // rows of one item

template <int WHAT, int KS>
__global__ __launch_bounds__(ROWS_THREADS) __attribute__((amdgpu_waves_per_eu(KS == 1 ? 4 : KS == 2 ? 3 : 2))) void k_rows_i8(RowsArgs r, QuantArgs a, int per)
{
    constexpr bool GRAD = WHAT == ROWS_GRAD;
    const int z = blockIdx.y;
    const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    CodeScale cs = {};
    if (WHAT != ROWS_GOODNESS) {
        cs = code_scale<ROWS_THREADS>(a, z);
        if (blockIdx.x == 0 && threadIdx.x == 0) a.scale[z * a.st_scale] = cs.live ? cs.amax / 127.0f : 1.0f;
    }
    const uint32_t tj = (uint32_t)(r.J + 31) >> 5, units = (uint32_t)(r.I + UNIT - 1) / UNIT, items = units * tj;
    const int rpad = (r.R + 15) & ~15;
    const uint32_t rps = (uint32_t)r.rows_per_sample;
    // (consecutive items: the columns of one group of rows after the other)
    const uint32_t item0 = (blockIdx.x * ROWS_WAVES + wave) * (uint32_t)per, item1 = min(items, item0 + (uint32_t)per);
    unsigned long long sq = 0;   // goodness sum and maximum of the sample (or of the block) at hand
    int vm = 0;
    for (uint32_t item = item0; item < item1; ++item) {
        const uint32_t unit = item / tj;
        const int i0 = (int)(unit * UNIT), j0 = (int)(item - unit * tj) << 5;
        const int smp = one_sample_of(i0, UNIT, r.I, rps);   // (-1: several)
        // rows and columns beyond the matrices read as zero (range check); so do chunks beyond the reduction, in Q
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void*)(r.P + z * r.st_p + (int64_t)i0 * r.ldp), 0, (int)(min(UNIT, r.I - i0) * r.ldp), 0x00020000);
        const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)(r.Q + (int64_t)j0 * r.ldq), 0, (int)(min(32, r.J - j0) * r.ldq), 0x00020000);
        v4i fq[KS], fp[4][KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int at = 32 * k + 16 * lh;
            fq[k] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rq, at < rpad ? lr * (int)r.ldq + at : 0x7FFFFFF0, 0, 0);
        }
        int row[4];   // of this lane, from i0
#pragma unroll
        for (int ti = 0; ti < 4; ++ti) {
            row[ti] = GRAD ? 16 * (lr >> 2) + 4 * ti + (lr & 3) : 32 * ti + lr;
#pragma unroll
            for (int k = 0; k < KS; ++k)
                fp[ti][k] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rp, row[ti] * (int)r.ldp + 32 * k + 16 * lh, 0, 0);
        }
        float rowf[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (GRAD) {
            const float* per_sample = a.per_sample + z * a.st_per_sample;
            if (smp >= 0) {
                const float f = 2.0f * per_sample[smp];
#pragma unroll
                for (int ti = 0; ti < 4; ++ti) rowf[ti] = f;
            } else {
#pragma unroll
                for (int ti = 0; ti < 4; ++ti) rowf[ti] = 2.0f * per_sample[(uint32_t)min(i0 + row[ti], r.I - 1) / rps];
            }
        }
        auto contract = [&](int ti) {
            v16i acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
            for (int k = 0; k < KS; ++k) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fq[k], fp[ti][k], acc, 0, 0, 0);
            return acc;
        };
        if constexpr (WHAT == ROWS_GOODNESS) {
#pragma unroll
            for (int ti = 0; ti < 4; ++ti) {
                const v16i acc = contract(ti);
                int v[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e] = acc[e];
                goodness_terms(r.relu, r.rshift, v, 16, sq, vm);
                if (smp >= 0) {   // one reduction and two atomics for all consecutive items of a sample
                    if (ti < 3) continue;
                    const int next = (int)((item + 1) / tj * UNIT);
                    if (item + 1 < item1 && (next == i0 || one_sample_of(next, UNIT, r.I, rps) == smp)) continue;
                    goodness_one(sq, vm, r.gsum + z * r.st_g + smp, r.vmax + z * r.st_g + smp);
                } else {
                    goodness_runs(sq, vm, i0 + 32 * ti, r.I, rps, r.gsum + z * r.st_g, r.vmax + z * r.st_g);
                }
                sq = 0;
                vm = 0;
            }
        } else {
            const uint32_t cols = (uint32_t)r.J, col = (uint32_t)(j0 + 4 * lh);
            auto codes = [&](auto form) {
                constexpr int FORM = decltype(form)::value;
                uint32_t w[4][4];
#pragma unroll
                for (int ti = 0; ti < 4; ++ti) {
                    const v16i acc = contract(ti);
                    const uint32_t idx = (uint32_t)(i0 + row[ti]) * cols + col;
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        w[ti][g] = quad_codes<GRAD, FORM>(cs, acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3], idx + 8u * g, rowf[ti]);
                    if (!GRAD) {
                        const uint4 o = words_row_major(w[ti]);
                        const int at = j0 + 16 * lh;
                        if (i0 + row[ti] < r.I && at < a.ldq)
                            *(uint4*)(a.q + z * a.st_q + (int64_t)(i0 + row[ti]) * a.ldq + at) = o;
                    }
                }
                if (GRAD) {
                    const int64_t at = i0 + 16 * (lr >> 2);   // first of this lane's 16 rows; up to the row pitch zeros are stored
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int j = j0 + 8 * g + 4 * lh + (lr & 3);
                        u32x4 o;
#pragma unroll
                        for (int ti = 0; ti < 4; ++ti) o[ti] = word_transposed(w[ti][g]);
                        if (j < r.J && at < a.ldqt) *(u32x4*)(a.q_t + z * a.st_qt + (int64_t)j * a.ldqt + at) = o;
                    }
                }
            };
            // (all uniform)
            if (!cs.fixed) codes(std::integral_constant<int, CODE_FLOAT>{});
            else if (!GRAD) codes(std::integral_constant<int, CODE_UP>{});
            else if (smp < 0) codes(std::integral_constant<int, CODE_LANE>{});
            else if (rowf[0] < 0.0f) codes(std::integral_constant<int, CODE_DOWN>{});
            else codes(std::integral_constant<int, CODE_UP>{});
        }
    }
}

template <int WHAT>
static hipError_t launch_rows_t(const RowsArgs& r, const QuantArgs& a, hipStream_t s)
{
    const int64_t items = ((int64_t)r.I + UNIT - 1) / UNIT * ((r.J + 31) >> 5);
    // as many wavefronts as the chip holds, each with the same number of items
    const int64_t most = (int64_t)num_cus() * 8 * ROWS_WAVES / r.nb;
    const int64_t rounds = (items + most - 1) / most, waves = (items + rounds - 1) / rounds;
    const dim3 grid((unsigned)((waves + ROWS_WAVES - 1) / ROWS_WAVES), (unsigned)r.nb);
    if (r.R <= 32) hipLaunchKernelGGL((k_rows_i8<WHAT, 1>), grid, dim3(ROWS_THREADS), 0, s, r, a, (int)rounds);
    else if (r.R <= 64) hipLaunchKernelGGL((k_rows_i8<WHAT, 2>), grid, dim3(ROWS_THREADS), 0, s, r, a, (int)rounds);
    else hipLaunchKernelGGL((k_rows_i8<WHAT, 4>), grid, dim3(ROWS_THREADS), 0, s, r, a, (int)rounds);
    return hipGetLastError();
}

hipError_t launch_rows(int what, const RowsArgs& r, const QuantArgs& a, hipStream_t s)
{
    if (r.I <= 0 || r.J <= 0) return hipSuccess;
    if (r.R > ROWS_MAX_R || (r.J & 3) != 0 || r.nb < 1 || r.nb > 2 || r.rows_per_sample < 1 ||
        ((int64_t)r.I + UNIT - 1) / UNIT * ((r.J + 31) >> 5) > 0x7FFFFFFF)
        return hipErrorInvalidValue;
    if (what == ROWS_GOODNESS) return r.gsum && r.vmax ? launch_rows_t<ROWS_GOODNESS>(r, a, s) : hipErrorInvalidValue;
    if (a.round_mode != FF_ROUND_STOCHASTIC || a.l2norm || a.rows != r.I || a.cols != r.J) return hipErrorInvalidValue;
    // (a row of codes is covered up to its pitch by whole 32-column items)
    if (what == ROWS_HANDOFF) return a.q && !a.q_t && a.ldq <= (((int64_t)r.J + 31) & ~31) ? launch_rows_t<ROWS_HANDOFF>(r, a, s) : hipErrorInvalidValue;
    if (what == ROWS_GRAD) return a.q_t && !a.q && a.per_sample && a.ldqt <= ((int64_t)r.I + UNIT - 1) / UNIT * UNIT ? launch_rows_t<ROWS_GRAD>(r, a, s) : hipErrorInvalidValue;
    return hipErrorInvalidValue;
}

}  // namespace ffi
