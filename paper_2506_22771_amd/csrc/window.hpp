// What the kernels of 3x3 stride-1 convolutions share: the numbering of a zero-bordered input window, copies into LDS, and what becomes of a
// wavefront's accumulators.  Include it only in files compiled with -ffp-contract=off.
#pragma once

#include "codes.hpp"

namespace ffi {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int BEYOND = 0x7FFFFFF0;   // a byte offset beyond any buffer: reads as zero

// 16 bytes per lane straight into LDS, tracked by hand with vmcnt (see gemm_i8.hip)
__device__ __forceinline__ void copy16(__amdgpu_buffer_rsrc_t rsrc, int voffset, unsigned lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_base), "v"(voffset), "s"(rsrc) : "memory", "m0");
}
__device__ __forceinline__ void lds_barrier()   // this wavefront's LDS operations are done, and so are the others'
{
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---- positions of the input with one column of zeros in front of every row and one row of zeros in front of every image: the end of a row, or
// of an image, meets the zeros of the next.  Tap (kh, kw) of an output pixel lies kh (W + 1) + kw positions behind tap (0, 0).
struct WindowGeom {   // reciprocals of H W, W, W + 1, H + 1: x / d = x * reciprocal >> 32
    uint32_t div_hw, div_w, div_wp, div_hp;
};
// position of tap (0, 0) of output pixel m
__device__ __forceinline__ int window_first(const WindowGeom& c, int H, int W, uint32_t m)
{
    const uint32_t b = __umulhi(m, c.div_hw), rem = m - b * (uint32_t)(H * W), ho = __umulhi(rem, c.div_w), wo = rem - ho * (uint32_t)W;
    return (int)((b * (uint32_t)(H + 1) + ho) * (uint32_t)(W + 1) + wo);
}
// byte offset of the pixel at position q, or BEYOND for a zero; beyond the last image: beyond the tensor
__device__ __forceinline__ int window_source(const WindowGeom& c, int H, int W, int cpitch, uint32_t q)
{
    const uint32_t wp = (uint32_t)W + 1u;
    const uint32_t row = __umulhi(q, c.div_wp), col = q - row * wp, b = __umulhi(row, c.div_hp), h = row - b * (uint32_t)(H + 1);
    return col != 0 && h != 0 ? (int)(((row - b - 1u) * (uint32_t)W + col - 1u) * (uint32_t)cpitch) : BEYOND;
}
// [host] positions between tap (0, 0) of the first of n consecutive pixels and the end of tap (2, 2) of the last, at most: every end of a row
// inside costs one position, every end of an image W + 1 more; taps reach 2 (W + 1) + 2 positions further (some maps do reach this)
static inline int64_t window_positions(int64_t H, int64_t W, int64_t n)
{
    const int64_t wp = W + 1, hw = H * W, rows = (n - 1 + W - 1) / W, images = (n - 1 + hw - 1) / hw;
    return n + rows + images * wp + 2 * wp + 2;
}
// [host] whether the reciprocals are exact for R pixels and copies that reach `beyond` positions further
static inline bool window_geom(int64_t H, int64_t W, int64_t R, int64_t beyond, WindowGeom* c)
{
    if (W < 2 || H < 1 || R < 1) return false;
    const int64_t hw = H * W, wp = W + 1, images = (R + hw - 1) / hw + 1, positions = images * (H + 1) * wp + beyond, most = int64_t(1) << 32;
    if (positions * wp >= most || positions / wp * (H + 1) >= most || (R + beyond) * hw >= most) return false;
    auto reciprocal = [](int64_t d) { return (uint32_t)(((int64_t(1) << 32) + d - 1) / d); };   // (exact where x d < 2^32)
    c->div_hw = reciprocal(hw);
    c->div_w = reciprocal(W);
    c->div_wp = reciprocal(wp);
    c->div_hp = reciprocal(H + 1);
    return true;
}

// ---- what becomes of the accumulators of a forward pass: stored, stored with the goodness sums, or the output of a residual block
enum Conv3Result { C3_STORE, C3_STORE_GOODNESS, C3_RESIDUAL };
template <int WHAT> using Conv3Args = std::conditional_t<WHAT == C3_RESIDUAL, GemmResidualArgs, GemmArgs>;

// 64 rows from r0 on x 32 TJ columns from j0 on of a wavefront: EROWS rows at a time through its slice of LDS (EROWS x (TJ * 128 + 16) bytes), then whole
// row segments.
template <int TJ, int EROWS, typename F>
__device__ __forceinline__ void conv3_exchange(const v16i (&acc)[2][TJ], int ti, int h, int8_t* slice, F store)
{
    constexpr int EROW = TJ * 128 + 16, LPR = 8 * TJ, RPI = 64 / LPR;   // lanes per row, rows per store instruction
    const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
    if (lr / EROWS == h) {
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(v4i*)(slice + (lr % EROWS) * EROW + (tj * 32 + 8 * g + 4 * lh) * 4) =
                    (v4i){acc[ti][tj][4 * g], acc[ti][tj][4 * g + 1], acc[ti][tj][4 * g + 2], acc[ti][tj][4 * g + 3]};
    }
    wave_lds_fence();
    store([&](int r) { return *(const v4i*)(slice + (r * RPI + lane / LPR) * EROW + 16 * (lane % LPR)); });   // four columns of row r RPI + lane / LPR
    wave_lds_fence();
}
template <int WHAT, int TJ, int EROWS>
__device__ __forceinline__ void conv3_store(const Conv3Args<WHAT>& a, int z, int r0, int j0, const v16i (&acc)[2][TJ], int8_t* slice)
{
    constexpr int LPR = 8 * TJ, RPI = 64 / LPR, NR = EROWS / RPI, NH = 32 / EROWS;
    const int lane = threadIdx.x & 63, rl = lane / LPR, col = j0 + 4 * (lane % LPR);
    const bool in = col < a.J;
    if constexpr (WHAT == C3_RESIDUAL) {
        const ResidualScale rs = residual_scale(a.res, z);
        ResidualMax x = residual_max_of(a.res, r0);
        // What is added to the accumulators is fetched ahead of the exchanges: all of it where registers are left (64 -> 64 channels on 256 images of
        // 32x32, two passes: 67 us with the loads of each slice behind the stores of the one before, 54 this way), else one slice ahead.
        auto output = [&](auto codes) {
            constexpr bool CODES = decltype(codes)::value;
            constexpr int DEPTH = CODES && TJ <= 2 ? 2 * NH : 2;
            ResidualSkip<CODES> u[DEPTH][NR];
#pragma unroll
            for (int b = 0; b < DEPTH - (DEPTH == 2 ? 1 : 0); ++b) residual_load<CODES, LPR, NR>(a.res, z, r0 + EROWS * b, col, in, u[b]);
#pragma unroll
            for (int b = 0; b < 2 * NH; ++b) {
                if (DEPTH == 2 && b + 1 < 2 * NH) residual_load<CODES, LPR, NR>(a.res, z, r0 + EROWS * (b + 1), col, in, u[(b + 1) % DEPTH]);
                conv3_exchange<TJ, EROWS>(acc, b / NH, b % NH, slice, [&](auto row) {
                    residual_rows<CODES, LPR, NR>(a.res, rs, z, r0 + EROWS * b, col, in, u[b % DEPTH], x, [&](int r, int v[4]) {
                        const v4i w = row(r);
                        v[0] = w[0]; v[1] = w[1]; v[2] = w[2]; v[3] = w[3];
                    });
                });
            }
        };
        if (a.res.skip == FF_SKIP_IDENTITY) output(std::true_type{});   // (uniform)
        else output(std::false_type{});
        residual_max_store<64>(a.res, z, r0, x);
    } else {
        const bool whole_lines = (a.ldc & 31) == 0;
        int32_t* const C = a.C + z * a.st_c;
#pragma unroll
        for (int b = 0; b < 2 * NH; ++b)
            conv3_exchange<TJ, EROWS>(acc, b / NH, b % NH, slice, [&](auto row) {
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const int m = r0 + EROWS * b + r * RPI + rl;
                    const v4i v = row(r);
                    // not read again before the caches have been streamed over (see gemm_i8.hip); but where a column block starts or ends
                    // inside a line, its other half has to meet it in L2
                    if (m < a.I && in) {
                        if (whole_lines) __builtin_nontemporal_store(v, (v4i*)(C + (int64_t)m * a.ldc + col));
                        else *(v4i*)(C + (int64_t)m * a.ldc + col) = v;
                    }
                }
            });
    }
}

// Goodness sums of the same block (rows beyond the matrix hold zeros): one reduction and two atomics per wavefront and run of tiles in which its
// rows belong to one sample.  `next`: first row of the wavefront's next block in this pass, or -1; sq, vm: what earlier blocks of the run left.
template <int TJ>
__device__ __forceinline__ void conv3_goodness(const GemmArgs& a, int z, int r0, int next, const v16i (&acc)[2][TJ], unsigned long long& sq, int& vm)
{
    const uint32_t hw = (uint32_t)a.rows_per_sample;
    const int smp = r0 < a.I ? one_sample_of(r0, 64, a.I, hw) : -1;
#pragma unroll
    for (int ti = 0; ti < 2; ++ti) {
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) {
            int v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = acc[ti][tj][e];
            goodness_terms(a.relu, a.rshift, v, 16, sq, vm);
        }
        if (smp >= 0) {
            if (ti == 0) continue;
            if (next >= 0 && next < a.I && one_sample_of(next, 64, a.I, hw) == smp) continue;
            goodness_one(sq, vm, a.gsum + z * a.st_g + smp, a.vmax + z * a.st_g + smp);
        } else {
            goodness_runs(sq, vm, r0 + 32 * ti, a.I, hw, a.gsum + z * a.st_g, a.vmax + z * a.st_g);
        }
        sq = 0;
        vm = 0;
    }
}

}  // namespace ffi
