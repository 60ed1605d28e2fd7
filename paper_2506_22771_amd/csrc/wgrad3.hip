// Weight gradient of 3x3 stride-1 convolutions from one input window per step:
//     dW[n][(kh, kw, ci)] = sum over output pixels m of gy_t[n][m] * x[pixel of tap (kh, kw) at m][ci]
//
// The implicit loop of gemm_i8.hip (CONV 2) copies every input pixel once per tap into its stages, and its wavefronts' tiles read an LDS
// fragment for every multiply or two of three.  Here a workgroup owns 64 output channels x 32 input channels x all nine taps.  A step covers 512
// output pixels: 64 x 512 bytes of the gradient and ONE window of the input, which the nine taps read at nine offsets with the transposing LDS
// read.  The four quarters of a step's pixels go to four pairs of wavefronts, of which one has taps 0 .. 4 and the other 5 .. 8 (160 and 128
// accumulator registers: two wavefronts per SIMD), and whose sums meet in LDS at the end: seven and six fragment reads for ten and eight multiplies,
// and a quarter of the partial results that four workgroups of a split reduction would write.
//
// Window: positions of the input with one column of zeros in front of every row and one row of zeros in front of every image (the
// end of a row, or of an image, meets the zeros of the next), 32 bytes each.  Tap (kh, kw) of an output pixel then lies at a fixed
// distance from tap (0, 0) everywhere, for any map: no masks in the loop.  What a copy's lane fetches follows from its position by two
// multiplications; positions of zeros fail the buffer's range check.  A table of the pixels' tap (0, 0) is worked out three steps ahead, one
// pixel a thread.
//
// What bounds it: LDS traffic (104 KB of fragments and 27 KB of copies per 256 pixels, about 1230 of 1640 clocks; the multiplies need 1152), on large
// launches the power limit (1.7 to 1.9 GHz on random codes).  64 -> 128 channels, both sets of 256 images of 32x32: 2 x 38 us in the
// implicit loop, 2 x 23 here; a ResNet-18-shaped step 2061 -> 1943 us, 3-64-128-256 at 32x32 898 -> 825.
#include <math.h>

#include "window.hpp"

namespace ffi {

constexpr int W3_STEP = 512;                 // output pixels of a step
constexpr int W3_BN = 64, W3_BC = 32;        // output and input channels of a workgroup
constexpr int W3_T = 512;
constexpr int W3_P = W3_BN * W3_STEP;        // bytes of a step's gradient
constexpr int W3_STAGE = 64 * 1024;          // operands of a step, two of them
constexpr int W3_TABLE = 2 * W3_STAGE;       // tables of four steps behind them
constexpr int W3_LDS = W3_TABLE + 8 * 1024;   // (the exchange of the sums at the end takes 12 x 9 KB of it)

constexpr int W3_CW = (W3_STAGE - W3_P) / (W3_T * 16);   // copy instructions of a thread for a window, at most
constexpr int W3_POSITIONS = W3_CW * W3_T / 2;
static_assert(W3_TABLE + 4 * W3_STEP * 4 <= W3_LDS && 12 * 9 * 1024 <= W3_LDS && W3_LDS <= 160 * 1024, "LDS");

__device__ __forceinline__ v2i w3_tr_read8(const int8_t* p)   // (see gemm_i8.hip)
{
    typedef __attribute__((address_space(3))) v2i* lds_ptr;
    return __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_ptr)p);
}
struct Wgrad3Geom {   // filled in by the launch
    WindowGeom div;
    int32_t window, tiles_c, tiles, items, per_xcd;   // positions of a window; tiles and work items
};

// What a wavefront needs to know of its workgroup's share.
struct W3Item {
    const int8_t* P;
    const int8_t* Q;
    int32_t* C;
    int n0, ch0, kt0, nk;   // first output and input channel; steps kt0 .. kt0 + nk - 1
};

// Wavefronts of the taps T0 .. T0 + NT - 1.
template <int T0, int NT>
__device__ __forceinline__ void wgrad3_body(const GemmArgs& a, const Wgrad3Geom& c, const W3Item& it, int8_t* lds)
{
    constexpr int SUBS = W3_STEP / 128;   // 32-pixel pieces of a quarter
    constexpr int CPR = W3_STEP / 16, PROWS = W3_T / CPR;   // chunks of a staged row of the gradient; rows of a copy
    unsigned long long at0 = 0, at1 = 0, at2 = 0;   // phase marks of the clock probe (see gemm_i8.hip)
    if (a.clk) at0 = clock64();
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), slice = wave & 3;
    int* const tbl = (int*)(lds + W3_TABLE);
    const int rpad = (a.R + 15) & ~15;
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void*)it.P, 0, (int)(min(W3_BN, a.I - it.n0) * a.ldp), 0x00020000);
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)it.Q, 0, (int)a.p_bytes, 0x00020000);

    auto first_tap = [&](uint32_t m) { return window_first(c.div, a.H, a.W, m); };
    // chunk c of row r lies at c ^ (r & 15): sixteen rows, one chunk, sixteen bank groups
    static_assert(PROWS % 16 == 0, "one pattern for all copies");
    const int col_p = ((tid % CPR) ^ ((tid / CPR) & 15)) << 4;   // pixel of this thread's gradient chunks
    const int off_p = tid / CPR * (int)a.ldp;
    const int cq = it.ch0 + 16 * (tid & 1);
    const bool have_q = cq < a.Cin;
    auto copy = [&](int kt, int stage) {
        const int m0 = __builtin_amdgcn_readfirstlane(kt * W3_STEP);
        const unsigned base = (unsigned)(uintptr_t)(lds + stage * W3_STAGE);
        const int at_p = m0 + col_p < rpad ? off_p + m0 + col_p : BEYOND;
        const int more = PROWS * (int)a.ldp;
#pragma unroll
        for (int s = 0; s < W3_BN / PROWS; ++s)   // (beyond any buffer stays beyond: unsigned offsets)
            copy16(rp, (int)((uint32_t)at_p + (uint32_t)(s * more)), base + (unsigned)(s * W3_T + wave * 64) * 16u);
        const int q0 = __builtin_amdgcn_readfirstlane(first_tap((uint32_t)m0));
#pragma unroll
        for (int s = 0; s < W3_CW; ++s) {
            if (s * (W3_T / 2) + wave * 32 >= c.window) break;   // (uniform)
            const int at = window_source(c.div, a.H, a.W, a.cpitch, (uint32_t)(q0 + s * (W3_T / 2) + (tid >> 1)));
            copy16(rq, have_q && at != BEYOND ? at + cq : BEYOND, base + W3_P + (unsigned)(s * W3_T + wave * 64) * 16u);
        }
    };
    auto table = [&](int kt) {   // (one pixel a thread)
        const int m0 = kt * W3_STEP, m = m0 + tid;
        tbl[((kt - it.kt0) & 3) * W3_STEP + tid] = m < a.R ? (first_tap((uint32_t)m) - first_tap((uint32_t)m0)) * W3_BC : 0;
    };

    v16i acc[2][NT];
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ti][t][v] = 0;

    // fragments of one piece; those of the next are read while it is multiplied
    v4i fp[2][2], fq[2][NT];
    int ent[2 * SUBS];   // table entries of this lane's pixels of every piece, eight pixels apart each
    auto entries = [&](int j) {
#pragma unroll
        for (int e = 0; e < 2 * SUBS; ++e)
            ent[e] = tbl[(j & 3) * W3_STEP + 32 * SUBS * slice + 32 * (e >> 1) + 16 * lh + 8 * (e & 1) + ((lane & 15) >> 1)];
    };
    const int lane_q = W3_P + 16 * ((lane >> 4) & 1) + 8 * (lane & 1);
    const int pitch_h = (a.W + 1) * W3_BC;
    auto fragments = [&](auto piece, int stage) {
        constexpr int U = decltype(piece)::value, F = U & 1;
        const int8_t* const base = lds + stage * W3_STAGE;
        const int kc = 2 * SUBS * slice + 2 * U + lh;
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) fp[F][ti] = *(const v4i*)(base + (32 * ti + lr) * W3_STEP + ((kc ^ (lr & 15)) << 4));
        const int8_t* const lo = base + lane_q + ent[2 * U];
        const int8_t* const hi = base + lane_q + ent[2 * U + 1];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int kh = (T0 + t) / 3, kw = (T0 + t) % 3;
            const v2i l = w3_tr_read8(lo + kh * pitch_h + kw * W3_BC), h = w3_tr_read8(hi + kh * pitch_h + kw * W3_BC);
            fq[F][t] = (v4i){l.x, l.y, h.x, h.y};
        }
        // (the compiler would put the reads off until right before their use)
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int F) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int ti = 0; ti < 2; ++ti) acc[ti][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fq[F][t], fp[F][ti], acc[ti][t], 0, 0, 0);
    };

    const int nk = it.nk;
    copy(it.kt0, 0);
#pragma unroll 1
    for (int j = 0; j < 3; ++j)
        if (j < nk) table(it.kt0 + j);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (1 < nk) copy(it.kt0 + 1, 1);
    entries(0);
    fragments(std::integral_constant<int, 0>{}, 0);
    if (a.clk) at1 = clock64();
    int cur = 0;
    for (int j = 0; j < nk; ++j, cur ^= 1) {
        fragments(std::integral_constant<int, 1>{}, cur);
        multiply(0);
        fragments(std::integral_constant<int, 2>{}, cur);
        multiply(1);
        fragments(std::integral_constant<int, 3>{}, cur);
        if (j + 1 < nk) entries(j + 1);
        multiply(0);
        // The last fragments of this stage are in registers, and the copies of the next one have landed: behind the barrier that is
        // so for every wavefront.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
        // (one of the two wavefronts of a SIMD multiplies while the other's copies queue up)
        if (j + 1 < nk) fragments(std::integral_constant<int, 0>{}, cur ^ 1);
        if (T0 == 0 && j + 2 < nk) copy(it.kt0 + j + 2, cur);
        multiply(1);
        if (T0 != 0 && j + 2 < nk) copy(it.kt0 + j + 2, cur);
        if (j + 3 < nk) table(it.kt0 + j + 3);
    }
    if (a.clk) at2 = clock64();

    // The four quarters' sums meet in LDS, 32 output channels at a time: the wavefronts of quarter `slice` finish columns 8 slice .. + 7 of their
    // taps and get them from the other three ([columns][source][tap][lane], 16 bytes each).
    auto finish = [&](auto mine) {
        constexpr int M = decltype(mine)::value;
        const int ci = it.ch0 + 8 * M + 4 * lh;
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) {
            lds_barrier();   // (every wavefront has read its last fragments, or the sums of the first rows)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    if (g != M)
                        *(v4i*)(lds + (((g * 3 + (M < g ? M : M - 1)) * 9 + T0 + t) * 64 + lane) * 16) =
                            (v4i){acc[ti][t][4 * g], acc[ti][t][4 * g + 1], acc[ti][t][4 * g + 2], acc[ti][t][4 * g + 3]};
            lds_barrier();
            const int n = it.n0 + 32 * ti + lr;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                v4i v = {acc[ti][t][4 * M], acc[ti][t][4 * M + 1], acc[ti][t][4 * M + 2], acc[ti][t][4 * M + 3]};
#pragma unroll
                for (int s = 0; s < 3; ++s) v += *(const v4i*)(lds + (((M * 3 + s) * 9 + T0 + t) * 64 + lane) * 16);
                if (n >= a.I || ci >= a.cin_out) continue;
                int32_t* const dst = it.C + (int64_t)n * a.ldc + (T0 + t) * a.cin_out + ci;
                if ((a.cin_out & 3) == 0) {
                    *(v4i*)dst = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (ci + e < a.cin_out) dst[e] = v[e];
                }
            }
        }
    };
    switch (slice) {   // (uniform)
    case 0: finish(std::integral_constant<int, 0>{}); break;
    case 1: finish(std::integral_constant<int, 1>{}); break;
    case 2: finish(std::integral_constant<int, 2>{}); break;
    default: finish(std::integral_constant<int, 3>{}); break;
    }
    if (a.clk && tid == 0) {
        atomicAdd(a.clk + 2, at1 - at0);
        atomicAdd(a.clk + 3, at2 - at1);
        atomicAdd(a.clk + 4, (unsigned long long)clock64() - at2);
        atomicAdd(a.clk + 6, 1ull);
    }
}

__global__ __launch_bounds__(W3_T) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_wgrad3_i8(GemmArgs a, Wgrad3Geom c)
{
    __shared__ __attribute__((aligned(16))) int8_t lds[W3_LDS];
    // Workgroups go to the eight XCDs in turn; each XCD takes consecutive items, the tiles of one share of the pixels one after
    // the other, so that they meet in its L2.
    const int item = (int)(blockIdx.x & 7) * c.per_xcd + (int)(blockIdx.x >> 3);
    if (item >= c.items) return;
    unsigned long long clk0 = 0, rt0 = 0;
    if (a.clk) {
        clk0 = clock64();
        rt0 = wall_clock64();
    }
    const int share = item / c.tiles, tile = item - share * c.tiles;
    const int z = share / a.splits, split = share - z * a.splits, zp = z / a.nc, zc = z - zp * a.nc;
    const int steps = (((a.R + 15) & ~15) + W3_STEP - 1) / W3_STEP, per = (steps + a.splits - 1) / a.splits;
    W3Item it;
    it.n0 = tile / c.tiles_c * W3_BN;
    it.ch0 = tile % c.tiles_c * W3_BC;
    it.kt0 = split * per;
    it.nk = min(steps, it.kt0 + per) - it.kt0;
    it.P = a.P + zp * a.st_p + zc * a.st_p2 + (int64_t)it.n0 * a.ldp;
    it.Q = a.Q + zp * a.st_q + zc * a.st_q2;
    it.C = a.C + zp * a.st_c + zc * a.st_c2 + split * a.st_split;
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) < 4) wgrad3_body<0, 5>(a, c, it, lds);
    else wgrad3_body<5, 4>(a, c, it, lds);
    if (a.clk && threadIdx.x == 0) {
        atomicAdd(a.clk + 0, (unsigned long long)clock64() - clk0);
        atomicAdd(a.clk + 1, (unsigned long long)wall_clock64() - rt0);
    }
}

static bool wgrad3_fits(const ConvGeom& g, int64_t R, WindowGeom* c)
{
    return g.ks == 3 && g.pad == 1 && g.stride == 1 && window_geom(g.H, g.W, R, 2 * W3_POSITIONS, c) && window_positions(g.H, g.W, W3_STEP) <= W3_POSITIONS;
}

int wgrad3_split_evenly(int64_t R, int64_t splits)
{
    const int64_t steps = (((R + 15) & ~int64_t(15)) + W3_STEP - 1) / W3_STEP, sp = max((int64_t)1, min(splits, steps)), per = (steps + sp - 1) / sp;
    return (int)((steps + per - 1) / per);
}

// Where the launch is long enough for its beginning and its end (a first window, the exchange: 11 to 13 thousand clocks together, six of the
// implicit loop's): from 16384 pixels on, or with 384 steps of tiles.  One pass's weight gradient with its gradient quantiser, the implicit loop against
// this, us: 64 -> 128 channels, 256 images of 32x32 85.2 and 67.8; 128 -> 128, 256 of 16x16 42.8 and 37.6; 512 -> 512, 256 of 4x4 (512 steps) 35.3
// and 30.4, 128 of 4x4 (512) 20.7 and 18.0; 64 -> 64, 16 of 32x32 20.5 and 17.6; 32 -> 32, 38 of 28x28 21.3 and 15.8; 240 -> 80, 16 of 28x28 (400)
// 24.7 and 22.9; 72 -> 200, 200 of 28x28 114 and 97; 512 -> 512, 60 of 16x16 71.9 and 55.9.  On the line 96 -> 96, 64 of 16x16, 22.5 and 23.3.
// Below it 32 -> 32, 128 of 8x8, 16.5 and 19.2; 64 -> 96, 32 of 14x14, 16.5 and 18.5; 512 -> 512, 38 of 4x4 (256 steps), 13.6 and 15.7; 64 -> 200, 100 of
// 9x9, 20.7 both.  Strided layers were measured with windows of all the pixels in between, 256 outputs a step: 64 -> 128, 256 of 32x32 38.0 and 35.5, but 128 -> 256 of
// 16x16 30.1 and 33.3, 256 -> 512 of 8x8 28.3 and 30.4: they keep the implicit loop.
int wgrad3_splits(const ConvGeom& g, int64_t N, int64_t R, int nb)
{
    WindowGeom c;
    if (g.Cin < 16 || !wgrad3_fits(g, R, &c)) return 0;
    const int64_t tiles = ((N + W3_BN - 1) / W3_BN) * ((g.Cin + W3_BC - 1) / W3_BC) * nb, steps = (R + W3_STEP - 1) / W3_STEP;
    if (R < 16384 && tiles * steps < 384) return 0;
    // 512 pixels take about 1.1 us, writing and adding up a workgroup's partial result 0.012: the least of 1.1 R / 512 splits + 0.012 tiles splits,
    // in one round of workgroups.  (With 0.03 for a result 128 -> 128, 256 of 16x16, 41.2 instead of 37.6 us, 64 -> 64, 16 of 32x32, 20.6 instead of
    // 17.2; with 0.007 256 -> 256, 128 of 8x8, 28.1 instead of 26.5.)
    const int64_t best = (int64_t)(0.5 + sqrt(46.0 / 256 * (double)R / (double)tiles));
    return wgrad3_split_evenly(R, min(best, num_cus() / tiles));
}

hipError_t launch_wgrad3(const GemmArgs& a_in, const ConvGeom& g, hipStream_t s)
{
    GemmArgs a = a_in;
    if (a.nc < 1) a.nc = 1;
    if (a.I <= 0 || a.nb < 1) return hipSuccess;
    Wgrad3Geom c;
    if (!wgrad3_fits(g, a.R, &c.div) || a.conv != 2 || !a.C || a.gsum || a.upd_w || a.residual || a.nb % a.nc != 0 || (a.Cin & 15) != 0 || a.Cin > a.cpitch ||
        a.cin_out > a.Cin || a.p_bytes >= (int64_t(1) << 31) || a.ldp >= (int64_t(1) << 22) || a.R % (a.Ho * a.Wo) != 0 || a.splits < 1 ||
        wgrad3_split_evenly(a.R, a.splits) != a.splits)
        return hipErrorInvalidValue;
    c.window = (int32_t)window_positions(g.H, g.W, W3_STEP);
    c.tiles_c = (a.Cin + W3_BC - 1) / W3_BC;
    c.tiles = (a.I + W3_BN - 1) / W3_BN * c.tiles_c;
    const int64_t items = (int64_t)c.tiles * a.nb * a.splits;
    if (items > (1 << 24)) return hipErrorInvalidValue;
    c.items = (int32_t)items;
    c.per_xcd = (int32_t)((items + 7) / 8);
    const dim3 grid((unsigned)c.per_xcd * 8u), block(W3_T);
    hipLaunchKernelGGL(k_wgrad3_i8, grid, block, 0, s, a, c);
    return hipGetLastError();
}

}  // namespace ffi
