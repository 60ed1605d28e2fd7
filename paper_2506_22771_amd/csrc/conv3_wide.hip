// Forward contraction of 3x3 stride-1 convolutions of more than 64 input channels: one input window per tile and 64 channels, the
// weights streamed tap by tap.
//
// The implicit loop of gemm_i8.hip copies every input pixel nine times.  Here a tile of output pixels goes through its input channels in groups of 64:
// a group's window (zero-bordered positions of 64 bytes, window.hpp) is in LDS once and the nine taps read it at nine offsets; a step is one tap, whose
// 64 weights of every column come in a ring of three.  The copies of a step go out three steps ahead, a piece of the next window with each of a group's
// first steps, and on across the tiles of a workgroup: a launch waits for memory once, at its beginning.  Two workgroups share a compute unit, so
// that one's stores run under the other's multiplies.
//
// What bounds it: a tile of 256 x 128 of 128 channels takes 22 thousand clocks of main loop beside another (18.4 of multiplies), 8 of goodness sums (a 64-bit
// multiply-add and a maximum per accumulator) and 16 to 23 of stores (the accumulators leave at 5.2 TB/s). The two workgroups of a compute unit start together and
// stay in step, so that little of the three overlaps: 128 -> 256 on 256 images of 16x16 takes 33 us, 13 of stores and 11 of multiplies.  A wave priority that
// lets one of the two run ahead changed nothing, stores without the streaming hint were slower (that layer's single operations 70.8 instead of 69.1 us; 73.6 with
// the implicit loop).
//
// LDS: 16-byte chunks of a position or a weight row are XOR-swizzled by its number / 4, so that sixteen consecutive ones put a chunk into sixteen
// different bank groups, at any offset.
#include "window.hpp"

namespace ffi {

constexpr int CW_T = 256, CW_RING = 3;

// WM of the four wavefronts side by side over the pixels, 64 pixels x 32 TJ columns each; CW copy instructions of a thread per window
// (64 positions each).
template <int WM, int TJ, int CW> struct CwShape {
    static constexpr int BM = 64 * WM, BN = 32 * TJ * (4 / WM);
    static constexpr int WINDOW = CW * CW_T * 16, WEIGHTS = BN * 64;   // bytes of a window, of a step's weights
    static constexpr int EROWS = 8, ESLICE = EROWS * (TJ * 128 + 16);  // staging of a wavefront's stores, in the window that was read last
    static constexpr int LDS = 2 * WINDOW + CW_RING * WEIGHTS;
    static_assert(LDS <= 80 * 1024 && 4 * ESLICE <= WINDOW, "LDS");
    // Piece s of the next window goes out in step s, and the wait of a step leaves the copies of the step before it in flight: an eighth piece
    // might still be on its way when step 8 reads that window.
    static_assert(CW <= 7, "pieces of a window");
};

template <int WHAT, int WM, int TJ, int CW>
__global__ __launch_bounds__(CW_T) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_conv3_wide_i8(Conv3Args<WHAT> a, WindowGeom c, int ncb)
{
    using S = CwShape<WM, TJ, CW>;
    constexpr int BM = S::BM, BN = S::BN, WCH = BN / 64;   // WCH: copy instructions of a thread for a step's weights
    __shared__ __attribute__((aligned(16))) int8_t lds[S::LDS];
    int8_t* const ring = lds + 2 * S::WINDOW;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave % WM, wn = wave / WM;
    // Workgroups go to the eight XCDs in turn: those of one XCD share their windows between column blocks.
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int j0 = idx % ncb * BN;
    const int tiles_z = (a.I + BM - 1) / BM, tiles = tiles_z * a.nb;
    const int slots = (int)(gridDim.x / (unsigned)ncb), t0 = xcd * (slots >> 3) + idx / ncb;   // this workgroup's tiles: t0, t0 + slots, ...
    if (t0 >= tiles) return;
    const int groups = (a.Cin + 63) >> 6;
    const int pitch_h = (a.W + 1) * 64;

    // where this thread's chunks of the window being copied come from (first channel group)
    int off[CW];
    __amdgpu_buffer_rsrc_t rp;
    auto aim = [&](int t) {
        const int z = t / tiles_z, m0 = (t - z * tiles_z) * BM;
        rp = __builtin_amdgcn_make_buffer_rsrc((void*)(a.P + z * a.st_p), 0, (int)a.p_bytes, 0x00020000);
        const int q0 = __builtin_amdgcn_readfirstlane(window_first(c, a.H, a.W, (uint32_t)m0));
#pragma unroll
        for (int s = 0; s < CW; ++s) {
            const int p = (s * CW_T + tid) >> 2, k = (tid & 3) ^ ((p >> 2) & 3);
            const int at = window_source(c, a.H, a.W, a.cpitch, (uint32_t)(q0 + p));
            off[s] = at == BEYOND ? BEYOND : at + 16 * k;
        }
    };
    auto copy_window = [&](int s, int g, int buf) {   // piece s
        const int k = (tid & 3) ^ ((((s * CW_T + tid) >> 2) >> 2) & 3);
        const bool in = 64 * g + 16 * k < a.Cin;   // (past the last channels: zeros, not the next pixel)
        copy16(rp, in ? (int)((uint32_t)off[s] + 64u * (uint32_t)g) : BEYOND, (unsigned)(uintptr_t)(lds + buf * S::WINDOW + (s * CW_T + wave * 64) * 16));
    };
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)(a.Q + (int64_t)j0 * a.ldq), 0, (int)(min(BN, a.J - j0) * a.ldq), 0x00020000);
    int off_w[WCH];
#pragma unroll
    for (int s = 0; s < WCH; ++s) {
        const int n = (s * CW_T + tid) >> 2;
        off_w[s] = n * (int)a.ldq + 16 * ((tid & 3) ^ ((n >> 2) & 3));
    }
    auto copy_weights = [&](int tap, int g, int slot, bool zeros = false) {   // (beyond a row's last channels: the next tap's, against zeros of the window)
        const uint32_t at = zeros ? (uint32_t)BEYOND : (uint32_t)(tap * a.cin_out + 64 * g);
#pragma unroll
        for (int s = 0; s < WCH; ++s)
            copy16(rq, (int)((uint32_t)off_w[s] + at), (unsigned)(uintptr_t)(ring + slot * S::WEIGHTS + (s * CW_T + wave * 64) * 16));
    };

    int ent[2];   // bytes from the window's start to tap (0, 0) of this lane's pixels
    auto enter = [&](int t) {
        const int m0 = (t - t / tiles_z * tiles_z) * BM;
        const int q0 = __builtin_amdgcn_readfirstlane(window_first(c, a.H, a.W, (uint32_t)m0));
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
            ent[ti] = (window_first(c, a.H, a.W, (uint32_t)min(m0 + 64 * wm + 32 * ti + lr, a.I - 1)) - q0) * 64;
    };
    const int row_w = wn * TJ * 32 + lr, lane_w = row_w * 64 + (((lh ^ (row_w >> 2)) & 3) << 4);
    v4i fp[2][2], fq[2][TJ];
    auto fragments = [&](auto piece, auto tap, int buf, int slot) {   // 32 of the group's channels
        constexpr int U = decltype(piece)::value, KH = decltype(tap)::value / 3, KW = decltype(tap)::value % 3;
        const int8_t* const win = lds + buf * S::WINDOW;
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) {
            const int px = ent[ti] + KH * pitch_h + KW * 64;
            fp[U][ti] = *(const v4i*)(win + px + ((((px >> 8) & 3) ^ (2 * U + lh)) << 4));
        }
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) fq[U][tj] = *(const v4i*)(ring + slot * S::WEIGHTS + tj * 2048 + (U ? lane_w ^ 32 : lane_w));
        __builtin_amdgcn_sched_barrier(0);   // (the compiler would put the reads off until right before their use)
    };
    v16i acc[2][TJ];
    auto multiply = [&](int U) {
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) acc[ti][tj] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fq[U][tj], fp[U][ti], acc[ti][tj], 0, 0, 0);
    };
    constexpr std::integral_constant<int, 0> P0{};
    constexpr std::integral_constant<int, 1> P1{};

    aim(t0);
#pragma unroll
    for (int s = 0; s < CW; ++s) copy_window(s, 0, 0);
#pragma unroll
    for (int s = 0; s < CW_RING; ++s) copy_weights(s, 0, s);
    enter(t0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * WCH) : "memory");
    lds_barrier();
    fragments(P0, std::integral_constant<int, 0>{}, 0, 0);

    unsigned long long sq = 0;   // goodness sum and maximum of the sample (or block of rows) at hand
    int vm = 0, buf = 0;
    for (int t = t0; t < tiles; t += slots) {
        const int z = t / tiles_z, i0 = (t - z * tiles_z) * BM;
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[ti][tj][v] = 0;
        for (int g = 0; g < groups; ++g) {
            const bool last = g + 1 == groups;
            // the copies of the first steps of a tile were waited for ahead of the last tile's stores
            const bool fresh = g == 0 && t > t0;
            asm volatile("" : "+v"(ent[0]), "+v"(ent[1]));   // (or the compiler keeps the addresses of all nine taps, beyond the registers there are)
            auto step = [&](auto tap_, auto next_) {
                constexpr int TAP = decltype(tap_)::value;
                constexpr int SLOT = TAP % CW_RING, AHEAD = (TAP + 3) % 9;
                fragments(P1, tap_, buf, SLOT);
                multiply(0);
                // What the next step reads has landed: all but the copies that went out one step ago.
                if (!(fresh && TAP < 2)) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(WCH + (TAP >= 1 && TAP <= CW ? 1 : 0)) : "memory");
                lds_barrier();
                if (TAP == 0 && last) {
                    if (t + slots < tiles) {
                        aim(t + slots);
                    } else {   // the counted waits want the copies of a next tile all the same: zeros, which cost no memory traffic
#pragma unroll
                        for (int s = 0; s < CW; ++s) off[s] = BEYOND;
                    }
                }
                if (TAP == 8 && last && t + slots < tiles) enter(t + slots);
                fragments(P0, next_, TAP == 8 ? buf ^ 1 : buf, (TAP + 1) % CW_RING);
                if (TAP < CW) copy_window(TAP, last ? 0 : g + 1, buf ^ 1);
                copy_weights(AHEAD, TAP + 3 < 9 ? g : (last ? 0 : g + 1), SLOT, TAP + 3 >= 9 && last && t + slots >= tiles);
                multiply(1);
            };
#define FFI_TAP(n) step(std::integral_constant<int, n>{}, std::integral_constant<int, (n + 1) % 9>{})
            FFI_TAP(0); FFI_TAP(1); FFI_TAP(2); FFI_TAP(3); FFI_TAP(4); FFI_TAP(5); FFI_TAP(6); FFI_TAP(7); FFI_TAP(8);
#undef FFI_TAP
            buf ^= 1;
        }
        if (i0 + BM > a.I) {   // (uniform) rows beyond the matrix
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
                if (i0 + 64 * wm + 32 * ti + lr >= a.I)
#pragma unroll
                    for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[ti][tj][v] = 0;
        }
        const int r0 = i0 + 64 * wm;
        if constexpr (WHAT == C3_STORE_GOODNESS) conv3_goodness<TJ>(a, z, r0, -1, acc, sq, vm);
        // copies before stores: they complete in issue order, and nothing of this workgroup may land after its end
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        conv3_store<WHAT, TJ, S::EROWS>(a, z, r0, j0 + wn * TJ * 32, acc, lds + (buf ^ 1) * S::WINDOW + wave * S::ESLICE);
    }
}

// Workgroups for a column block at once (two for each compute unit in all), and how many tiles of a block each of them goes through at most.
static int64_t conv3_wide_slots(int ncb) { return max(1, num_cus() / 8 * 2 / ncb) * 8; }
static int64_t conv3_wide_rounds(int64_t tiles, int ncb) { return (tiles + conv3_wide_slots(ncb) - 1) / conv3_wide_slots(ncb); }

template <int WM, int TJ, int CW>
static hipError_t launch_conv3_wide_cfg(const GemmArgs& a, const WindowGeom& c, hipStream_t s)
{
    using S = CwShape<WM, TJ, CW>;
    static_assert(S::BN == 128, "conv3_wide_ok");
    const int ncb = (a.J + S::BN - 1) / S::BN;
    const int64_t tiles = ((int64_t)a.I + S::BM - 1) / S::BM * a.nb;
    // as many workgroups per column block as give each the same number of tiles
    const int64_t rounds = conv3_wide_rounds(tiles, ncb), slots = ((tiles + rounds - 1) / rounds + 7) / 8 * 8;
    const dim3 grid((unsigned)(slots * ncb));
    if (a.residual) hipLaunchKernelGGL((k_conv3_wide_i8<C3_RESIDUAL, WM, TJ, CW>), grid, dim3(CW_T), 0, s, GemmResidualArgs{a, *a.residual}, c, ncb);
    else if (a.gsum) hipLaunchKernelGGL((k_conv3_wide_i8<C3_STORE_GOODNESS, WM, TJ, CW>), grid, dim3(CW_T), 0, s, a, c, ncb);
    else hipLaunchKernelGGL((k_conv3_wide_i8<C3_STORE, WM, TJ, CW>), grid, dim3(CW_T), 0, s, a, c, ncb);
    return hipGetLastError();
}

// copy instructions per window, or 0 where it does not fit
static int conv3_wide_copies(const GemmArgs& a, int bm) { return (int)((window_positions(a.H, a.W, bm) + 63) / 64); }

static bool conv3_wide_fits(const GemmArgs& a, WindowGeom* c)
{
    return a.conv == 1 && a.ks == 3 && a.stride == 1 && a.pad == 1 && (a.J & 3) == 0 && a.J >= 1 && a.splits == 1 && a.nb >= 1 && a.nb <= 2 &&
           a.p_bytes < (int64_t(1) << 30) && a.H == a.Ho && a.W == a.Wo && (int64_t)a.I * a.cpitch == a.p_bytes && (a.cin_out & 3) == 0 &&
           (a.Cin & 15) == 0 && a.cin_out <= a.Cin && a.Cin <= a.cpitch && a.rows_per_sample == a.H * a.W && a.ldq < (int64_t(1) << 22) &&
           (a.J + 63) / 64 <= num_cus() / 4 && window_geom(a.H, a.W, a.I, 4096, c) && conv3_wide_copies(a, 128) <= 6;
}

// Tiles of 256 x 128, or of 128 x 128 in launches of fewer than one such tile per compute unit and for maps whose windows of 256 pixels do not fit.
static bool conv3_wide_large(const GemmArgs& a)
{
    return conv3_wide_copies(a, 256) <= 7 && ((int64_t)a.I + 255) / 256 * a.nb * ((a.J + 127) / 128) >= num_cus();
}

// Where this is faster than the implicit loop, whose tiles are finer and which starts 2 us sooner: short launches of few channel groups stay with it, and on
// small maps, whose windows hold more zeros, the two are close.  ff_layer_forward of one pass, the implicit loop and this, us:
//  - Channel groups at least three quarters full (72 -> 128, 256 images of 32x32 61 and 67), more than 64 columns (96 -> 64, 256 of 32x32 45 and 52).
//  - Up to 3 x 2^25 outputs: 128 -> 256, 305 of 32x32 (80 M) 161 and 141, 512 (134 M) 231 and 244, 6103 of 8x8 (100 M) 166 and 170.  (From 256
//    channels on it stays 2 to 7 % ahead beyond.)
//  - Maps without windows of 256 pixels up to 5 x 2^22 outputs (128 -> 256 on 24x82, 33 images 99 and 65, 133 images 141 and 157), from three groups
//    on up to twice that (256 -> 256, 66 images 127 and 122, 133 images 201 and 218).
//  - Five groups and more everywhere: 320 -> 320, 56 of 3x3 19.2 and 18.2; 512 -> 512, 32 of 28x28 118 and 74.
//  - Three and four on maps from 16x16 on (192 -> 200, 1 of 20x30 15.1 and 14.3); below from 3 x 2^16 outputs on (256 -> 128, 5 of 10x10 (64 K) 15.5 and 16.0,
//    192 -> 68, 14 of 14x14 (187 K) 15.3 and 14.3), below 8x8 with more than one tile for every second compute unit (256 -> 128, 1024 of 4x4 17.7 and 17.9, 6272
//    of 4x4 49.7 and 43.5).
//  - Two from 2^19 outputs on: 128 -> 128, 2 of 28x28 (201 K) 12.2 and 12.8, 7 (702 K) 15.5 and 14.3; maps below 16x16 from 2^20 on: 96 -> 96, 10 of 14x14
//    11.4 and 12.4, 128 -> 128, 64 of 14x14 15.2 and 14.7.  Maps from 4x4 to below 14x14 in rounds that are three quarters full, or from the third on, with tiles of
//    256 x 128 only from 97 channels on: 128 -> 128, 512 of 8x8 15.9 and 15.6, 784 of 8x8 24.2 and 20.7, 128 -> 256, 549 of 6x6 18.0 and 20.2; 96 -> 96, 8192 of 4x4
//    30.0 and 31.7, 128 -> 128 34.3 and 33.6; 112 -> 320, 867 of 5x5, whose 3 x 170 tiles make two rounds, 23.0 and 32.0; 96 -> 96, 227 of 3x3 10.8 and 13.1.
//  - Not one large tile per compute unit in one column block: 128 -> 128, 1024 of 8x8 20.4 and 23.2.
bool conv3_wide_ok(const GemmArgs& a)
{
    WindowGeom c;
    const int groups = (a.Cin + 63) / 64, pixels = a.H * a.W;
    const int64_t outputs = (int64_t)a.I * a.J * a.nb;
    if (a.Cin <= 64 || 4 * a.cin_out < 192 * groups || a.J <= 64 || outputs > (int64_t(3) << 25) || !conv3_wide_fits(a, &c)) return false;
    if (conv3_wide_copies(a, 256) > 7 && outputs > (int64_t(5) << (groups == 2 || pixels < 16 ? 22 : 23))) return false;
    if (groups >= 5) return true;
    const bool large = conv3_wide_large(a);
    const int bm = large ? 256 : 128, ncb = (a.J + 127) / 128;
    const int64_t tiles = ((int64_t)a.I + bm - 1) / bm * a.nb, rounds = conv3_wide_rounds(tiles, ncb);   // of a column block
    if (large && pixels < 256 && ncb == 1 && tiles <= num_cus()) return false;
    if (groups > 2) return pixels >= 256 || (pixels < 64 ? 2 * tiles * ncb > num_cus() : outputs >= 3 << 16);
    if (pixels >= 196) return outputs >= 1 << (pixels < 256 ? 20 : 19);
    return pixels >= 16 && (rounds > 2 || 4 * tiles >= 3 * rounds * conv3_wide_slots(ncb)) && (!large || a.cin_out > 96);
}

hipError_t launch_conv3_wide(const GemmArgs& a, hipStream_t s)
{
    WindowGeom c;
    if (a.I <= 0 || a.J <= 0) return hipSuccess;
    if (!conv3_wide_fits(a, &c) || (!a.C && !a.residual) || (a.gsum && (a.residual || !a.vmax))) return hipErrorInvalidValue;
    if (a.residual && (a.residual->M != a.I || a.residual->N != a.J || a.residual->rows_per_sample < RESIDUAL_MIN_ROWS)) return hipErrorInvalidValue;
    if (conv3_wide_large(a)) return conv3_wide_copies(a, 256) <= 6 ? launch_conv3_wide_cfg<4, 4, 6>(a, c, s) : launch_conv3_wide_cfg<4, 4, 7>(a, c, s);
    return conv3_wide_copies(a, 128) <= 4 ? launch_conv3_wide_cfg<2, 2, 4>(a, c, s) : launch_conv3_wide_cfg<2, 2, 6>(a, c, s);
}

}  // namespace ffi
