// Forward contraction of 3x3 stride-1 convolutions of more than 64 input channels: one input window per tile and 64 channels, the
// weights streamed tap by tap.
//
// The implicit loop of gemm_i8.hip copies every input pixel nine times.  Here a tile of output pixels goes through its input channels in groups of 64:
// a group's window (zero-bordered positions of 64 bytes, window.hpp) is in LDS once and the nine taps read it at nine offsets; a step is one tap, whose
// 64 weights of every column come in a ring of three.  The copies of a step go out three steps ahead, a piece of the next window with each of a group's
// first steps, and on across the tiles of a workgroup: a launch waits for memory once, at its beginning.  Two workgroups share a compute unit, so
// that one's stores run under the other's multiplies.
//
// What bounds it: the int32 accumulators, which leave at 5.2 TB/s while hardly anything else happens (two workgroups of a compute unit start
// together), then the multiplies: a tile of 256 x 128 of 128 channels takes 22 thousand clocks of main loop beside another (18.4 of multiplies), 8 of goodness
// sums and 16 to 23 of stores.  A wave priority that lets one of the two run ahead changed nothing, stores without the streaming hint were slower (the single
// operations of 128 -> 256 on 256 images of 16x16 70.8 instead of 69.1 us; 73.6 with the implicit loop).
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

template <int WM, int TJ, int CW>
static hipError_t launch_conv3_wide_cfg(const GemmArgs& a, const WindowGeom& c, hipStream_t s)
{
    using S = CwShape<WM, TJ, CW>;
    const int ncb = (a.J + S::BN - 1) / S::BN, per_xcd = num_cus() / 8 * 2;
    const int64_t tiles = ((int64_t)a.I + S::BM - 1) / S::BM * a.nb;
    // as many workgroups per column block as give each the same number of tiles
    const int64_t most = max(1, per_xcd / ncb) * 8, rounds = (tiles + most - 1) / most;
    const int64_t slots = ((tiles + rounds - 1) / rounds + 7) / 8 * 8;
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

// Forward launches of one pass, the implicit loop against this, us: 128 -> 256 channels, 64 images of 32x32 46.4 and 36.8, 256 images 122 and 104; 128 ->
// 128, 128 of 32x32 42.4 and 37.1, 512 131 and 112; 256 -> 256, 256 of 32x32 185 and 170; 96 -> 96, 256 of 28x28 56.7 and 51.9; 160 -> 200, 64 of
// 20x20 36.1 and 26.9; 128 -> 256, 512 of 16x16 58.3 and 55.8; 512 -> 512, 512 of 4x4 30.0 and 27.9; 128 -> 128, 512 of 16x16 32.5 and 32.9; 256 -> 256,
// 512 of 8x8 28.8 and 29.4, 474 of 7x7 23.7 and 25.3.  Not where a quarter of the groups' channels is padding (72 -> 64, 512 of 32x32 76 and 99), not for
// up to 64 columns (96 -> 64, 256 of 32x32 42.4 and 47.3), and not beyond 3 x 2^25 outputs, more than the memory-side cache: 128 -> 256, 512 of 32x32
// (134 M) 241 and 248, in a step 215 and 230.
bool conv3_wide_ok(const GemmArgs& a)
{
    WindowGeom c;
    return a.Cin > 64 && 4 * a.cin_out >= 192 * ((a.Cin + 63) / 64) && a.J > 64 && (int64_t)a.I * a.J * a.nb <= (int64_t(3) << 25) && conv3_wide_fits(a, &c);
}

hipError_t launch_conv3_wide(const GemmArgs& a, hipStream_t s)
{
    WindowGeom c;
    if (a.I <= 0 || a.J <= 0) return hipSuccess;
    if (!conv3_wide_fits(a, &c) || (!a.C && !a.residual) || (a.gsum && (a.residual || !a.vmax))) return hipErrorInvalidValue;
    if (a.residual && (a.residual->M != a.I || a.residual->N != a.J || a.residual->rows_per_sample < RESIDUAL_MIN_ROWS)) return hipErrorInvalidValue;
    const int copies = conv3_wide_copies(a, 256);
    const int64_t tiles = ((int64_t)a.I + 255) / 256 * a.nb * ((a.J + 127) / 128);
    if (copies <= 7 && tiles >= num_cus()) return copies <= 6 ? launch_conv3_wide_cfg<4, 4, 6>(a, c, s) : launch_conv3_wide_cfg<4, 4, 7>(a, c, s);
    return conv3_wide_copies(a, 128) <= 4 ? launch_conv3_wide_cfg<2, 2, 4>(a, c, s) : launch_conv3_wide_cfg<2, 2, 6>(a, c, s);
}

}  // namespace ffi
