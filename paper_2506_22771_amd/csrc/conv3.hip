// Forward contraction of 3x3 stride-1 convolutions of up to 64 input channels: resident weights, one input window per tile.
//
// The implicit loop of gemm_i8.hip copies every input pixel nine times (once per tap) and meets at a barrier every 128
// reduction bytes; with five or fewer such steps per tile that, not the multiplies, is what its launches last for (64 -> 64
// channels, 512 images of 32x32: 66 us, 56 without a single store, 16 of multiplies; 37 here, 26 without stores).  Here a workgroup keeps the weights of
// its 64 (or 32) output channels in LDS for the whole launch and walks over tiles of 256 output pixels.  With stride 1 and
// padding 1 the input pixel of tap (kh, kw) of output pixel m is m + (kh - 1) W + kw - 1 in the flat NHWC tensor: a tile's
// window is 256 + 2 W + 2 consecutive pixels, one contiguous copy, and the nine taps read it at nine offsets.  Taps outside
// the image read a pixel of zeros behind the window.  The copy of the next window runs under the multiplies of this one; a
// tile has two barriers.
//
// LDS rows: a weight row has an odd number of 16-byte chunks, a pixel one or three, or two or four XOR-swizzled by its address,
// so that sixteen consecutive rows or pixels fall into sixteen different bank groups at any offset.
#include "window.hpp"

namespace ffi {

constexpr int C3_PIX = 256;        // output pixels of a tile
constexpr int C3_SLOTS = 7;        // copy instructions of a thread per window, at most

// KT: 32-byte pieces of a pixel (C_in <= 32 KT).  A workgroup has four wavefronts of 64 pixels x 32 TJ columns.
template <int KT, int TJ> struct C3Shape {
    static constexpr int T = 256, BN = 32 * TJ;
    static constexpr int KW = 288 * KT + 16;                // bytes of a weight row
    static constexpr int LDS = 80 * 1024;                   // two workgroups per compute unit
    static constexpr int BUF = (LDS - BN * KW) / 2 / 1024 * 1024;
    static constexpr int EROWS = 16, ESLICE = EROWS * (TJ * 128 + 16);   // staging of a wavefront's stores, in the window just read
    static_assert(BUF >= 4 * ESLICE, "staging");
};

template <int WHAT, int KT, int TJ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_conv3_i8(Conv3Args<WHAT> a, Conv3Geom c)
{
    using S = C3Shape<KT, TJ>;
    constexpr int T = S::T, BN = S::BN, KW = S::KW;
    __shared__ __attribute__((aligned(16))) int8_t lds[S::LDS];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups go to the eight XCDs in turn: those of one XCD share their windows between column blocks.
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int j0 = idx % c.ncb * BN;
    const int tiles_z = (a.I + C3_PIX - 1) / C3_PIX;
    const int t0 = (idx / c.ncb * 8 + xcd) * c.per, t1 = min(t0 + c.per, tiles_z * a.nb);   // consecutive tiles

    // where this thread's chunks of a window come from (bytes from its first pixel; negative: a chunk of zeros)
    int off[C3_SLOTS];
#pragma unroll
    for (int s = 0; s < C3_SLOTS; ++s) {
        const int at = s * T + tid, p = at / c.pc, k = at - p * c.pc, kc = k ^ ((at * 16 >> 8) & c.swz_mask);
        off[s] = p < c.window && kc < c.cpp ? p * a.cpitch + kc * 16 : (int)0x80000000;
    }
    auto copy_window = [&](int t, int buf) {
        const int z = t / tiles_z, m0 = (t - z * tiles_z) * C3_PIX;
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void*)(a.P + z * a.st_p), 0, (int)a.p_bytes, 0x00020000);
        const int start = (m0 - a.W - 1) * a.cpitch;
        const unsigned base = (unsigned)(uintptr_t)(lds + BN * KW + buf * S::BUF);
#pragma unroll
        for (int s = 0; s < C3_SLOTS; ++s)
            if (s * T + wave * 64 < c.chunks) {   // (uniform in a wavefront)
                const int at = (int)((uint32_t)off[s] + (uint32_t)start);   // before or beyond the tensor: zeros
                copy16(rp, at < 0 ? BEYOND : at, base + (unsigned)(s * T + wave * 64) * 16u);
            }
    };
    if (t0 < t1) copy_window(t0, 0);
    // weights: tap by tap, 32 KT bytes each; zeros where a tap's channels end and in rows beyond the matrix
    for (int e = tid; e < BN * 18 * KT; e += T) {
        const int n = e / (18 * KT), r = e - n * (18 * KT), tap = r / (2 * KT), k = r - tap * (2 * KT);
        v4i v = {0, 0, 0, 0};
        if (j0 + n < a.J && k < c.cpp) {
            const int* src = (const int*)(a.Q + (int64_t)(j0 + n) * a.ldq + tap * a.cin_out + 16 * k);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = src[i];
        }
        *(v4i*)(lds + n * KW + r * 16) = v;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    const int HW = a.H * a.W;
    unsigned long long sq = 0;   // goodness sum and maximum of the sample (or block of rows) at hand
    int vm = 0;
    int cur = 0;
    for (int t = t0; t < t1; ++t, cur ^= 1) {
        if (t + 1 < t1) copy_window(t + 1, cur ^ 1);
        const int z = t / tiles_z, i0 = (t - z * tiles_z) * C3_PIX;
        int8_t* const win = lds + BN * KW + cur * S::BUF;
        int row[2], mask[2];   // this lane's pixel of block ti (from i0) and which of its taps lie inside the image
#pragma unroll
        for (int ti = 0; ti < 2; ++ti) {
            row[ti] = 64 * wave + 32 * ti + lr;
            const int m = i0 + row[ti], rem = (int)((uint32_t)m % (uint32_t)HW), ho = (int)((uint32_t)rem / (uint32_t)a.W), wo = rem - ho * a.W;
            const int cols = (wo > 0 ? 1 : 0) | 2 | (wo + 1 < a.W ? 4 : 0);
            mask[ti] = m >= a.I ? 0 : (ho > 0 ? cols : 0) | (cols << 3) | (ho + 1 < a.H ? cols << 6 : 0);
        }
        v16i acc[2][TJ];
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[ti][tj][v] = 0;
        // Fragments of step (tap, 32 bytes) + 1 are read before the multiplies of the step at hand.
        const int8_t* const wrow = lds + lr * KW + 16 * lh;
        const int pitch = c.pc * 16, zeros = c.window * pitch;
        const int at0[2] = {row[0] * pitch, row[1] * pitch};
        int px[2], sw[2];
        v4i fp[2][2], fq[2][TJ];
        auto fragments = [&](int step) {
            const int tap = step / KT, k = step % KT;
            if (k == 0) {
#pragma unroll
                for (int ti = 0; ti < 2; ++ti) {
                    px[ti] = (mask[ti] >> tap) & 1 ? at0[ti] + ((tap / 3) * a.W + tap % 3) * pitch : zeros;
                    sw[ti] = ((px[ti] >> 8) & c.swz_mask) ^ lh;
                }
            }
#pragma unroll
            for (int ti = 0; ti < 2; ++ti) fp[step & 1][ti] = *(const v4i*)(win + px[ti] + (((2 * k) ^ sw[ti]) << 4));
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) fq[step & 1][tj] = *(const v4i*)(wrow + tj * 32 * KW + step * 32);
        };
        fragments(0);
#pragma unroll
        for (int step = 0; step < 9 * KT; ++step) {
            if (step + 1 < 9 * KT) fragments(step + 1);
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj)
                    acc[ti][tj] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fq[step & 1][tj], fp[step & 1][ti], acc[ti][tj], 0, 0, 0);
        }
        // The next window has landed (and the previous tile's stores have left: both count in issue order) before this tile's
        // stores go out; behind the barrier it is every wavefront's, and this one is free.
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");

        // sixteen rows at a time through the window that was just read
        const int r0 = i0 + 64 * wave;
        conv3_store<WHAT, TJ, S::EROWS>(a, z, r0, j0, acc, win + wave * S::ESLICE);
        if constexpr (WHAT == C3_STORE_GOODNESS) conv3_goodness<TJ>(a, z, r0, t + 1 < t1 ? r0 + C3_PIX : -1, acc, sq, vm);
        __builtin_amdgcn_s_barrier();   // (behind the fence of the last exchange; the staging slices lie in the window that the copy after next fills)
    }
}

template <int KT, int TJ>
static hipError_t launch_conv3_cfg(const GemmArgs& a, Conv3Geom c, hipStream_t s)
{
    using S = C3Shape<KT, TJ>;
    c.ncb = (a.J + S::BN - 1) / S::BN;
    const int per_xcd = num_cus() / 8 * 2;
    const int64_t tiles = ((int64_t)a.I + C3_PIX - 1) / C3_PIX * a.nb;
    // as many workgroups per column block as give each the same number of tiles
    const int64_t most = (int64_t)(per_xcd / c.ncb) * 8, rounds = (tiles + most - 1) / most;
    const int64_t slots = ((tiles + rounds - 1) / rounds + 7) / 8 * 8;
    c.per = (int)rounds;
    const dim3 grid((unsigned)(slots * c.ncb));
    if (a.residual) hipLaunchKernelGGL((k_conv3_i8<C3_RESIDUAL, KT, TJ>), grid, dim3(S::T), 0, s, GemmResidualArgs{a, *a.residual}, c);
    else if (a.gsum) hipLaunchKernelGGL((k_conv3_i8<C3_STORE_GOODNESS, KT, TJ>), grid, dim3(S::T), 0, s, a, c);
    else hipLaunchKernelGGL((k_conv3_i8<C3_STORE, KT, TJ>), grid, dim3(S::T), 0, s, a, c);
    return hipGetLastError();
}

// Whether a launch qualifies: 32-byte pieces per pixel, 32-column blocks of a wavefront, a window that fits the LDS.
struct Conv3Plan {
    int kt, tj;
    Conv3Geom c;
};
static bool conv3_plan(const GemmArgs& a, Conv3Plan* p)
{
    if (a.conv != 1 || a.ks != 3 || a.stride != 1 || a.pad != 1 || a.Cin > 64 || (a.J & 3) != 0 || a.J < 1 || a.J > 512 || a.splits != 1 || a.nb < 1 ||
        a.nb > 2 || a.p_bytes >= (int64_t(1) << 30) || a.H != a.Ho || a.W != a.Wo || (int64_t)a.I * a.cpitch != a.p_bytes || (a.cin_out & 3) != 0 ||
        a.cin_out > a.Cin || a.Cin > a.cpitch || a.rows_per_sample != a.H * a.W)
        return false;
    p->kt = (a.Cin + 31) / 32;
    p->tj = (a.J - 1) % 64 >= 32 ? 2 : 1;   // narrow blocks where a wide last one would be half empty
    Conv3Geom& c = p->c;
    c.cpp = a.Cin / 16;
    c.pc = c.cpp;
    c.swz_mask = (c.cpp & 1) ? 0 : c.cpp - 1;
    c.window = C3_PIX + 2 * a.W + 2;
    const int bn = 32 * p->tj, kw = 288 * p->kt + 16, buf = (80 * 1024 - bn * kw) / 2 / 1024 * 1024;
    // (a pixel of zeros behind the window, and the chunk more that an odd pixel's last piece reads)
    c.chunks = ((c.window + 1) * c.pc + 1 + 63) & ~63;
    return c.chunks <= C3_SLOTS * 256 && c.chunks * 16 <= buf && (a.J + bn - 1) / bn <= num_cus() / 4;
}

// From 64 tiles on, and for maps of at least half a tile (a wavefront's rows then belong to one or two samples).  The implicit
// loop against this, forward launches of two passes: 64 -> 64 channels, 8 images of 32x32 (64 tiles) 18.9 and 13.9 us, 64 images
// 24.5 and 20.4, 256 66 and 37; 64 -> 128, 256 images 100 and 65; 16 -> 64 51 and 31; 48 -> 96, 100 images of 28x28 36 and 26; 64
// -> 64, 256 images of 16x16 17.2 and 17.3.  Below the line: 64 -> 512, 16 images of 8x8 11.2 and 13.7; 64 -> 64, 200 of 7x7 8.8 and
// 13.0.  (Weights of 96 and 128 channels, 64 columns and two windows, fill the LDS of a
// compute unit: 128 -> 256 at 32x32 239 us in the implicit loop, 376 that way.  They are streamed instead, see conv3_wide.hip.)
bool conv3_ok(const GemmArgs& a)
{
    Conv3Plan p;
    if (a.rows_per_sample < C3_PIX / 2 || !conv3_plan(a, &p)) return false;
    return ((int64_t)a.I + C3_PIX - 1) / C3_PIX * a.nb * ((a.J + 32 * p.tj - 1) / (32 * p.tj)) >= 64;
}

hipError_t launch_conv3(const GemmArgs& a, hipStream_t s)
{
    Conv3Plan p;
    if (a.I <= 0 || a.J <= 0) return hipSuccess;
    if (!conv3_plan(a, &p) || (!a.C && !a.residual) || (a.gsum && (a.residual || !a.vmax))) return hipErrorInvalidValue;
    if (a.residual && (a.residual->M != a.I || a.residual->N != a.J || a.residual->rows_per_sample < RESIDUAL_MIN_ROWS)) return hipErrorInvalidValue;
    if (p.kt == 1) return p.tj == 2 ? launch_conv3_cfg<1, 2>(a, p.c, s) : launch_conv3_cfg<1, 1>(a, p.c, s);
    return p.tj == 2 ? launch_conv3_cfg<2, 2>(a, p.c, s) : launch_conv3_cfg<2, 1>(a, p.c, s);
}

}  // namespace ffi
