// int8 x int8 -> int32 contraction C[i][j] = sum_r P[i][r] * Q[j][r] of dense operands with few outputs: tiles of 32 x 32, each
// contracted by the four wavefronts of a workgroup, which share out its reduction.
//
// What bounds these launches is latency: in tiles of 64 x 128 a dense layer of 500 units on 200 samples has 16 workgroups, which walk
// through a reduction of 4704 in steps of 128 bytes, each step behind the round trip of its copies and two barriers.  Here the same
// layer has 112 workgroups, and a wavefront takes every fourth step by itself: two steps of loads in flight in registers, through
// 8 KB of LDS of its own into the layout the multiplies read, no barrier until the four partial sums meet at the end.
// Eight lanes load the 128 bytes of a row: lanes that read what they multiply themselves (a row each, no LDS) touch 32 lines with
// every load, and the four loads of a line do not meet in the L1 (13.3 us against 8.7 for the layer above).  Eight wavefronts gain
// nothing up to reductions of 2000 (8.3 us above, but 512 x 784 x 1000 7.8 instead of 7.3), nor does a third step in flight.
// Measured as single launches, samples x inputs x units, tiles of 64 x 128 against this: 200 x 4704 x 500 19.3 -> 8.7 us, 100 x 784 x 500
// 8.5 -> 5.8, 512 x 784 x 1000 8.6 -> 7.3, 512 x 4704 x 1000 25.2 -> 12.5, 64 x 50 x 500 6.4 -> 5.1 (an empty launch is about 4).
#include "ff_internal.hpp"
#include "device_math.hpp"
#include "codes.hpp"

namespace ffi {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int WAVES = 4, D = 2;   // wavefronts of a workgroup, steps of each in flight

template <bool EPI>
__global__ __launch_bounds__(WAVES * 64) void k_few_nt_i8(GemmArgs a, int ntiles, int per_xcd)
{
    constexpr int EROW = 36;   // words between rows of partial sums
    __shared__ __attribute__((aligned(16))) int8_t lds[WAVES * 8192];
    unsigned long long clk0 = 0, rt0 = 0, ph1 = 0, ph2 = 0;   // clock probe
    if (a.clk) {
        clk0 = clock64();
        rt0 = wall_clock64();
    }
    // Workgroups go to the eight XCDs in turn: each XCD gets consecutive tiles, which share their columns' rows of Q in its L2.
    const int t = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (t >= ntiles) return;
    const int tiles_i = (a.I + 31) / 32, tiles_z = tiles_i * ((a.J + 31) / 32);
    const int z = t / tiles_z, tz = t - z * tiles_z;
    const int bj = tz / tiles_i, bi = tz - bj * tiles_i;
    const int zp = EPI ? z : z / a.nc, zc = EPI ? 0 : z - zp * a.nc;
    const int i0 = bi * 32, j0 = bj * 32;
    const int8_t* const P = a.P + zp * a.st_p + zc * a.st_p2 + (int64_t)i0 * a.ldp;
    const int8_t* const Q = a.Q + zp * a.st_q + zc * a.st_q2 + (int64_t)j0 * a.ldq;
    int32_t* const C = a.C + zp * a.st_c + zc * a.st_c2;
    // rows beyond the matrix and bytes beyond the reduction read as zero (range check of the buffer)
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void*)P, 0, (int)(min(32, a.I - i0) * a.ldp), 0x00020000);
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)Q, 0, (int)(min(32, a.J - j0) * a.ldq), 0x00020000);
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5, r8 = lane >> 3, ch = lane & 7;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Rpad = (a.R + 15) & ~15;
    const int nk = (Rpad + 127) >> 7;
    const int n = nk > wave ? (nk - wave + WAVES - 1) / WAVES : 0;   // this wavefront's steps
    const int prow = r8 * (int)a.ldp, qrow = r8 * (int)a.ldq, p8 = 8 * (int)a.ldp, q8 = 8 * (int)a.ldq;
    int8_t* const mine = lds + wave * 8192;

    v4i p[D][4], q[D][4];
    // load c: rows 8 c .. 8 c + 7, eight lanes to a row's 128 bytes
    auto load = [&](int s, int u) {
        const int k = (wave + s * WAVES) * 128 + ch * 16;
        const bool in = k < Rpad;
#pragma unroll
        for (int c = 0; c < 4; ++c) p[u][c] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rp, in ? prow + c * p8 + k : 0x7FFFFFF0, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) q[u][c] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rq, in ? qrow + c * q8 + k : 0x7FFFFFF0, 0, 0);
    };
    v16i acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0;
#pragma unroll
    for (int u = 0; u < D; ++u) load(u, u);
    for (int s = 0; s < n; s += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (s + u >= n) break;   // (uniform)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int row = 8 * c + r8, at = row * 128 + ((ch ^ ((row >> 1) & 7)) << 4);
                *(v4i*)(mine + at) = p[u][c];
                *(v4i*)(mine + 4096 + at) = q[u][c];
            }
            load(s + u + D, u);
            wave_lds_fence();
            v4i fp[4], fq[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int at = lr * 128 + (((2 * m + lh) ^ ((lr >> 1) & 7)) << 4);
                fp[m] = *(const v4i*)(mine + at);
                fq[m] = *(const v4i*)(mine + 4096 + at);
            }
            wave_lds_fence();
            if (a.clk && ph1 == 0) ph1 = clock64();
#pragma unroll
            for (int m = 0; m < 4; ++m) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fq[m], fp[m], acc, 0, 0, 0);
        }
    }
    if (a.clk) ph2 = clock64();
    // lane: row lr of C, columns 8 g + 4 lh .. + 3
    int* const part = (int*)lds;
#pragma unroll
    for (int g = 0; g < 4; ++g)
        *(v4i*)(part + wave * 2048 + lr * EROW + 8 * g + 4 * lh) = (v4i){acc[4 * g + 0], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    __syncthreads();
    const int row = tid >> 3, cc = (tid & 7) * 4, i = i0 + row;
    v4i v = *(const v4i*)(part + row * EROW + cc);
#pragma unroll
    for (int w = 1; w < WAVES; ++w) v += *(const v4i*)(part + w * 2048 + row * EROW + cc);
    if (i < a.I && j0 + cc < a.J) *(v4i*)(C + (int64_t)i * a.ldc + j0 + cc) = v;
    if (EPI) {
        // eight consecutive lanes hold a row, which is one sample; columns beyond the matrix are zeros
        const int y[4] = {v[0], v[1], v[2], v[3]};
        unsigned long long sq = 0;
        int vm = 0;
        goodness_terms(a.relu, a.rshift, y, 4, sq, vm);
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
            sq += xor_lane_u64(sq, d);
            vm = max(vm, __shfl_xor(vm, d));
        }
        if ((tid & 7) == 0 && i < a.I) {
            atomicAdd(a.gsum + z * a.st_g + i, sq);
            atomicMax(a.vmax + z * a.st_g + i, vm);
        }
    }
    if (a.clk && tid == 0) {
        const unsigned long long end = clock64();
        atomicAdd(a.clk + 0, end - clk0);
        atomicAdd(a.clk + 1, (unsigned long long)wall_clock64() - rt0);
        unsigned long long* pc = a.clk + (EPI ? 8 : 2);
        atomicAdd(pc + 0, ph1 - clk0);
        atomicAdd(pc + 1, ph2 - ph1);
        atomicAdd(pc + 2, end - ph2);
        atomicAdd(pc + 4, 1ull);
    }
}

// Up to two workgroups per compute unit: 512 tiles of 32 x 32 are 48 to 64 of 64 x 128.  Beyond, the larger tiles' fewer bytes per
// multiply count: 768 x 400 x 1024 (768 tiles) 7.65 us there and 7.83 here, 896 x 784 x 1024 8.6 and 9.1, 1000 x 784 x 1201 9.0 and 10.5.
// Goodness sums: a row's tiles add to one word each, so more than 32 of them need a reduction long enough to pay for that:
// 64 x 1200 x 4000 10.05 us there and 10.36 here, with 2000 inputs 12.1 and 10.8; 250 x 16 x 2000 6.7 and 7.3, 784 inputs 8.8 and 8.4.
// Sums of samples of several rows stay with the kernel that adds them up across rows first.
bool gemm_few_ok(const GemmArgs& a)
{
    if (a.conv || a.splits != 1 || a.upd_w || a.residual) return false;
    if (a.gsum && (a.rows_per_sample != 1 || a.J > max(1024, 2 * a.R))) return false;
    return (int64_t)((a.I + 31) / 32) * ((a.J + 31) / 32) * a.nb <= 2 * num_cus();
}

hipError_t launch_gemm_few(const GemmArgs& a, hipStream_t s)
{
    const int ntiles = ((a.I + 31) / 32) * ((a.J + 31) / 32) * a.nb, per_xcd = (ntiles + 7) / 8;
    const dim3 grid((unsigned)(8 * per_xcd)), block(WAVES * 64);
    if (a.gsum) hipLaunchKernelGGL(k_few_nt_i8<true>, grid, block, 0, s, a, ntiles, per_xcd);
    else hipLaunchKernelGGL(k_few_nt_i8<false>, grid, block, 0, s, a, ntiles, per_xcd);
    return hipGetLastError();
}

}  // namespace ffi
