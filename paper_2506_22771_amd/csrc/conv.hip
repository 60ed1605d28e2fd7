// Patch matrices and depthwise convolutions of the FF-INT8 step (gfx950).
//
// A convolution's forward pass runs as an implicit GEMM inside k_gemm_nt_i8 whenever C_in is a multiple of 4 greater than
// 4, and its weight gradient (Section IV-B: only g^W is formed) reads the NHWC input reduction-major there.  Another channel
// count -- above all that of a first layer with one or three channels, whose reduction rows of 9 or 27 bytes no 16-byte
// copy can address -- has its patches written row-major, col[m][(kh,kw,ci)], for the forward contraction; up to four channels
// the weight gradient reads them as well.  Pure data movement; taps outside the image give 0.
#include "codes.hpp"

namespace ffi {

__device__ __forceinline__ int gather_byte(const int8_t* __restrict__ a, const ConvGeom& g, int b, int ho, int wo,
                                           int kh, int kw, int ci)
{
    const int hi = ho * g.stride - g.pad + kh, wi = wo * g.stride - g.pad + kw;
    if ((unsigned)hi >= (unsigned)g.H || (unsigned)wi >= (unsigned)g.W) return 0;
    return (int)(uint8_t)a[(((int64_t)b * g.H + hi) * g.W + wi) * g.cpitch + ci];
}

// col[m][j] for every output pixel m of all samples, j < K, row pitch ld_out; one thread per 16-byte chunk.
__global__ __launch_bounds__(256) void k_im2col(Im2colArgs p)
{
    const int z = blockIdx.z;
    const int8_t* __restrict__ a = p.a + z * p.st_a;
    int8_t* __restrict__ out = p.out + z * p.st_out;
    const ConvGeom& g = p.g;
    const int64_t chunks_per_row = p.ld_out >> 4;
    const int hw = g.Ho * g.Wo;
    const int64_t M = (int64_t)p.B * hw;
    const int64_t total = M * chunks_per_row;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int64_t m = e / chunks_per_row;
        const int j0 = (int)(e - m * chunks_per_row) << 4;
        const int b = (int)(m / hw);
        const int rem = (int)(m - (int64_t)b * hw);
        const int ho = rem / g.Wo, wo = rem - ho * g.Wo;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int j = j0 + t;
            if (j < p.K) {
                const int tap = j / g.Cin, ci = j - tap * g.Cin;
                const int kh = tap / g.ks, kw = tap - kh * g.ks;
                w[t >> 2] |= (uint32_t)gather_byte(a, g, b, ho, wo, kh, kw, ci) << (8 * (t & 3));
            }
        }
        *(uint4*)(out + m * p.ld_out + j0) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// The same for 3x3 kernels over one to four channels (a first layer): one thread per output pixel.  A tap is one 4-byte
// load (the pad channels of a pixel are zero), the nine taps are packed in registers and leave as whole 16-byte pieces.
// Bound by the patch rows written: 3 channels, 32x32 maps, 512 images (16.8 MB out) 10.6 us against 35.8 us byte by byte.
template <int CIN>
__global__ __launch_bounds__(256) void k_im2col_small(Im2colArgs p)
{
    constexpr int PIECES = (9 * CIN + 15) / 16;
    const ConvGeom& g = p.g;
    const int z = blockIdx.z;
    const int8_t* __restrict__ a = p.a + z * p.st_a;
    const int hw = g.Ho * g.Wo;
    const int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (m >= (int64_t)p.B * hw) return;
    const int b = (int)(m / hw);
    const int rem = (int)(m - (int64_t)b * hw);
    const int ho = rem / g.Wo, wo = rem - ho * g.Wo;
    const int hi0 = ho * g.stride - g.pad, wi0 = wo * g.stride - g.pad;
    const int8_t* __restrict__ ab = a + (int64_t)b * g.H * g.W * g.cpitch;
    uint32_t w[4 * PIECES + 1];
#pragma unroll
    for (int i = 0; i <= 4 * PIECES; ++i) w[i] = 0u;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int hi = hi0 + t / 3, wi = wi0 + t % 3;
        uint32_t x = 0u;
        if ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W)
            x = *(const uint32_t*)(ab + ((int64_t)hi * g.W + wi) * g.cpitch);
        const int at = t * CIN, sh = 8 * (at & 3);
        w[at >> 2] |= x << sh;
        if ((at & 3) + CIN > 4) w[(at >> 2) + 1] |= x >> (32 - sh);
    }
    uint4* o = (uint4*)(p.out + z * p.st_out + m * p.ld_out);
#pragma unroll
    for (int i = 0; i < PIECES; ++i) o[i] = make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
}

hipError_t launch_im2col(const Im2colArgs& p, hipStream_t s)
{
    const ConvGeom& g = p.g;
    const int64_t M = (int64_t)p.B * g.Ho * g.Wo;
    const int64_t total = M * (p.ld_out >> 4);
    if (total <= 0) return hipSuccess;
    if (g.ks == 3 && g.Cin <= 4) {
        const dim3 grid((unsigned)((M + 255) / 256), 1, (unsigned)p.nb);
        if (g.Cin == 1) hipLaunchKernelGGL(k_im2col_small<1>, grid, dim3(256), 0, s, p);
        else if (g.Cin == 2) hipLaunchKernelGGL(k_im2col_small<2>, grid, dim3(256), 0, s, p);
        else if (g.Cin == 3) hipLaunchKernelGGL(k_im2col_small<3>, grid, dim3(256), 0, s, p);
        else hipLaunchKernelGGL(k_im2col_small<4>, grid, dim3(256), 0, s, p);
        return hipGetLastError();
    }
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65535) blocks = 65535;
    const dim3 grid((unsigned)blocks, 1, (unsigned)p.nb);
    hipLaunchKernelGGL(k_im2col, grid, dim3(256), 0, s, p);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Depthwise convolution.  Forward: a thread owns four channels of one output pixel (nine 4-byte taps, 16-byte
// store of the accumulators); blockIdx.y = sample, so the per-sample goodness sums / maxima are reduced in the
// workgroup and leave as one atomic each.  HBM-bound on the int32 output (4 bytes written per input byte).
// ------------------------------------------------------------------------------------------------------------
constexpr int DW_PIX = 8;   // output pixels per thread

__device__ __forceinline__ unsigned long long dw_wave_sum_u64(unsigned long long v)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)v, d), hi = (unsigned)__shfl_xor((int)(unsigned)(v >> 32), d);
        v += ((unsigned long long)hi << 32) | lo;
    }
    return v;
}

// 4x4 byte transpose: word j of x holds bytes (channels) 0..3 of item j; word e of o holds byte e of items 0..3.
__device__ __forceinline__ void dw_transpose4x4(const uint32_t x[4], uint32_t o[4])
{
    const uint32_t t0 = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u);
    const uint32_t t1 = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u);
    const uint32_t t2 = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u);
    const uint32_t t3 = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
    o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

// blockIdx.x = share of the sample's output pixels, blockIdx.y = sample, blockIdx.z = pass * channel groups + group.
// A thread keeps the 36 weights of its four channels in registers and walks over DW_PIX pixels, 256 / quads apart.
__global__ __launch_bounds__(256) void k_dwconv_forward(DwArgs p, int cgroups)
{
    const ConvGeom& g = p.g;
    const int z = blockIdx.z / cgroups, cg0 = (blockIdx.z - z * cgroups) * 64;
    const int b = blockIdx.y;
    const int C = g.Cin;
    const int nq = min(16, (C - cg0 + 3) >> 2);          // channel quads of this workgroup
    const int lanes = 256 / nq;                          // pixel lanes
    const int q = threadIdx.x % nq, pl = threadIdx.x / nq;
    const int c0 = cg0 + 4 * q;
    const int hw = g.Ho * g.Wo;
    const int8_t* __restrict__ a = p.a + z * p.st_a;
    unsigned long long sq = 0;
    int vm = 0;
    if (pl < lanes) {
        // the nine taps of a channel are nine consecutive bytes of its weight row: three packed words per channel
        uint32_t w[4][3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint4 wr = make_uint4(0u, 0u, 0u, 0u);
            if (c0 + e < C) wr = *(const uint4*)(p.w_q + (int64_t)(c0 + e) * 16);
            w[e][0] = wr.x; w[e][1] = wr.y; w[e][2] = wr.z;
        }
        if (g.stride == 1 && (g.Wo & 3) == 0) {
            // Stride 1, rows of whole 4-pixel groups: four consecutive output pixels at a time.  The six input columns
            // they touch are loaded once per kernel row and transposed to (channel word x pixel bytes); the word of
            // output j is a byte alignment of two such words, and a kernel row is one packed dot product with the
            // three taps of that row (fourth byte zero): half the loads and address arithmetic of the loop below.
            uint32_t wk[4][3];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                wk[e][0] = w[e][0] & 0x00FFFFFFu;
                wk[e][1] = __builtin_amdgcn_alignbyte(w[e][1], w[e][0], 3u) & 0x00FFFFFFu;
                wk[e][2] = __builtin_amdgcn_alignbyte(w[e][2], w[e][1], 2u) & 0x00FFFFFFu;
            }
            const int ngrp = hw >> 2;
            const int grp0 = (int)blockIdx.x * lanes * (DW_PIX / 4) + pl;
            for (int it = 0; it < DW_PIX / 4; ++it) {
                const int grp = grp0 + it * lanes;
                if (grp >= ngrp) break;
                const int pix = 4 * grp;
                const int ho = pix / g.Wo, wo = pix - ho * g.Wo;
                int acc[4][4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[j][e] = 0;
#pragma unroll
                for (int kh = 0; kh < 3; ++kh) {
                    const int hi = ho + kh - g.pad;
                    if ((unsigned)hi >= (unsigned)g.H) continue;
                    const int8_t* arow = a + (((int64_t)b * g.H + hi) * g.W) * g.cpitch + c0;
                    uint32_t X[8];
#pragma unroll
                    for (int j = 0; j < 6; ++j) {
                        const int wi = wo - g.pad + j;
                        X[j] = (unsigned)wi < (unsigned)g.W ? *(const uint32_t*)(arow + (int64_t)wi * g.cpitch) : 0u;
                    }
                    X[6] = 0u;
                    X[7] = 0u;
                    uint32_t TA[4], TB[4];
                    dw_transpose4x4(X, TA);
                    dw_transpose4x4(X + 4, TB);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc[0][e] = __builtin_amdgcn_sdot4((int)TA[e], (int)wk[e][kh], acc[0][e], false);
                        acc[1][e] = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_alignbyte(TB[e], TA[e], 1u), (int)wk[e][kh], acc[1][e], false);
                        acc[2][e] = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_alignbyte(TB[e], TA[e], 2u), (int)wk[e][kh], acc[2][e], false);
                        acc[3][e] = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_alignbyte(TB[e], TA[e], 3u), (int)wk[e][kh], acc[3][e], false);
                    }
                }
                typedef int i32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    __builtin_nontemporal_store((i32x4){acc[j][0], acc[j][1], acc[j][2], acc[j][3]},
                                                (i32x4*)(p.acc + z * p.st_acc + ((int64_t)b * hw + pix + j) * p.ldacc + c0));
                    if (p.gsum && p.relu && p.rshift == 0) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const unsigned y = (unsigned)max(acc[j][e], 0);
                            sq += (unsigned long long)y * y;
                            vm = max(vm, (int)y);
                        }
                    } else if (p.gsum) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            int y = acc[j][e];
                            if (p.relu) y = max(y, 0);
                            const long long yl = (long long)y;
                            sq += ((unsigned long long)(yl * yl)) >> p.rshift;
                            vm = max(vm, y < 0 ? -y : y);
                        }
                    }
                }
            }
        } else {
        const int pix0 = (int)blockIdx.x * lanes * DW_PIX + pl;
#pragma unroll 2
        for (int it = 0; it < DW_PIX; ++it) {
            const int pix = pix0 + it * lanes;
            if (pix >= hw) break;
            const int ho = pix / g.Wo, wo = pix - ho * g.Wo;
            uint32_t x[9];   // tap words: byte e = channel c0 + e
#pragma unroll
            for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                for (int kw = 0; kw < 3; ++kw) {
                    const int hi = ho * g.stride + kh - g.pad, wi = wo * g.stride + kw - g.pad;
                    x[kh * 3 + kw] = ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W)
                                         ? *(const uint32_t*)(a + (((int64_t)b * g.H + hi) * g.W + wi) * g.cpitch + c0)
                                         : 0u;
                }
            // two 4x4 byte transposes turn (tap words x channel bytes) into (channel words x tap bytes), which is
            // the operand order of the packed int8 dot product
            int acc[4];
            {
                uint32_t lo[4], hi4[4];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t* xs = x + 4 * h;
                    const uint32_t t0 = __builtin_amdgcn_perm(xs[1], xs[0], 0x05010400u);
                    const uint32_t t1 = __builtin_amdgcn_perm(xs[1], xs[0], 0x07030602u);
                    const uint32_t t2 = __builtin_amdgcn_perm(xs[3], xs[2], 0x05010400u);
                    const uint32_t t3 = __builtin_amdgcn_perm(xs[3], xs[2], 0x07030602u);
                    uint32_t* o = h ? hi4 : lo;
                    o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
                    o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
                    o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
                    o[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    int sacc = (int)(int8_t)(x[8] >> (8 * e)) * (int)(int8_t)(w[e][2] & 0xFFu);
                    sacc = __builtin_amdgcn_sdot4((int)lo[e], (int)w[e][0], sacc, false);
                    sacc = __builtin_amdgcn_sdot4((int)hi4[e], (int)w[e][1], sacc, false);
                    acc[e] = sacc;
                }
            }
            {   // like the contraction's forward output: not read again soon, non-temporal store
                typedef int i32x4 __attribute__((ext_vector_type(4)));
                __builtin_nontemporal_store((i32x4){acc[0], acc[1], acc[2], acc[3]},
                                            (i32x4*)(p.acc + z * p.st_acc + ((int64_t)b * hw + pix) * p.ldacc + c0));
            }
            if (p.gsum) {
                // channels beyond C read zero inputs and zero weights: their y is 0
                if (p.relu && p.rshift == 0) {        // the usual case: one 32x32+64-bit multiply-add per activity
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const unsigned y = (unsigned)max(acc[e], 0);
                        sq += (unsigned long long)y * y;
                        vm = max(vm, (int)y);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        int y = acc[e];
                        if (p.relu) y = max(y, 0);
                        const long long yl = (long long)y;
                        sq += ((unsigned long long)(yl * yl)) >> p.rshift;
                        vm = max(vm, y < 0 ? -y : y);
                    }
                }
            }
        }
        }
    }
    if (p.gsum) {
        __shared__ unsigned long long rs[4];
        __shared__ int rm[4];
        sq = dw_wave_sum_u64(sq);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) vm = max(vm, __shfl_xor(vm, d));
        if ((threadIdx.x & 63) == 0) { rs[threadIdx.x >> 6] = sq; rm[threadIdx.x >> 6] = vm; }
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long t = rs[0] + rs[1] + rs[2] + rs[3];
            const int m = max(max(rm[0], rm[1]), max(rm[2], rm[3]));
            if (t) atomicAdd(p.gsum + z * p.st_g + b, t);
            if (m) atomicMax(p.vmax + z * p.st_g + b, m);
        }
    }
}

hipError_t launch_dwconv_forward(const DwArgs& p, hipStream_t s)
{
    const ConvGeom& g = p.g;
    if (p.B <= 0) return hipSuccess;
    const int cgroups = (g.Cin + 63) / 64;
    if (g.ks != 3 || p.B > 65535 || (int64_t)cgroups * p.nb > 65535) return hipErrorInvalidValue;
    // pixels per workgroup depend on the group's quad count; size the grid for full groups (16 quads, 16 lanes),
    // narrower groups have more lanes and finish their share early
    const int64_t hw = (int64_t)g.Ho * g.Wo;
    const unsigned bx = (unsigned)((hw + 16 * DW_PIX - 1) / (16 * DW_PIX));
    hipLaunchKernelGGL(k_dwconv_forward, dim3(bx, (unsigned)p.B, (unsigned)(cgroups * p.nb)), dim3(256), 0, s, p, cgroups);
    return hipGetLastError();
}

// Depthwise layers whose accumulators are not stored: nine taps are worked out again by each pass that needs them (goodness sums,
// codes handed on, codes of the local gradient, all row-major), where the stored form writes four bytes per output and reads them
// twice.  Threads are numbered through (piece, channel quad), so that every lane has channels whatever their number; blockIdx.y =
// sample, blockIdx.z = pass.  A piece is a strip of four columns x DW_STRIP rows: the input rows slide through a window of three,
// each loaded and transposed once.  Bound by integer and quantiser arithmetic.  144 channels, two passes of 256 images of 32x32:
// forward with stores, hand-off and local gradient 122 + 81 + 103 us, goodness, hand-off and local gradient here 32 + 64 + 70 (beside
// other chains up to 119).
constexpr int DW_STRIP = 8;

// input row hi of columns wi0 .. wi0 + 5, four channels: word [e][j] = bytes of channel e from column j on
__device__ __forceinline__ void dw_row_words(const ConvGeom& g, const int8_t* __restrict__ ab, int hi, int wi0, int c0, uint32_t row[4][4])
{
    uint32_t X[8];
    const bool in = (unsigned)hi < (unsigned)g.H;
    const int8_t* arow = ab + (int64_t)hi * g.W * g.cpitch + c0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const int wi = wi0 + j;
        X[j] = in && (unsigned)wi < (unsigned)g.W ? *(const uint32_t*)(arow + wi * g.cpitch) : 0u;
    }
    X[6] = 0u;
    X[7] = 0u;
    uint32_t TA[4], TB[4];
    dw_transpose4x4(X, TA);
    dw_transpose4x4(X + 4, TB);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        row[e][0] = TA[e];
        row[e][1] = __builtin_amdgcn_alignbyte(TB[e], TA[e], 1u);
        row[e][2] = __builtin_amdgcn_alignbyte(TB[e], TA[e], 2u);
        row[e][3] = __builtin_amdgcn_alignbyte(TB[e], TA[e], 3u);
    }
}

template <int WHAT>
__global__ __launch_bounds__(256) void k_dwconv_rework(DwArgs p, QuantArgs qa, int nq)
{
    constexpr bool GRAD = WHAT == ROWS_GRAD;
    const ConvGeom& g = p.g;
    const int z = blockIdx.z, b = blockIdx.y;
    CodeScale cs = {};
    float rowf = 0.0f;
    if (WHAT != ROWS_GOODNESS) {
        cs = code_scale<256>(qa, z);
        if (blockIdx.x == 0 && b == 0 && threadIdx.x == 0) qa.scale[z * qa.st_scale] = cs.live ? cs.amax / 127.0f : 1.0f;
        if (GRAD) rowf = 2.0f * qa.per_sample[z * qa.st_per_sample + b];
    }
    const int hw = g.Ho * g.Wo, wgroups = g.Wo >> 2;
    const int pieces = wgroups * ((g.Ho + DW_STRIP - 1) / DW_STRIP);
    const int at = (int)blockIdx.x * 256 + (int)threadIdx.x, piece = at / nq, c0 = 4 * (at - piece * nq);
    const int8_t* __restrict__ ab = p.a + z * p.st_a + (int64_t)b * g.H * g.W * g.cpitch;
    unsigned long long sq = 0;
    int vm = 0;
    auto run = [&](auto form) {
        constexpr int FORM = decltype(form)::value;
        // four channels of output pixel `pix`
        auto result = [&](int pix, const int acc[4]) {
            if constexpr (WHAT == ROWS_GOODNESS) {
                goodness_terms(p.relu, p.rshift, acc, 4, sq, vm);
            } else {
                const uint32_t m = (uint32_t)(b * hw + pix);
                *(uint32_t*)(qa.q + z * qa.st_q + (int64_t)m * qa.ldq + c0) =
                    quad_codes<GRAD, FORM>(cs, acc[0], acc[1], acc[2], acc[3], m * (uint32_t)g.Cin + (uint32_t)c0, rowf);
            }
        };
        // the nine taps of a channel are nine consecutive bytes of its weight row
        uint32_t w[4][3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint4 wr = make_uint4(0u, 0u, 0u, 0u);
            if (c0 + e < g.Cin) wr = *(const uint4*)(p.w_q + (int64_t)(c0 + e) * 16);
            w[e][0] = wr.x; w[e][1] = wr.y; w[e][2] = wr.z;
        }
        uint32_t wk[4][3];   // three taps of a kernel row, fourth byte zero
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            wk[e][0] = w[e][0] & 0x00FFFFFFu;
            wk[e][1] = __builtin_amdgcn_alignbyte(w[e][1], w[e][0], 3u) & 0x00FFFFFFu;
            wk[e][2] = __builtin_amdgcn_alignbyte(w[e][2], w[e][1], 2u) & 0x00FFFFFFu;
        }
        const int hb = piece / wgroups, wo = 4 * (piece - hb * wgroups), h0 = hb * DW_STRIP;
        uint32_t win[3][4][4];
        dw_row_words(g, ab, h0 - 1, wo - 1, c0, win[0]);
        dw_row_words(g, ab, h0, wo - 1, c0, win[1]);
#pragma unroll
        for (int r = 0; r < DW_STRIP; ++r) {
            if (h0 + r >= g.Ho) break;
            dw_row_words(g, ab, h0 + r + 1, wo - 1, c0, win[(r + 2) % 3]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int acc[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[e] = 0;
#pragma unroll
                    for (int kh = 0; kh < 3; ++kh) acc[e] = __builtin_amdgcn_sdot4((int)win[(r + kh) % 3][e][j], (int)wk[e][kh], acc[e], false);
                }
                result((h0 + r) * g.Wo + wo + j, acc);
            }
        }
    };
    if (piece < pieces) {   // (the forms are uniform)
        if (WHAT == ROWS_GOODNESS) run(std::integral_constant<int, CODE_FLOAT>{});
        else if (!cs.fixed) run(std::integral_constant<int, CODE_FLOAT>{});
        else if (GRAD && rowf < 0.0f) run(std::integral_constant<int, GRAD ? CODE_DOWN : CODE_UP>{});
        else run(std::integral_constant<int, CODE_UP>{});
    }
    if constexpr (WHAT == ROWS_GOODNESS) {
        __shared__ unsigned long long rs[4];
        __shared__ int rm[4];
        sq = dw_wave_sum_u64(sq);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) vm = max(vm, __shfl_xor(vm, d));
        if ((threadIdx.x & 63) == 0) { rs[threadIdx.x >> 6] = sq; rm[threadIdx.x >> 6] = vm; }
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long t = rs[0] + rs[1] + rs[2] + rs[3];
            const int m = max(max(rm[0], rm[1]), max(rm[2], rm[3]));
            if (t) atomicAdd(p.gsum + z * p.st_g + b, t);
            if (m) atomicMax(p.vmax + z * p.st_g + b, m);
        }
    }
}

// threads per sample of a launch over nq channel quads
static int64_t dwconv_rework_threads(const ConvGeom& g, int64_t nq) { return (int64_t)(g.Wo >> 2) * ((g.Ho + DW_STRIP - 1) / DW_STRIP) * nq; }

template <int WHAT>
static hipError_t launch_dwconv_rework_t(const DwArgs& p, const QuantArgs& q, hipStream_t s)
{
    // (codes: quads up to the row pitch, whose pad bytes become zeros)
    const int nq = (int)((WHAT == ROWS_GOODNESS ? p.g.Cin : q.ldq) + 3) >> 2;
    const int64_t blocks = (dwconv_rework_threads(p.g, nq) + 255) / 256;
    if (blocks > (int64_t(1) << 22)) return hipErrorInvalidValue;   // (thread numbers in 32 bits)
    hipLaunchKernelGGL(k_dwconv_rework<WHAT>, dim3((unsigned)blocks, (unsigned)p.B, (unsigned)p.nb), dim3(256), 0, s, p, q, nq);
    return hipGetLastError();
}

// Stride one and rows of whole 4-pixel groups (strips), from 2^23 outputs a pass on, where the stored accumulators no longer stay
// in the caches, and not where the last workgroup of a sample leaves more than a quarter of its threads idle.  Steps of 1x1, depthwise
// and 1x1 layers, stored and reworked: 144 channels, 32x32, 64 images (9.4 M outputs) 212 and 201 us, 256 images 601 and 471; 64
// channels, 128 images (8.4 M) 171.9 and 171.4; 240 channels, 16x16, 256 images (15.7 M) 244 and 219.  Above the line and slower: 64
// channels, 28x28, 256 images (12.8 M) 213 and 218, 192, 16x16, 256 (12.6 M) 201 and 204.  Below it: 64 channels, 28x28, 128 images (6.4 M) 161
// and 170, 64, 16x16, 256 (4.2 M) 127 and 143, 240, 16x16, 128 (7.9 M) 171 and 171.  Idle threads: 144 channels, 16x16, 256 images (9.4 M,
// 288 threads a sample) 187 and 196.  Pixels one by one, each with its nine loads, are slower reworked: stride two, 192 channels, 32x32, 256 images 401
// and 419, 384 785 and 813; widths of 14, 192 channels, 256 images 252 and 270, of 30 863 and 940.
bool dwconv_rework_pays(const ConvGeom& g, int64_t B)
{
    if (g.stride != 1 || (g.Wo & 3) != 0 || B * g.Ho * g.Wo * g.Cin < (int64_t(1) << 23)) return false;
    const int64_t threads = dwconv_rework_threads(g, (g.Cin + 3) >> 2);
    return 4 * threads >= 3 * ((threads + 255) / 256 * 256);
}

hipError_t launch_dwconv_rework(int what, const DwArgs& p, const QuantArgs& q, hipStream_t s)
{
    const ConvGeom& g = p.g;
    if (p.B <= 0) return hipSuccess;
    if (g.ks != 3 || g.stride != 1 || (g.Wo & 3) != 0 || p.B > 65535 || (g.Cin & 3) != 0 || p.nb < 1 || p.nb > 2) return hipErrorInvalidValue;
    if (what == ROWS_GOODNESS) return p.gsum && p.vmax ? launch_dwconv_rework_t<ROWS_GOODNESS>(p, q, s) : hipErrorInvalidValue;
    if (q.round_mode != FF_ROUND_STOCHASTIC || q.l2norm || !q.q || q.q_t || q.ldq != g.cpitch || q.cols != g.Cin || q.rows != (int64_t)p.B * g.Ho * g.Wo)
        return hipErrorInvalidValue;
    if (what == ROWS_HANDOFF) return launch_dwconv_rework_t<ROWS_HANDOFF>(p, q, s);
    return what == ROWS_GRAD && q.per_sample ? launch_dwconv_rework_t<ROWS_GRAD>(p, q, s) : hipErrorInvalidValue;
}

// Weight gradient of a depthwise convolution: dw[c][tap] = sum over output pixels of gy[m][c] * a[pixel(m) + tap][c].
// A workgroup owns a share of the output pixels of one sample chunk and a group of up to 64 channels; a thread owns four
// channels and every (256 / quads)-th piece of the share, keeps 36 int32 partial sums and adds them to LDS accumulators with
// LDS atomics.  The workgroup stores its sums as one of `splits` partial results, which the update adds up; callers
// without scratch have them added to dw with integer atomics instead (exact and order-free; dw must be zero on entry).
// Stride 1, rows of whole 4-pixel groups: a piece is a strip of four columns x DW_STRIP rows.  The input rows slide through
// a window of three: each is loaded, byte-transposed to (channel word x pixel bytes) and shifted once and serves three
// output rows, a (channel, tap) of a group is one packed dot product over its four pixels.  Integer issue and 4-byte loads
// bound it (10 loads and 68 operations a group, 22 and 116 when every group fetched its three rows).  Together with the
// partial results in place of 900 thousand atomics: step of the MobileNet-shaped stack 2489 -> 2474 us.
__device__ __forceinline__ void dw_load_row(const DwArgs& p, const int8_t* __restrict__ ab, int hi, int wi0, int c0, uint32_t row[4][3])
{
    const ConvGeom& g = p.g;
    uint32_t X[8];
    const bool in = (unsigned)hi < (unsigned)g.H;
    const int8_t* arow = ab + (int64_t)hi * g.W * g.cpitch + c0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const int wi = wi0 + j;
        X[j] = in && (unsigned)wi < (unsigned)g.W ? *(const uint32_t*)(arow + wi * g.cpitch) : 0u;
    }
    X[6] = 0u;
    X[7] = 0u;
    uint32_t TA[4], TB[4];
    dw_transpose4x4(X, TA);
    dw_transpose4x4(X + 4, TB);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        row[e][0] = TA[e];
        row[e][1] = __builtin_amdgcn_alignbyte(TB[e], TA[e], 1u);
        row[e][2] = __builtin_amdgcn_alignbyte(TB[e], TA[e], 2u);
    }
}

// pieces of one chunk: strips, or single output pixels
__host__ __device__ static inline bool dw_strips(const ConvGeom& g) { return g.stride == 1 && (g.Wo & 3) == 0; }
__host__ __device__ static inline int dw_pieces_per_sample(const ConvGeom& g)
{
    return dw_strips(g) ? (g.Wo >> 2) * ((g.Ho + DW_STRIP - 1) / DW_STRIP) : g.Ho * g.Wo;
}

__global__ __launch_bounds__(256) void k_dwconv_wgrad(DwArgs p)
{
    const ConvGeom& g = p.g;
    const int z = blockIdx.z / p.nc, chunk = blockIdx.z - z * p.nc;
    const int C = g.Cin;
    const int cg0 = blockIdx.y * 64;
    const int nq = min(16, (C - cg0 + 3) >> 2);          // channel quads of this workgroup
    const int lanes = 256 / nq;                          // piece lanes
    const int q = threadIdx.x % nq, rl = threadIdx.x / nq;
    const int c0 = cg0 + 4 * q;
    const int hw = g.Ho * g.Wo;
    const int b0 = chunk * p.chunk_b, b1 = min(p.B, b0 + p.chunk_b);
    const int8_t* __restrict__ a = p.a + z * p.st_a;
    const int8_t* __restrict__ gy = p.gy + z * p.st_gy;
    __shared__ int lacc[64 * 9];
    for (int e = threadIdx.x; e < 64 * 9; e += 256) lacc[e] = 0;
    __syncthreads();
    int part[4][9];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < 9; ++t) part[e][t] = 0;
    const int pps = dw_pieces_per_sample(g);
    const int total = (b1 - b0) * pps;
    const int per = (total + (int)gridDim.x - 1) / (int)gridDim.x;
    const int s0 = (int)blockIdx.x * per, s1 = min(total, s0 + per);
    if (rl < lanes && dw_strips(g)) {
        const int wgroups = g.Wo >> 2;
        for (int s = s0 + rl; s < s1; s += lanes) {
            const int bl = s / pps, r = s - bl * pps;
            const int hb = r / wgroups, wo = 4 * (r - hb * wgroups);
            const int h0 = hb * DW_STRIP;
            const int8_t* ab = a + (int64_t)(b0 + bl) * g.H * g.W * g.cpitch;
            const int8_t* gp = gy + ((int64_t)(b0 + bl) * hw + h0 * g.Wo + wo) * p.ldg + c0;
            uint32_t win[3][4][3];
            dw_load_row(p, ab, h0 - 1, wo - 1, c0, win[0]);
            dw_load_row(p, ab, h0, wo - 1, c0, win[1]);
#pragma unroll
            for (int j = 0; j < DW_STRIP; ++j) {
                if (h0 + j >= g.Ho) break;
                uint32_t gq[4], G[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) gq[i] = *(const uint32_t*)(gp + (j * g.Wo + i) * p.ldg);
                dw_load_row(p, ab, h0 + j + 1, wo - 1, c0, win[(j + 2) % 3]);
                dw_transpose4x4(gq, G);
#pragma unroll
                for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int kw = 0; kw < 3; ++kw)
                            part[e][kh * 3 + kw] = __builtin_amdgcn_sdot4((int)G[e], (int)win[(j + kh) % 3][e][kw],
                                                                          part[e][kh * 3 + kw], false);
            }
        }
    } else if (rl < lanes) {
        for (int s = s0 + rl; s < s1; s += lanes) {
            const int bl = s / hw, pix = s - bl * hw;
            const int64_t m = (int64_t)(b0 + bl) * hw + pix;
            const int ho = pix / g.Wo, wo = pix - ho * g.Wo;
            const uint32_t gw = *(const uint32_t*)(gy + m * p.ldg + c0);
            if (gw == 0u) continue;   // a rectified gradient is zero wherever the activity is
            int gv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) gv[e] = (int)(int8_t)(gw >> (8 * e));
#pragma unroll
            for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                for (int kw = 0; kw < 3; ++kw) {
                    const int hi = ho * g.stride + kh - g.pad, wi = wo * g.stride + kw - g.pad;
                    if ((unsigned)hi < (unsigned)g.H && (unsigned)wi < (unsigned)g.W) {
                        const uint32_t x = *(const uint32_t*)(a + (((int64_t)(b0 + bl) * g.H + hi) * g.W + wi) * g.cpitch + c0);
#pragma unroll
                        for (int e = 0; e < 4; ++e) part[e][kh * 3 + kw] += gv[e] * (int)(int8_t)(x >> (8 * e));
                    }
                }
        }
    }
    if (rl < lanes) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < 9; ++t)
                if (part[e][t]) atomicAdd(&lacc[(4 * q + e) * 9 + t], part[e][t]);
    }
    __syncthreads();
    int32_t* dw = p.dw + z * p.st_dw + chunk * p.st_dw2;
    if (p.st_split) {
        dw += (int64_t)blockIdx.x * p.st_split;
        for (int e = threadIdx.x; e < 64 * 12; e += 256) {
            const int cl = e / 12, t = e - cl * 12;
            if (cg0 + cl < C) dw[(int64_t)(cg0 + cl) * 12 + t] = t < 9 ? lacc[cl * 9 + t] : 0;
        }
    } else {
        for (int e = threadIdx.x; e < 64 * 9; e += 256) {
            const int cl = e / 9, t = e - cl * 9;
            if (cg0 + cl < C && lacc[e]) atomicAdd(dw + (int64_t)(cg0 + cl) * 12 + t, lacc[e]);
        }
    }
}

// Workgroups per chunk and channel group: about four per compute unit over all of them, each with at least two pieces per lane.
int dwconv_wgrad_splits(const ConvGeom& g, int64_t chunk_b, int problems)
{
    const int64_t cgroups = (g.Cin + 63) / 64;
    const int64_t most = chunk_b * dw_pieces_per_sample(g) / 32;
    const int64_t want = (int64_t)4 * num_cus() / (cgroups * problems);
    return (int)max((int64_t)1, min(want, most));
}

hipError_t launch_dwconv_wgrad(const DwArgs& p, hipStream_t s)
{
    const ConvGeom& g = p.g;
    if (p.B <= 0) return hipSuccess;
    if (g.ks != 3 || p.nc < 1 || p.splits < 1 || (int64_t)p.chunk_b * dw_pieces_per_sample(g) > 0x7FFFFFFF ||
        (g.Cin + 63) / 64 > 65535 || (int64_t)p.nb * p.nc > 65535)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_dwconv_wgrad, dim3((unsigned)p.splits, (unsigned)((g.Cin + 63) / 64), (unsigned)(p.nb * p.nc)), dim3(256),
                       0, s, p);
    return hipGetLastError();
}

}  // namespace ffi
