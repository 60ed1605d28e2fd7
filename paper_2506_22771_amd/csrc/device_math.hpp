// Device-side arithmetic shared by the HIP translation units of libffint8 (gfx950): wavefront reductions, the
// counter-based random word and the quantiser's code rule (Section IV: symmetric uniform quantiser; Section IV-B:
// stochastic rounding), and the exponential behind the loss derivatives (Eq. (1), Eq. (2)).  Every fp32 operation
// that decides an int8 code is a single correctly rounded IEEE operation in a fixed order: include this header only
// in files compiled with -ffp-contract=off.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ffi {

// ------------------------------------------------------------------------------------------------
// wavefront (64 lanes) reductions with DPP row operations + readlane across the four rows
// ------------------------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false);
}

// After this every lane of a 16-lane row holds the row's maximum.
__device__ __forceinline__ uint32_t row_max_u32(uint32_t v)
{
    v = max(v, dpp_u32<0xB1>(v));   // quad_perm [1,0,3,2]
    v = max(v, dpp_u32<0x4E>(v));   // quad_perm [2,3,0,1]
    v = max(v, dpp_u32<0x141>(v));  // row_half_mirror
    v = max(v, dpp_u32<0x140>(v));  // row_mirror
    return v;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = row_max_u32(v);
    uint32_t a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
    uint32_t c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(c, d));
}

// Waits for this wavefront's LDS operations.  The builtin and not inline assembly: the compiler counts it, where behind an assembly wait
// it still takes the reads before it for outstanding and, once younger ones are on their way, waits for those as well.
__device__ __forceinline__ void wait_lds()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    asm volatile("" ::: "memory");
}

// one random word per element: two multiply / xor-shift stages over (low index word ^ key).  sr_head leaves out the last
// xor-shift; the 24 bits that decide a code are then (head ^ head >> 16) >> 8 of what it returns (sr_top).
__device__ __forceinline__ uint32_t sr_head(uint32_t v)
{
    v ^= v >> 16;
    v *= 0x7FEB352Du;
    v ^= v >> 15;
    v *= 0x846CA68Bu;
    return v;
}
__device__ __forceinline__ uint32_t sr_mix(uint32_t v)
{
    v = sr_head(v);
    return v ^ (v >> 16);
}

// The same for four elements whose indices are base, base + 1, base + 2, base + 3 with base a multiple of four (v = base ^
// key, w[c] = sr_head(v ^ c)).  The four inputs differ in their two lowest bits only, so the first xor-shift is shared
// and the first of the two multiplies becomes one multiply plus additions:
// (x ^ 1) * m = x * m + (x & 1 ? -m : m), (x ^ 2) * m = x * m + (x & 2 ? -2m : 2m).
__device__ __forceinline__ void sr_head4(uint32_t v, uint32_t w[4])
{
    constexpr uint32_t M = 0x7FEB352Du;
    const uint32_t x = v ^ (v >> 16);
    const uint32_t s1 = (uint32_t)((int32_t)(x << 31) >> 31), s2 = (uint32_t)((int32_t)(x << 30) >> 31);   // all ones or zero
    const uint32_t d1 = (M ^ s1) - s1, d2 = ((2u * M) ^ s2) - s2;
    w[0] = x * M;
    w[1] = w[0] + d1;
    w[2] = w[0] + d2;
    w[3] = w[1] + d2;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        w[c] ^= w[c] >> 15;
        w[c] *= 0x846CA68Bu;
    }
}

// ------------------------------------------------------------------------------------------------
// Stochastic rounding in fixed point.  The code of t = v * inv is floor(t) + [k * 2^-24 < frac(t)], k the element's 24 random
// bits (quant_code below says it in floating point).  With X = ceil(t * 2^24) that is floor((X + 2^24 - 1 - k) / 2^24): the top
// byte of ~(k - 2^24 - X), |X| <= 127 * 2^24 once t is clamped.  t >= 1/2 is a multiple of 2^-24 already; for t < 0
// the floating-point form rounds frac(t) = t + 1 to fp32, which (t + 1) - 1 does here.  One clamp, one conversion and one
// addition instead of floor, two conversions, a compare, a carry and a clamp; the gfx950 VALU issues additions, multiplications and
// shifts at twice the rate of those.  Quantisers of tensors that fit the caches are bound by that issue.
// `sr_top` holds -X - 2^24 + k; four of them make a word of codes.  t may be infinite, where the bounds make it a code as any other
// t beyond them (activities that are rectified away only here may overflow on their way), but no NaN.
// ------------------------------------------------------------------------------------------------
constexpr float SR_MOST = 127.0f * 0x1p24f;
__device__ __forceinline__ int floor_to_int(float x)   // |x| < 2^31
{
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}
// scaled: -t * 2^24, rounded as above where t < 0; lo, hi: bounds of it (-SR_MOST, SR_MOST, or 0 where one sign is rectified away)
__device__ __forceinline__ uint32_t sr_top(float scaled, float lo, float hi, uint32_t head)
{
    const float c = __builtin_amdgcn_fmed3f(scaled, lo, hi);
    // (ones shifted in from above: one operation for the shift and the 0xFF000000; the other shift is an operand's byte select)
    return (__builtin_amdgcn_alignbit(0xFFFFFFFFu, head, 8) ^ (head >> 24)) + (uint32_t)floor_to_int(c);
}
// -t * 2^24 for t of either sign; one = 1 where t < 0, else 0
__device__ __forceinline__ float sr_scale(float t, float one) { return __builtin_fmaf(t + one, -0x1p24f, one * 0x1p24f); }
__device__ __forceinline__ float sr_one_if_negative(float t) { return __uint_as_float((uint32_t)(__float_as_int(t) >> 31) & 0x3F800000u); }
__device__ __forceinline__ uint32_t sr_pack(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    return ~(__builtin_amdgcn_perm(b, a, 0x0C0C0703u) | __builtin_amdgcn_perm(d, c, 0x07030C0Cu));
}

// STOCH: floor + Bernoulli(frac) from the counter-based word; else round-to-nearest-even.
// (quant_code: `word_in` is the element index ^ key; tensors have fewer than 2^32 elements.)
template <bool STOCH>
__device__ __forceinline__ int quant_code_of_word(float v, float inv, uint32_t random_word)
{
    const float t = v * inv;
    int code;
    if (STOCH) {
        const float f = floorf(t);
        const float frac = t - f;
        const float u = (float)(random_word >> 8) * 0x1p-24f;
        code = (int)f + (u < frac ? 1 : 0);
    } else {
        code = (int)rintf(t);
    }
    return min(max(code, -127), 127);
}
template <bool STOCH>
__device__ __forceinline__ int quant_code(float v, float inv, uint32_t word_in)
{
    return quant_code_of_word<STOCH>(v, inv, STOCH ? sr_mix(word_in) : 0u);
}

// v / d for v >= 0, d > 0 given y = 1 / d correctly rounded: one multiplication, the exact remainder, one correction
// (Markstein's theorem: the result is the correctly rounded quotient as long as nothing leaves the normal range).
__device__ __forceinline__ float div_by_reciprocal(float v, float d, float y)
{
    const float q = v * y;
    return __builtin_fmaf(__builtin_fmaf(-q, d, v), y, q);
}

// goodness of a sample from its integer sum: G = fp32(((fp64(sum) * 2^r) * s_y) * s_y)
__device__ __forceinline__ float goodness_value(unsigned long long gs, double pow2r, double s_yd)
{
    double g = (double)gs;
    g = g * pow2r;
    g = g * s_yd;
    g = g * s_yd;
    return (float)g;
}

// exp(z) for z <= 0 with a fixed operation sequence (it feeds the gradient quantiser through the sigmoid)
__device__ __forceinline__ float exp_nonpos(float z)
{
    // exp(z) for z <= 0 with a fixed operation sequence (it feeds the gradient quantiser through the sigmoid)
    z = fmaxf(z, -87.0f);
    z = fminf(z, 0.0f);
    const float kf = rintf(z * 0x1.715476p+0f);
    float r = __builtin_fmaf(-kf, 0x1.62e4p-1f, z);
    r = __builtin_fmaf(-kf, 0x1.7f7d1cp-20f, r);
    float p = 0x1.a01a02p-13f;
    p = __builtin_fmaf(p, r, 0x1.6c16c2p-10f);
    p = __builtin_fmaf(p, r, 0x1.111112p-7f);
    p = __builtin_fmaf(p, r, 0x1.555556p-5f);
    p = __builtin_fmaf(p, r, 0x1.555556p-3f);
    p = __builtin_fmaf(p, r, 0.5f);
    p = __builtin_fmaf(p, r, 1.0f);
    p = __builtin_fmaf(p, r, 1.0f);
    return ldexpf(p, (int)kf);
}

// dL/dG of one sample (Eq. (1): sign > 0, Eq. (2): sign < 0) from x = G - theta; xs: the argument of the softplus loss
__device__ __forceinline__ float loss_derivative(float x, int sign, float& xs)
{
    const float e = exp_nonpos(-fabsf(x));
    const float den = 1.0f + e;
    const float sig_big = 1.0f / den, sig_small = e / den;
    xs = sign > 0 ? -x : x;
    return sign > 0 ? -(x >= 0.0f ? sig_small : sig_big) : (x >= 0.0f ? sig_big : sig_small);
}
// softplus; it feeds no quantiser, so any accurate exp / log1p will do
__device__ __forceinline__ float loss_term(float xs) { return fmaxf(xs, 0.0f) + log1pf(expf(-fabsf(xs))); }

// Lanes of one wavefront exchange data through LDS: the hardware executes a wave's LDS
// instructions in order, but the compiler reasons per thread and, without a fence, may keep a value it loaded
// earlier instead of re-reading a location another lane has written since.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
}  // namespace ffi
