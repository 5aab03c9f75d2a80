// Device-side random-number primitives for gfx950.
//
// Method: Cuneo & Variansyah, "An Alternative to Stride-Based RNG for Monte
// Carlo Transport" (arXiv 2403.06362).
//   lcg_next ....... eq. (1), X <- (g X + c) mod 2^m; the new state is the output
//   affine_apply ... one factor of the skip-ahead of eq. (2): X <- G X + C mod 2^m
//   murmur_hash .... Listing 1, hash(k, s) with wrapping 64-bit multiplies
//   to_uniform ..... top 53 state bits, plus one, times 2^-53 (exact, in (0, 1])
//   fixed_neg_log .. natural log with a fixed IEEE operation sequence
//
// All 64-bit products are the low 64 bits of the full product; reduction
// modulo 2^m is a mask because 2^m divides 2^64.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mcrng {

struct LcgDev {
    uint64_t g;
    uint64_t c;
    uint64_t mask;      // 2^m - 1 (all ones for m = 64)
    uint32_t shift53;   // m - 53: right shift that keeps the top 53 state bits
    uint32_t m;
    uint64_t cz;        // c << up: the increment of the top-aligned state
    uint32_t up;        // 64 - m: the top-aligned state is Z = X << up
};

__device__ __forceinline__ uint64_t lcg_next(const LcgDev& L, uint64_t x) {
    return (L.g * x + L.c) & L.mask;
}

__device__ __forceinline__ uint64_t affine_apply(uint64_t G, uint64_t C, uint64_t mask, uint64_t x) {
    return (G * x + C) & mask;
}

constexpr uint64_t kMurmurM = 0xC6A4A7935BD1E995ull;

__host__ __device__ __forceinline__ uint64_t murmur_sub(uint64_t x) {
    const uint64_t y = x * kMurmurM;
    return y ^ (y >> 47);
}

// seed_hash = subhash(s ^ 8M) depends on the seed only; callers hoist it.
__host__ __device__ __forceinline__ uint64_t murmur_seed_part(uint64_t s) {
    return murmur_sub(s ^ (8ull * kMurmurM));
}

// The steps of hash(k, s) after the first product y = k M.
__host__ __device__ __forceinline__ uint64_t murmur_from_product(uint64_t y, uint64_t seed_part) {
    return murmur_sub(seed_part ^ ((y ^ (y >> 47)) * kMurmurM));
}

__host__ __device__ __forceinline__ uint64_t murmur_with_seed_part(uint64_t k, uint64_t seed_part) {
    return murmur_from_product(k * kMurmurM, seed_part);
}

__host__ __device__ __forceinline__ uint64_t murmur_hash(uint64_t k, uint64_t s) {
    return murmur_with_seed_part(k, murmur_seed_part(s));
}

// ------------------------------------------------------------ top-aligned states
// The transport and pulse kernels carry the state as Z = X << (64 - m).  One
// step is Z <- g Z + (c << (64 - m)) modulo 2^64, which is eq. (1) shifted, so
// no mask is left in the chain, and the 53 bits of the uniform sit in Z's top
// bits whatever m is, so every shift is a constant.
__device__ __forceinline__ uint64_t lcg_next_z(const LcgDev& L, uint64_t z) { return L.g * z + L.cz; }

// u = ((Z >> 11) + 1) 2^-53 = (hi 2^32 + (lo | 0x7ff) + 1) 2^-64: the low
// word goes into the mantissa of 2^-12 + lo 2^-64 (no conversion), the high
// word is converted; both sums are exact, u has 53 bits.  Five instructions
// (shift, 64-bit add, two conversions, multiply-add and scaling take seven).
__device__ __forceinline__ double uniform_z(uint64_t z) {
    const uint32_t lo = static_cast<uint32_t>(z) | 0x7ffu;
    const double a = __longlong_as_double(static_cast<long long>(0x3f30000000000000ull | lo));
    double hi;   // (a plain conversion of z >> 32 is widened to 64 bits: one more addition)
    asm("v_cvt_f64_u32 %0, %1" : "=v"(hi) : "v"(static_cast<uint32_t>(z >> 32)));
    return __builtin_fma(hi, 0x1p-32, a + (0x1p-64 - 0x1p-12));
}

// u < c for the uniform of state Z is Z < uniform_below(c): (T + 1) 2^-53 < c
// with T = Z >> 11 is T + 1 < ceil(c 2^53) (c 2^53 is exact).  0 <= c <= 1.
__host__ __device__ __forceinline__ uint64_t uniform_below(double c) {
    const uint64_t t = static_cast<uint64_t>(__builtin_ceil(c * 0x1p53));
    return t == 0 ? 0ull : (t - 1ull) << 11;
}

// ------------------------------------------------------------ lane masks and selects
// Wave masks live in scalar registers; a lane's bit is a condition again.
__device__ __forceinline__ uint64_t wave_mask(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

__device__ __forceinline__ uint32_t mask_count(uint64_t m) { return static_cast<uint32_t>(__popcll(m)); }

// A lane's rank among the lanes of a mask.
__device__ __forceinline__ uint32_t mask_rank(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

// A value that is the same on every lane, in scalar registers.
__device__ __forceinline__ uint64_t uniform_value(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
__device__ __forceinline__ double uniform_value(double v) {
    return __longlong_as_double(static_cast<long long>(uniform_value(static_cast<uint64_t>(__double_as_longlong(v)))));
}
__device__ __forceinline__ float uniform_value(float v) {
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}

// mask bit ? a : b, in the three-operand encoding.  The compiler selects with
// the short encoding through vcc, and on this chip two of those back to back
// (the halves of a 64-bit select) take 28 issue cycles, against 9 for the
// long encoding (measured at 8 waves per SIMD).  A mask that a vector
// compare has just written may be read as an operand two wait states later.
__device__ __forceinline__ uint32_t sel(uint64_t m, uint32_t a, uint32_t b) {
    uint32_t r;
    asm("s_nop 1\n\tv_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(b), "v"(a), "s"(uniform_value(m)));
    return r;
}
__device__ __forceinline__ float sel(uint64_t m, float a, float b) {
    return __uint_as_float(sel(m, __float_as_uint(a), __float_as_uint(b)));
}
__device__ __forceinline__ uint64_t sel(uint64_t m, uint64_t a, uint64_t b) {
    uint32_t lo, hi;
    asm("s_nop 1\n\tv_cndmask_b32_e64 %0, %2, %3, %6\n\tv_cndmask_b32_e64 %1, %4, %5, %6"
        : "=&v"(lo), "=v"(hi)
        : "v"(static_cast<uint32_t>(b)), "v"(static_cast<uint32_t>(a)), "v"(static_cast<uint32_t>(b >> 32)),
          "v"(static_cast<uint32_t>(a >> 32)), "s"(uniform_value(m)));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
__device__ __forceinline__ double sel(uint64_t m, double a, double b) {
    return __longlong_as_double(static_cast<long long>(sel(m, static_cast<uint64_t>(__double_as_longlong(a)),
                                                           static_cast<uint64_t>(__double_as_longlong(b)))));
}
// mask bit ? A : B with small constants (-16 .. 64).
template <int A, int B>
__device__ __forceinline__ uint32_t sel_const(uint64_t m) {
    uint32_t r;
    asm("s_nop 1\n\tv_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "n"(B), "n"(A), "s"(uniform_value(m)));
    return r;
}
// mask bit ? v : 0
__device__ __forceinline__ uint32_t sel_or_zero(uint64_t m, uint32_t v) {
    uint32_t r;
    asm("s_nop 1\n\tv_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(v), "s"(uniform_value(m)));
    return r;
}

// Minima and maxima of numbers (never NaN), one instruction each: fmin and
// fmax of a loaded value first quiet it with another.
__device__ __forceinline__ double min_num(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double max_num(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float min_num(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float max_num(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// ------------------------------------------------------------ division
// A correctly rounded quotient a / b is, on this hardware, the reciprocal
// r = rcp(b) refined by Newton steps r <- r + r (1 - b r) (two in double
// precision, one in single), the product q = a r and residual corrections
// q <- q + (a - b q) r (one in double, two in single), each a fused
// multiply-add, wrapped in operand scaling that acts only near the ends of
// the exponent range.  The refined reciprocal depends on b alone, so a
// divisor used many times (a cell's sigma_t, a flight's direction cosine)
// has it computed once.  quot(a, b, recip_refined(b)) then equals a / b bit
// for bit wherever the scaling does not act and no intermediate leaves the
// normal range, which holds when |a| is at least 2^-900 (single: 2^-100), the
// quotient is at least 2^-700 (single: 2^-36), b is nonzero with |b| in
// [2^-64, 2^64] and |a| is at most 2^42: what the transport's validated
// geometry allows above the smallest quotient.  The callers take the plain
// division for a smaller one (below_quot_min).  a = 0 gives 0 (its sign never
// matters); b = 0 gives NaN.
__device__ __forceinline__ double recip_refined(double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
    return r;
}

__device__ __forceinline__ double quot(double a, double b, double r) {
    const double q = a * r;
    return __builtin_fma(__builtin_fma(-b, q, a), r, q);
}

__device__ __forceinline__ float recip_refined(float b) {
    const float r = __builtin_amdgcn_rcpf(b);
    return __builtin_fmaf(__builtin_fmaf(-b, r, 1.0f), r, r);
}

__device__ __forceinline__ float quot(float a, float b, float r) {
    float q = a * r;
    q = __builtin_fmaf(__builtin_fmaf(-b, q, a), r, q);
    return __builtin_fmaf(__builtin_fmaf(-b, q, a), r, q);
}

// With b a cross section in [2^-64, 2^64] or a direction cosine (a multiple
// of 2^-52, at most 1), a quotient of at least 2^-700
// (single: 2^-36) has |a| >= 2^-764
// (single: 2^-100), so one comparison of the smaller of a flight's two
// distances covers both divisions.
// The comparison is on the bits (s >= 0; a -0 counts as large, and its
// quotient is right), so that the bound is a literal.
__device__ __forceinline__ bool below_quot_min(double s) {   // s < 2^-700
    return static_cast<uint32_t>(static_cast<uint64_t>(__double_as_longlong(s)) >> 32) < 0x14300000u;
}
__device__ __forceinline__ bool below_quot_min(float s) {    // s < 2^-36
    return __float_as_uint(s) < 0x2d800000u;
}

// Natural logarithm of u in (0, 1] (any positive normal double works).
// Fixed sequence of IEEE double operations, each rounded to nearest, no
// fused multiply-add (the library is compiled with -ffp-contract=off):
//   u = f 2^e, f in [1, 2); f >= 3/2 -> f/2, e+1;  a = f - 1 (exact)
//   s = a / (2 + a);  w = s s;  p = 2/23, then p = p w + 2/(2k+1) for
//   k = 10 .. 1 (multiply and add rounded separately);  h = w p;
//   ln(1 + a) = a - s (a - h);  ln u = e LN2_HI + (ln(1 + a) + e LN2_LO)
// ln(1 + a) = 2 atanh(s) = 2s + sum_k 2 s^(2k+1)/(2k+1) and 2s = a - a s.
// LN2_HI is ln 2 truncated to 40 fraction bits, LN2_LO the double nearest
// to the rest.  Within 1.25 ulp of the exact logarithm.
// Returns -ln u (the negation is exact).
__device__ __forceinline__ double fixed_neg_log(double u) {
    constexpr double kLn2Hi = 0x1.62e42fefa2000p-1;
    constexpr double kLn2Lo = 0x1.9ef35793c7673p-41;
    constexpr double kC[12] = {0.0,        2.0 / 3.0,  2.0 / 5.0,  2.0 / 7.0,
                               2.0 / 9.0,  2.0 / 11.0, 2.0 / 13.0, 2.0 / 15.0,
                               2.0 / 17.0, 2.0 / 19.0, 2.0 / 21.0, 2.0 / 23.0};
    // u = m 2^E, m in [1/2, 1): m < 3/4 gives f = 2m, e = E - 1, else f = m, e = E
    const double m = __builtin_amdgcn_frexp_mant(u);
    const uint32_t i = sel_const<1, 0>(wave_mask(m < 0.75));
    const int e = __builtin_amdgcn_frexp_exp(u) - static_cast<int>(i);
    const double f = __builtin_amdgcn_ldexp(m, static_cast<int>(i));
    const double a = f - 1.0;
    const double b = 2.0 + a;
    const double s = quot(a, b, recip_refined(b));   // a in {0} or [2^-53, 1/2), b in [7/4, 5/2)
    const double w = s * s;
    double p = kC[11];
#pragma unroll
    for (int k = 10; k >= 1; --k) {
        p = p * w;
        p = p + kC[k];
    }
    const double h = w * p;
    const double t = a - h;
    const double c = s * t;
    const double l = a - c;
    const double ed = static_cast<double>(e);
    const double r = l + ed * kLn2Lo;
    return ed * -kLn2Hi - r;   // -(ed kLn2Hi + r)
}

// Quantised track length: q = round-half-even(s * 2^56) for 0 <= s < 2^7.
__device__ __forceinline__ uint64_t quantise(double s) {
    return static_cast<uint64_t>(__builtin_rint(s * 0x1p56));
}

// q as two limbs, q = lo + 2^32 hi, 0 <= hi < 2^31, |lo| <= 2^31, each a
// 64-bit word (lo signed).  Adding 1.5 x 2^28 rounds s to a multiple of 2^-24
// and leaves that multiple in the sum's low word; the exact rest (at most
// 2^-25) plus 1.5 x 2^-4 rounds half-even to a multiple of 2^-56 (2^32 hi is
// even, so ties go the same way as in one rounding of s), left in the low
// word with its sign borrowed from the high word.
struct Limbs {
    uint64_t lo, hi;
};
__device__ __forceinline__ Limbs quantise_limbs(double s) {
    const double t = s + 0x1.8p28;
    const double rest = s - (t - 0x1.8p28);
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(rest + 0x1.8p-4));
    Limbs q;
    q.lo = (static_cast<uint64_t>(static_cast<uint32_t>(u >> 32) - 0x3fb80000u) << 32) | static_cast<uint32_t>(u);
    q.hi = static_cast<uint32_t>(static_cast<uint64_t>(__double_as_longlong(t)));
    return q;
}

}  // namespace mcrng
