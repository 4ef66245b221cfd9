// Device-side helpers shared by the gfx950 NVFP4 kernels: format conversions,
// exact rounding decisions, wavefront reductions.  (Sec. 2.2 "NVFP4
// Preliminaries"; Appendix "Scale Search NVFP4 Quantization", Eq. 12.)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));

namespace nvfp4 {

constexpr int kWave = 64;
constexpr float kFp4Max = 6.0f;      // M^FP4
constexpr float kFp8Max = 448.0f;    // M^FP8

__device__ __forceinline__ float bf16lo_to_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi_to_f32(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// two fp32 -> packed bf16 (round to nearest even), one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef float float2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
    float2v v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
}

// max of the absolute values of two packed bf16 pairs, on their bit patterns
// (|bf16| patterns order like unsigned integers).
__device__ __forceinline__ uint32_t pk_absmax_u16(uint32_t acc, uint32_t w)
{
    uint32_t a = w & 0x7FFF7FFFu;
    ushort2v x = __builtin_bit_cast(ushort2v, acc), y = __builtin_bit_cast(ushort2v, a);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(x, y));
}
__device__ __forceinline__ uint32_t pk_hmax_u16(uint32_t p) { return max(p & 0xFFFFu, p >> 16); }

// ---- wavefront max over 64 lanes with DPP (unsigned compare) -------------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max_step(uint32_t v)
{
    uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
    return max(v, o);
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = dpp_max_step<0xB1>(v);    // quad_perm [1,0,3,2]
    v = dpp_max_step<0x4E>(v);    // quad_perm [2,3,0,1]
    v = dpp_max_step<0x124>(v);   // row_ror:4
    v = dpp_max_step<0x128>(v);   // row_ror:8  -> every lane holds its 16-lane row max
    uint32_t a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
    uint32_t c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(c, d));
}

// ---- E4M3 (1-4-3, bias 7, max 448) ---------------------------------------
// byte 0x00..0x7E -> value, exact
__device__ __forceinline__ float e4m3_to_f32(uint32_t b)
{
    float normal = __uint_as_float((b << 20) + (120u << 23));
    float sub = (float)(b & 7u) * 0.001953125f;    // m * 2^-9
    return (b >> 3) ? normal : sub;
}

// ---- Four-over-Six scale search (Appendix "Scale Search NVFP4 Quantization", Eq. 12-13) ----
// The squared errors of a block under two encodings, as the fp64 definition evaluates them: every difference x - m s_b s_g
// (m signed like x) taken once in fp64, squared, and summed in element order, each operation rounded on its own (no fused
// multiply-add), so that "is candidate 4 strictly better" has one answer everywhere.
// Taken by a few blocks of every tensor (equal errors are common), and a launch ends with the slowest of its waves: the
// two chains run side by side, unrolled (a rolled loop over the elements took 4 us, as long as the rest of a small call).
__device__ __forceinline__ bool second_is_closer_f64(const uint32_t (&w)[8], const uint32_t (&ca)[2], const uint32_t (&cb)[2], float sba, float sbb, float sg)
{
    // (under the default contraction mode the compiler fuses these into multiply-adds: one rounding where the
    //  definition has two, and a different answer on blocks whose two errors are equal in exact arithmetic.  Plain
    //  operators: contraction is switched off for this function; the rounding intrinsics are inlined with the
    //  contraction mode of their own header and would be fused all the same)
#pragma clang fp contract(off)
    typedef float float2v __attribute__((ext_vector_type(2)));
    // (the codes are decoded anew: kept from the comparison before, the decoded values would cost the kernel 20 registers)
    uint32_t a[2] = {ca[0], ca[1]}, b[2] = {cb[0], cb[1]};
    asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(b[0]), "+v"(b[1]));
    const double dena = (double)sba * (double)sg, denb = (double)sbb * (double)sg;      // exact
    double ea = 0.0, eb = 0.0;
    auto one = [&](float x, float ma, float mb) {
#pragma clang fp contract(off)
        const double pa = (double)ma * dena, pb = (double)mb * denb;
        const double da = (double)x - pa, db = (double)x - pb;
        const double qa = da * da, qb = db * db;
        ea = ea + qa;
        eb = eb + qb;
    };
#define NVFP4_STEP(K, SEL)                                                                       \
    {                                                                                            \
        const float2v ma = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(a[K >> 2], 1.0f, SEL);       \
        const float2v mb = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(b[K >> 2], 1.0f, SEL);       \
        one(bf16lo_to_f32(w[K]), ma.x, mb.x);                                                    \
        one(bf16hi_to_f32(w[K]), ma.y, mb.y);                                                    \
        __builtin_amdgcn_sched_barrier(0);      /* two elements at a time: more would cost waves their registers */ \
    }
    NVFP4_STEP(0, 0) NVFP4_STEP(1, 1) NVFP4_STEP(2, 2) NVFP4_STEP(3, 3)
    NVFP4_STEP(4, 0) NVFP4_STEP(5, 1) NVFP4_STEP(6, 2) NVFP4_STEP(7, 3)
#undef NVFP4_STEP
    return eb < ea;
}

// ---- tensor scales outside the range in which the fp32 quotients above are safe ----------------------
// Below s_g = 2^-100 or above 2^100 the reciprocal 1 / (M s_g) or the products s_b s_g leave the normal fp32
// range.  Every decision of the quantizer compares ratios, so it commutes with multiplying the tensor AND its
// scale by a power of two: such tensors are encoded as (x 2^k, s_g 2^k) with k = +96 or -96, which puts the scale
// back into range.  The scaled elements are exact (bf16 has the exponent range of fp32) except those that underflow
// when a huge tensor is scaled down: they are below 2^-30, more than a hundred binades under a quarter of the
// smallest block scale times s_g, so their code is zero either way, and so is the scale of a block made of them.
// The stored tensor scale is the unscaled one.  The test is the same for every lane: a scalar branch.
__device__ __forceinline__ void rescale_block16(uint32_t (&w)[8], float f)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = pack_bf16x2(bf16lo_to_f32(w[i]) * f, bf16hi_to_f32(w[i]) * f);
}

// sixteen values -> their largest magnitude through a tree of three-operand maxima (depth 3 instead of 8)
__device__ __forceinline__ float absmax16_tree(const float (&f)[16])
{
    auto m3 = [](float a, float b, float c) { return fmaxf(fmaxf(fabsf(a), fabsf(b)), fabsf(c)); };
    const float t0 = m3(f[0], f[1], f[2]), t1 = m3(f[3], f[4], f[5]), t2 = m3(f[6], f[7], f[8]);
    const float t3 = m3(f[9], f[10], f[11]), t4 = m3(f[12], f[13], f[14]);
    return fmaxf(m3(t0, t1, t2), m3(t3, t4, f[15]));
}

__device__ __forceinline__ void unpack16(const uint32_t (&w)[8], float (&f)[16])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        f[2 * i] = bf16lo_to_f32(w[i]);
        f[2 * i + 1] = bf16hi_to_f32(w[i]);
    }
}

// ---- one-sided encoder ------------------------------------------------------------------------------
// Every rounding decision of the plain rule compares a short number with a multiple of the tensor scale: an element
// |x| with c s_g, c = T s_b (T a midpoint between two E2M1 magnitudes, s_b an E4M3 value), or a block maximum with
// c s_g, c = M q (q a midpoint between two E4M3 values, M the target magnitude 6 or 4).  Up to powers of two |x| is an
// integer below 2^8 and c is one of the odd numbers below 2^7 that tie_candidate() lists, so two different quotients
// |x| / c differ by more than 2^-15 of their value and at most ONE of them lies near s_g.  A quotient within 2^-17 of
// s_g is therefore always the same one for the whole tensor: all the near-ties of a tensor lie on the same side of
// their midpoints, the side on which s_g lies of that quotient.  So instead of converting both ends of a bracket and
// settling the codes on which they differ, the tensor scale that the quotients are formed with is moved by 2^-18 away
// from it, once per tensor: a near-tie then lands on its own side (2^-18 is eight times what the fp32 evaluation can
// be off by), anything else is further than 2^-17 from a midpoint and does not cross it.  Where s_g equals the
// quotient exactly (an eighth of the bf16 maxima) the near-ties are ties, and the quotients are rounded to 17
// significant bits, which puts them exactly on the midpoint; the conversions then round to the even code.
// About 75 instruction slots per block against 190 for the bracket (16 unpack, 8 maximum, about 10 scale, 16 multiplies,
// 8 conversions of up to three slots), and no data-dependent loop: the streaming pass of the plain rule issues vector
// instructions in half of the SIMDs' cycles and is bound by memory.
struct TensorScale {
    float sg;          // the tensor scale, shifted into the fp32-safe range
    float nudged;      // sg (1 -+ 2^-18), what quotients are formed with
    float inv6, inv4;  // 1 / (6 nudged), 1 / (4 nudged)
    float shift;       // 1, or the power of two that the tensor is multiplied by before it is encoded (see above)
    bool snap;         // sg is a tie itself: round the quotients to 17 bits
};

// the odd parts of all c: {1,3,5,7} x {1..15} (elements; subnormal block scales' midpoints; 4-bit scale midpoints
// with M = 6), 3 x {17..31} and {17..31} (block scales with M = 6 and M = 4)
__device__ __forceinline__ uint32_t tie_candidate(uint32_t lane)
{
    if (lane < 32u) return (2u * (lane & 3u) + 1u) * (2u * (lane >> 2) + 1u);
    return (lane < 40u ? 3u : 1u) * (17u + 2u * (lane & 7u));
}

// Every lane of the wave calls this (lane l tests candidate l); the result is the same for all of them.
__device__ __forceinline__ TensorScale tensor_scale(float sg_given)
{
    TensorScale t;
    const float g = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sg_given)));
    t.shift = g < 0x1p-100f ? 0x1p96f : (g > 0x1p100f ? 0x1p-96f : 1.0f);
    t.sg = g * t.shift;
    const float c = (float)tie_candidate(threadIdx.x & 63u), m = c * t.sg;
    const float x = bf16lo_to_f32(pack_bf16x2(m, 0.0f));                   // the nearest 8-bit number
    const float d = __builtin_fmaf(c, t.sg, -x);                           // exact where it is small
    const bool near = fabsf(d) <= 0x1p-17f * m;
    const bool below = __ballot(near & (d > 0.0f)) != 0ull;                // quotients lie below their midpoints
    const bool above = __ballot(near & (d < 0.0f)) != 0ull;
    t.snap = __ballot(near & (d == 0.0f)) != 0ull;
    const float f = below ? 1.0f + 0x1p-18f : (above ? 1.0f - 0x1p-18f : 1.0f);
    t.nudged = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(t.sg * f)));
    t.inv6 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(1.0f / (6.0f * t.nudged))));
    t.inv4 = 1.5f * t.inv6;                                                // (one more rounding: 2^-18 is far above it)
    return t;
}

// nearest number of 17 significant bits (either sign; ties away from zero, which no quotient meets)
__device__ __forceinline__ float snap17(float y) { return __uint_as_float((__float_as_uint(y) + 0x40u) & 0xFFFFFF80u); }

// E4M3 byte nearest to q >= 0 (ties to even, gradual underflow, at most 448) and its value, by the hardware conversions
// (checked against integer arithmetic for every float from 0 to 512)
__device__ __forceinline__ uint32_t e4m3_byte(float q)
{
    const float s = fminf(q, kFp8Max);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(s, s, 0, false) & 0xFFu;
}
__device__ __forceinline__ float e4m3_value(uint32_t b) { return __builtin_amdgcn_cvt_f32_fp8((int)b, 0); }

// scale byte of a block from its largest magnitude (inv_m: 1 / (M nudged) for the target magnitude M), its value, and
// the factor that turns the block's elements into quotients
__device__ __forceinline__ void block_scale(float bmax, float inv_m, const TensorScale &t, uint32_t &sbyte, float &sb, float &inv)
{
    float q = bmax * inv_m;
    if (t.snap) q = snap17(q);
    sbyte = e4m3_byte(q);
    sb = e4m3_value(sbyte);
    const float r = __builtin_amdgcn_rcpf(sb * t.nudged);
    inv = sbyte == 0u ? 0.0f : r;
}
__device__ __forceinline__ void block_scale(float bmax, const TensorScale &t, uint32_t &sbyte, float &inv)
{
    float sb;
    block_scale(bmax, t.inv6, t, sbyte, sb, inv);
}

// Sixteen values -> sixteen codes, N chains side by side (a conversion writes one byte of its destination, so the four
// that fill a code word wait on one another; a second chain hides that).  step 0: every chain encodes the same values.
template <int N>
struct Rows16 {
    const float (*row)[16];
    int step;
    __device__ __forceinline__ float at(int n, int i) const { return row[n * step][i]; }
};
template <bool SNAP, int N>
__device__ __forceinline__ void convert_codes(const Rows16<N> f, const float (&inv)[N], uint32_t (&c)[N][2])
{
    auto q = [&](int n, int i) {
        const float y = f.at(n, i) * inv[n];
        return SNAP ? snap17(y) : y;
    };
#pragma unroll
    for (int n = 0; n < N; ++n) c[n][0] = c[n][1] = 0u;
#define NVFP4_STEP(SEL)                                                                                              \
    _Pragma("unroll") for (int h = 0; h < 2; ++h) _Pragma("unroll") for (int n = 0; n < N; ++n)                     \
        c[n][h] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c[n][h], q(n, 8 * h + 2 * SEL), q(n, 8 * h + 2 * SEL + 1), 1.0f, SEL);
    NVFP4_STEP(0) NVFP4_STEP(1) NVFP4_STEP(2) NVFP4_STEP(3)
#undef NVFP4_STEP
}
template <int N>
__device__ __forceinline__ void encode_values(const Rows16<N> f, const float (&inv)[N], bool snap, uint32_t (&c)[N][2])
{
    if (__builtin_expect(snap, 0)) convert_codes<true, N>(f, inv, c);      // (the same for every lane)
    else convert_codes<false, N>(f, inv, c);
}

// Plain rule (Eq. 1: block maximum -> 6) on one block of eight packed pairs, already inside the fp32-safe range
__device__ __forceinline__ void quantize_block16(const uint32_t (&w)[8], const TensorScale &t, uint32_t &sbyte, uint32_t &c0, uint32_t &c1)
{
    float f[1][16], inv[1];
    uint32_t c[1][2];
    unpack16(w, f[0]);
    block_scale(absmax16_tree(f[0]), t, sbyte, inv[0]);
    encode_values<1>({f, 1}, inv, t.snap, c);
    c0 = c[0][0];
    c1 = c[0][1];
}
// ... and on two blocks side by side
__device__ __forceinline__ void quantize_pair16(const uint32_t (&wa)[8], const uint32_t (&wb)[8], const TensorScale &t,
                                                uint32_t &sa, uint32_t &a0, uint32_t &a1, uint32_t &sb, uint32_t &b0, uint32_t &b1)
{
    float f[2][16], inv[2];
    uint32_t c[2][2];
    unpack16(wa, f[0]);
    unpack16(wb, f[1]);
    block_scale(absmax16_tree(f[0]), t, sa, inv[0]);
    block_scale(absmax16_tree(f[1]), t, sb, inv[1]);
    encode_values<2>({f, 1}, inv, t.snap, c);
    a0 = c[0][0]; a1 = c[0][1];
    b0 = c[1][0]; b1 = c[1][1];
}

// Scale search (Eq. 12-13) on one block: the block maximum mapped to 6 and to 4, both encodings settled as above, the
// one with the strictly smaller squared error kept (equal errors keep 6).  Which error is smaller is decided by the
// cheapest evaluation that is sure of it:
//  1. with m the decoded magnitudes (signed like x) and den = s_b s_g, the error is sum x^2 - den (2 S - den Q),
//     S = sum x m, Q = sum m^2, so the candidate with the larger gain den (2 S - den Q) wins.  S and Q are two-element
//     dot products on the packed bf16 pairs themselves.  Q is exact (quarter integers up to 576); all terms of S are
//     non-negative, a dot product step is off by less than 2^-22 of its sum (two fp32 roundings: 2^-23 measured), so
//     S is off by less than 2^-20.8 of itself over chains of two steps and the additions behind them, and the gain by
//     less than 2^-19.5 den S.  About one block in a thousand of Gaussian data is closer than the 2^-19 den S taken here;
//  2. the errors themselves in fp32.  |d~ - d| <= 2^-24 (|x| + |x^| + 6 den) < u; |d~^2 - d^2| <= u (2 |d~| + u), and
//     the sixteen |d~| add up to at most 4 sqrt(sum d~^2) (Cauchy-Schwarz; 4.01 covers the approximate square root
//     and the rounding of the sum); sixteen fused accumulations add at most 2^-19 of the sum.  One block in 10^4 to
//     10^5 is still open;
//  3. the fp64 definition.
// Gains and errors below 2^-100, where fp32 may lose its relative accuracy, or that are no finite numbers are never sure.
// Bound by VALU issue (in 69 % of the SIMDs' cycles in the streaming passes of the search and of the smoothed keys) and by the latency
// of the one block in flight: 224 vector instructions per block in the compiled pass (the bracketed search took about 450), the
// largest groups 16 unpack, 8 maximum, 20 scales, 32 multiplies, 32 conversions, 32 dot products.
__device__ __forceinline__ float block_error_f32(const float (&f)[16], const uint32_t (&c)[2], float den)
{
    typedef float float2v __attribute__((ext_vector_type(2)));
    float err = 0.0f;
#define NVFP4_STEP(K, SEL)                                                                 \
    {                                                                                      \
        const float2v q = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[K >> 2], 1.0f, SEL);  \
        const float d0 = __builtin_fmaf(-q.x, den, f[2 * K]), d1 = __builtin_fmaf(-q.y, den, f[2 * K + 1]); \
        err = __builtin_fmaf(d0, d0, err);                                                 \
        err = __builtin_fmaf(d1, d1, err);                                                 \
    }
    NVFP4_STEP(0, 0) NVFP4_STEP(1, 1) NVFP4_STEP(2, 2) NVFP4_STEP(3, 3)
    NVFP4_STEP(4, 0) NVFP4_STEP(5, 1) NVFP4_STEP(6, 2) NVFP4_STEP(7, 3)
#undef NVFP4_STEP
    return err;
}
// S and Q of one candidate
__device__ __forceinline__ void block_products(const uint32_t (&w)[8], const uint32_t (&c)[2], float &S, float &Q)
{
    typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f}, q[2] = {0.0f, 0.0f};
#define NVFP4_STEP(K, SEL)                                                                                        \
    {                                                                                                             \
        const bf16x2v m = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c[K >> 2], 1.0f, SEL);                        \
        s[K & 3] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, w[K]), m, s[K & 3], false);        \
        q[K & 1] = __builtin_amdgcn_fdot2_f32_bf16(m, m, q[K & 1], false);                                        \
    }
    NVFP4_STEP(0, 0) NVFP4_STEP(1, 1) NVFP4_STEP(2, 2) NVFP4_STEP(3, 3)
    NVFP4_STEP(4, 0) NVFP4_STEP(5, 1) NVFP4_STEP(6, 2) NVFP4_STEP(7, 3)
#undef NVFP4_STEP
    S = (s[0] + s[1]) + (s[2] + s[3]);
    Q = q[0] + q[1];
}
__device__ __forceinline__ void quantize_block16_4over6(const uint32_t (&w)[8], const TensorScale &t, uint32_t &sbyte, uint32_t &c0, uint32_t &c1)
{
    float f[16], sb[2], inv[2];
    uint32_t s[2], c[2][2];                                    // [0]: maximum -> 6, [1]: maximum -> 4
    unpack16(w, f);
    const float bmax = absmax16_tree(f);
    block_scale(bmax, t.inv6, t, s[0], sb[0], inv[0]);
    block_scale(bmax, t.inv4, t, s[1], sb[1], inv[1]);
    encode_values<2>({&f, 0}, inv, t.snap, c);                 // both candidates of the one block
    const float den6 = sb[0] * t.sg, den4 = sb[1] * t.sg;
    float S6, Q6, S4, Q4;
    block_products(w, c[0], S6, Q6);
    block_products(w, c[1], S4, Q4);
    const float g6 = den6 * __builtin_fmaf(-den6, Q6, 2.0f * S6), g4 = den4 * __builtin_fmaf(-den4, Q4, 2.0f * S4);
    const float r = 0x1p-19f * __builtin_fmaf(den6, S6, den4 * S4), diff = g4 - g6;
    bool pick4 = diff > r;
    const bool same = s[0] == s[1];                            // (saturated scales, zero blocks: same codes, same error, 6 is kept)
    const bool sure = (fabsf(diff) > r) & (fminf(g6, g4) > 0x1p-100f) & (fmaxf(g6, g4) < 0x1p120f);
    if (__builtin_expect(!(sure | same), 0)) {
        const float e6 = block_error_f32(f, c[0], den6), e4 = block_error_f32(f, c[1], den4);
        const float u6 = 0x1p-22f * (bmax + 6.0f * den6), u4 = 0x1p-22f * (bmax + 6.0f * den4);
        const float r6 = u6 * (8.02f * __builtin_amdgcn_sqrtf(e6) + 16.0f * u6) + 0x1p-19f * e6;
        const float r4 = u4 * (8.02f * __builtin_amdgcn_sqrtf(e4) + 16.0f * u4) + 0x1p-19f * e4;
        pick4 = e4 + r4 < e6 - r6;
        const bool settled = !(fminf(e4, e6) < 0x1p-100f) & (pick4 | (e4 - r4 > e6 + r6));
        if (__builtin_expect(!settled, 0))
            pick4 = second_is_closer_f64(w, c[0], c[1], sb[0], sb[1], t.sg);
    }
    pick4 &= !same;
    sbyte = pick4 ? s[1] : s[0];
    c0 = pick4 ? c[1][0] : c[0][0];
    c1 = pick4 ? c[1][1] : c[0][1];
}

// Round a non-negative exact product held in a double to bf16 once (nearest
// even): go through fp32 with round-to-odd so the second rounding is innocuous.
__device__ __forceinline__ uint32_t bf16_rne_from_f64(double p)
{
    float hi = (float)p;
    double rem = p - (double)hi;                  // exact
    uint32_t u = __float_as_uint(hi);
    if (rem < 0.0) u -= 1u;                       // truncate toward zero
    if (rem != 0.0) u |= 1u;                      // sticky
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// Signed variant: nearest-even bf16 of any finite double (sign kept, also for zero results).
__device__ __forceinline__ uint32_t bf16_rne_signed_from_f64(double v)
{
    const uint32_t sign = (uint32_t)(__double_as_longlong(v) >> 48) & 0x8000u;
    return sign | bf16_rne_from_f64(fabs(v));
}

// K-smoothing (Sec. 3.2, Eq. 6) of one 16-element block given its row mean (a bf16 value):
// x_j -> RN_bf16(x_j - mean), one rounding of the exact difference.  An fp32 subtraction
// followed by the rounding to bf16 gives exactly that for every pair of finite bf16 numbers:
// when the exponents are at most 15 apart the fp32 difference is exact (8 + 15 + 1 bits), and
// when they are further apart the smaller operand is below 2^-15 of the larger, which is a
// bf16 number at least 2^-10 of its magnitude away from the nearest rounding boundary, so both
// the exact difference and its fp32 rounding round to that operand.
__device__ __forceinline__ void smooth_block16(uint32_t (&w)[8], float mu)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = pack_bf16x2(bf16lo_to_f32(w[i]) - mu, bf16hi_to_f32(w[i]) - mu);
}

// Mean of a row of d = 16 nb_row features (nb_row a power of two up to 64, one 16-element block per lane, the row's
// lanes neighbours), rounded to bf16: RN_bf16(sum / d) of the exact sum.  Every lane of the wave calls this.
// The sum is taken in fp32: 4 + log2(nb_row) <= 10 rounded levels, each off by at most 2^-24 of the sum of magnitudes, and
// one more rounding for either end of the interval, so the exact mean lies between the ends at e = 11.1 * 2^-24 * (row
// maximum) around the fp32 one; where both round to the same bf16 number, that is the mean.  Otherwise (one row in a few hundred, rows whose terms cancel, and rows that fp32
// could overflow on) the wave takes the sum in fp64, which is exact for rows whose values span less than 2^40.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) { return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, true)); }
__device__ __forceinline__ uint32_t row_mean_bits(const uint32_t (&w)[8], int nb_row)
{
    float f[16], s[16];
    unpack16(w, f);
    float mx = absmax16_tree(f);
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = f[i];
#pragma unroll
    for (int h = 8; h > 0; h >>= 1)
#pragma unroll
        for (int i = 0; i < h; ++i) s[i] += s[i + h];
    float sum = s[0];
    // lane ^ 1, ^ 2 by quad permutations; ^ 4, ^ 8 by mirrors (the lanes of a half already agree); then shuffles
    if (nb_row > 1) { sum += dpp_f32<0xB1>(sum); mx = fmaxf(mx, dpp_f32<0xB1>(mx)); }
    if (nb_row > 2) { sum += dpp_f32<0x4E>(sum); mx = fmaxf(mx, dpp_f32<0x4E>(mx)); }
    if (nb_row > 4) { sum += dpp_f32<0x141>(sum); mx = fmaxf(mx, dpp_f32<0x141>(mx)); }
    if (nb_row > 8) { sum += dpp_f32<0x140>(sum); mx = fmaxf(mx, dpp_f32<0x140>(mx)); }
    for (int m = 16; m < nb_row; m <<= 1) { sum += __shfl_xor(sum, m, 64); mx = fmaxf(mx, __shfl_xor(mx, m, 64)); }
    const float mean = sum * (1.0f / (float)(16 * nb_row)) + 0.0f;           // (a power of two; a zero is +0)
    const float e = 11.1f * 0x1p-24f * mx;
    const uint32_t ends = pack_bf16x2(mean - e, mean + e);
    uint32_t bits = ends & 0xFFFFu;
    const bool sure = (bits == ends >> 16) & (mx < 0x1p110f);
    if (__ballot(!sure) != 0ull) {
        double d = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) d += (double)f[i];
        for (int m = 1; m < nb_row; m <<= 1) d += __shfl_xor(d, m, 64);
        const uint32_t exact = bf16_rne_signed_from_f64(d * (1.0 / (double)(16 * nb_row)));
        bits = sure ? bits : exact;
    }
    return bits;
}

// Random Hadamard transform (Sec. 2.2, weight-gradient operands) of one group of 16 values
// held as eight packed bf16 pairs: y = (1/4) H16 diag(s) v, H16[i][j] = (-1)^popcount(i & j),
// s_j = -1 where bit j of sign_mask is set.  Fast Walsh-Hadamard butterflies in fp64 (exact
// while the 16 values span less than 2^40), one rounding to bf16.
__device__ __forceinline__ void rht_block16(uint32_t (&w)[8], uint32_t sign_mask)
{
    double v[16];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        v[2 * i] = (double)bf16lo_to_f32(w[i]);
        v[2 * i + 1] = (double)bf16hi_to_f32(w[i]);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if ((sign_mask >> j) & 1u) v[j] = -v[j];
#pragma unroll
    for (int h = 1; h < 16; h <<= 1)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if ((i & h) == 0) {
                const double a = v[i], b = v[i + h];
                v[i] = a + b;
                v[i + h] = a - b;
            }
#pragma unroll
    for (int i = 0; i < 8; ++i)
        // (+ 0.0: a sum that is zero is +0, as when the terms are added up from zero; only groups of negative zeros differ)
        w[i] = bf16_rne_signed_from_f64(0.25 * v[2 * i] + 0.0) | (bf16_rne_signed_from_f64(0.25 * v[2 * i + 1] + 0.0) << 16);
}

// The same transform in fp32 arithmetic, and the test that tells when it returns the same bits.  With all non-zero
// magnitudes of the group within 12 binades of the largest, every value is a multiple of 2^(e_min - 7) and every
// partial sum stays below 2^(e_max + 5): at most 24 significant bits, so fp32 sums of the sixteen terms are exact in
// any order and the one rounding to bf16 (v_cvt_pk_bf16_f32, nearest even) is the rounding of the exact value, as in
// the fp64 form.  Groups near the ends of the exponent range (sums that could overflow, results that could be
// subnormal) fail the test; a group of zeros passes it.  Gaussian data fails it in about 1 % of the groups.
// e_max and e_min are the largest and the smallest exponent field among the non-zero elements.
__device__ __forceinline__ void rht_exponent_range(const uint32_t (&w)[8], int &emax, int &emin, bool &all_zero)
{
    const ushort2v one = {1, 1};
    ushort2v mx = {0, 0}, mn = {0xFFFF, 0xFFFF};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const ushort2v a = __builtin_bit_cast(ushort2v, w[i]) << one;          // sign dropped: exponent in bits 15..8
        mx = __builtin_elementwise_max(mx, a);
        mn = __builtin_elementwise_min(mn, a - one);                            // zeros wrap to 0xFFFF and never win
    }
    const uint32_t hmax = max((uint32_t)mx.x, (uint32_t)mx.y), hmin = min((uint32_t)mn.x, (uint32_t)mn.y) + 1u;
    emax = (int)(hmax >> 8);
    emin = max((int)(hmin >> 8), 1);
    all_zero = hmax == 0u;
}
__device__ __forceinline__ bool rht_fp32_is_exact(const uint32_t (&w)[8])
{
    int emax, emin;
    bool all_zero;
    rht_exponent_range(w, emax, emin, all_zero);
    return all_zero | (emax >= 40 && emax <= 240 && emax - emin <= 12);
}

// The fp32 sums are taken on the matrix pipes.  v_mfma_f32_4x4x4_16B_bf16 multiplies, for each group of four
// lanes, a 4x4 matrix A (lane i of the group supplies row i) by a 4x4 matrix B (lane j supplies column j, four bf16
// in two registers) and adds a 4x4 fp32 matrix whose column j lane j holds: a lane's own four values go in, its own
// four sums come out, nothing crosses lanes but the constant A.  H16 = H4 (x) H4, so with the group's sixteen values
// x[4 g + k] and output index 4 a + b,   y[4 a + b] = sum_g sum_k ( (1/4) H4[a][g] H4[b][k] s[4 g + k] ) x[4 g + k]:
// sixteen instructions (four accumulating chains of four), A = +-(1/4) H4 diag(s) for k-group g.  The products
// (+-1/4 times a bf16 number) are exact and the sums are the ones the test above covers.  A sum of zero terms and a
// sum that cancels come out as +0, as in the fp64 form.
struct RhtRows {
    uint32_t pos[4][2], neg[4][2];      // row (lane % 4) of (1/4) H4 diag(s_4g .. s_4g+3), and of its negative, as bf16 pairs
};
__device__ __forceinline__ RhtRows rht_rows(uint32_t sign_mask, uint32_t lane)
{
    RhtRows h;
    const uint32_t b0 = lane & 1u, b1 = (lane >> 1) & 1u;                 // H4[b][k] = (-1)^popcount(b & k)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const uint32_t s = sign_mask >> (4 * g);
        const uint32_t n0 = s & 1u, n1 = (b0 ^ (s >> 1)) & 1u, n2 = (b1 ^ (s >> 2)) & 1u, n3 = (b0 ^ b1 ^ (s >> 3)) & 1u;
        h.pos[g][0] = 0x3E803E80u ^ (n0 << 15) ^ (n1 << 31);              // 0x3E80: 1/4 in bf16
        h.pos[g][1] = 0x3E803E80u ^ (n2 << 15) ^ (n3 << 31);
        h.neg[g][0] = h.pos[g][0] ^ 0x80008000u;
        h.neg[g][1] = h.pos[g][1] ^ 0x80008000u;
    }
    return h;
}
// (no branch around this function may diverge within a wave: matrix instructions are issued for the whole wave)
__device__ __forceinline__ void rht_block16_mfma(const uint32_t (&w)[8], const RhtRows &h, float (&y)[16])
{
    float4v acc[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) acc[a] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const uint2v bw = {w[2 * g], w[2 * g + 1]};
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const bool minus = ((a & g) == 1) | ((a & g) == 2);            // H4[a][g] = -1
            const uint2v aw = {minus ? h.neg[g][0] : h.pos[g][0], minus ? h.neg[g][1] : h.pos[g][1]};
            acc[a] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(short4v, aw), __builtin_bit_cast(short4v, bw),
                                                            acc[a], 0, 0, 0);
        }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) y[4 * a + i] = acc[a][i];
}
__device__ __forceinline__ void pack16(const float (&y)[16], uint32_t (&w)[8])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = pack_bf16x2(y[2 * i], y[2 * i + 1]);
}

// Groups that span up to 25 binades: the elements within 12 binades of the largest and the smaller ones are
// transformed separately (each set passes the test above on its own), which gives the exact result as the sum of
// two fp32 numbers L + S.  fl(L + S) lies within half an fp32 ulp of it, and nearest-even rounding to bf16 is
// constant between consecutive bf16 midpoints, which are fp32 numbers: the two round alike unless fl(L + S) is
// itself such a midpoint (low sixteen bits 0x8000).  Returns false, and leaves w as it was, for a group it cannot
// settle this way (a wider span, the ends of the exponent range, a sum on a midpoint): those take the fp64 form.
__device__ __forceinline__ bool rht_block16_mfma_split(uint32_t (&w)[8], const RhtRows &h)
{
    int emax, emin;
    bool all_zero;
    rht_exponent_range(w, emax, emin, all_zero);
    const bool in_range = emax >= 40 && emax <= 240 && emax - emin <= 25;
    const uint32_t t = ((uint32_t)max(emax - 12, 1) << 8) - 1u;           // keep halves whose (bits << 1) exceed this
    const ushort2v thr = {(unsigned short)t, (unsigned short)t}, one = {1, 1}, ones = {0xFFFF, 0xFFFF};
    uint32_t big[8], small[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const ushort2v a = __builtin_bit_cast(ushort2v, w[i]) << one;
        const ushort2v keep = __builtin_elementwise_min(__builtin_elementwise_sub_sat(a, thr), one) * ones;   // 0xFFFF or 0
        big[i] = w[i] & __builtin_bit_cast(uint32_t, keep);
        small[i] = w[i] ^ big[i];
    }
    float L[16], S[16];
    rht_block16_mfma(big, h, L);
    rht_block16_mfma(small, h, S);
    uint32_t r[8], hit = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float y0 = L[2 * i] + S[2 * i], y1 = L[2 * i + 1] + S[2 * i + 1];
        const uint32_t low = __builtin_amdgcn_perm(__float_as_uint(y1), __float_as_uint(y0), 0x05040100u) ^ 0x80008000u;
        hit = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(ushort2v, hit), __builtin_bit_cast(ushort2v, low)));
        r[i] = pack_bf16x2(y0, y1);
    }
    const bool ok = in_range & ((hit & 0xFFFFu) != 0u) & ((hit >> 16) != 0u);
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = ok ? r[i] : w[i];
    return ok;
}

// global scale from the tensor's largest |bf16| pattern: RN_fp32(amax / 2688), 1 if zero
__device__ __forceinline__ float global_scale_from_amax_bits(uint32_t amax_bits16)
{
    float amax = __uint_as_float(amax_bits16 << 16);
    // IEEE division; 2688 = 448 * 6
    return amax_bits16 == 0u ? 1.0f : __fdiv_rn(amax, kFp8Max * kFp4Max);
}

}  // namespace nvfp4
