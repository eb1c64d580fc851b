// Device helpers shared by all kernel families: gradient widening, code fields, the
// Philox4x32-10 counter-based generator and the stochastic-rounding decision of eq. (3).
// Compiled with -ffp-contract=off: every fused multiply-add below is written explicitly.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plan.h"

namespace conef {

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

__device__ __forceinline__ float load_grad(const void *g, int dtype, int64_t idx)
{
    if (dtype == 0) return reinterpret_cast<const float *>(g)[idx];
    return bf16_bits_to_f32(reinterpret_cast<const uint16_t *>(g)[idx]);
}

// Signed b-bit field number e (0-based, LSB first) of a code word.
__device__ __forceinline__ int code_field(uint32_t w, int e, int bits)
{
    return (int)(w << (32 - bits * (e + 1))) >> (32 - bits);
}

// signed 4-bit field in the low nibble of byte `byte` of w, divided by 16 (exact), as fp32: the
// conversion instruction reads the nibble through its byte selector, so no shift or mask is spent
template <int byte>
__device__ __forceinline__ float nibble_over_16(uint32_t w)
{
    float r;
    if constexpr (byte == 0) asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0" : "=v"(r) : "v"(w));
    else if constexpr (byte == 1) asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1" : "=v"(r) : "v"(w));
    else if constexpr (byte == 2) asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2" : "=v"(r) : "v"(w));
    else asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3" : "=v"(r) : "v"(w));
    return r;
}

// the eight fields of a code word, each divided by 16
__device__ __forceinline__ void fields_over_16(uint32_t w, float q[8])
{
    const uint32_t w4 = w >> 4;
    q[0] = nibble_over_16<0>(w); q[1] = nibble_over_16<0>(w4);
    q[2] = nibble_over_16<1>(w); q[3] = nibble_over_16<1>(w4);
    q[4] = nibble_over_16<2>(w); q[5] = nibble_over_16<2>(w4);
    q[6] = nibble_over_16<3>(w); q[7] = nibble_over_16<3>(w4);
}

__device__ __forceinline__ float inv_levels(int bits)
{
    // fl32(1/s) for s = 2^(b-1)-1: 1, 1/7, 1/127
    return bits == 2 ? 1.0f : (bits == 4 ? 0.142857149243354797363281250f : 0.007874015718698501586914062500f);
}

// a ^ b ^ c in one instruction (v_bitop3_b32 with the parity truth table)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// signed byte `byte` of w as fp32: one conversion, which reads the byte through its selector
template <int byte>
__device__ __forceinline__ float signed_byte(uint32_t w)
{
    return (float)(int)(int8_t)(w >> (8 * byte));
}

// What code_values leaves in a field's value: the caller's step size takes its inverse.  (inv_levels * field_unit is a
// constant, and scaling by a power of two is exact as long as step * field_unit is a normal number, that is for scales of
// 7.6e-37 (2-bit codes), 1.4e-36 (4-bit) and 1.5e-36 (8-bit) and more.  The fields of blocks below 1.9e-34 are zero, see
// levels_over.)
__device__ __forceinline__ constexpr float field_unit(int bits) { return bits == 8 ? 1.0f : (bits == 4 ? 1.0f / 16.0f : 1.0f / 64.0f); }

// The eight fields of an octet (8-bit codes: c0 elements 0..3, c1 elements 4..7; else all in c0, bits beyond the octet zero) as fp32, over field_unit.
// Narrow fields are moved to the top of a byte, four at a time, and converted as signed bytes: 11 instructions for 4-bit
// fields and 14 for 2-bit ones (16 to extract and convert each; 17 through the conversion of nibbles, whose sixteenths would
// have to be multiplied back, since the factor 16 in the step size overflows for scales above 1.5e38).
// NIBBLES: 4-bit fields through that conversion, the same values: for kernels at their limit of registers, where the two
// shifted and masked copies of the word cost more than the instructions (octet_device.h, Q+ pass).
template <int BITS, bool NIBBLES = false>
__device__ __forceinline__ void code_values(uint32_t c0, uint32_t c1, float q[8])
{
    static_assert(!NIBBLES || BITS == 4, "4-bit fields only");
    auto bytes = [](uint32_t v, float &a, float &b, float &c, float &d) {
        a = signed_byte<0>(v); b = signed_byte<1>(v); c = signed_byte<2>(v); d = signed_byte<3>(v);
    };
    if constexpr (NIBBLES) {
        fields_over_16(c0, q);
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] *= 256.0f;
    } else if constexpr (BITS == 8) {
        bytes(c0, q[0], q[1], q[2], q[3]);
        bytes(c1, q[4], q[5], q[6], q[7]);
    } else if constexpr (BITS == 4) {
        bytes((c0 << 4) & 0xF0F0F0F0u, q[0], q[2], q[4], q[6]);
        bytes(c0 & 0xF0F0F0F0u, q[1], q[3], q[5], q[7]);
    } else {
        bytes(((c0 << 6) | (c0 << 20)) & 0xC0C0C0C0u, q[0], q[4], q[1], q[5]);
        bytes(((c0 << 2) | (c0 << 16)) & 0xC0C0C0C0u, q[2], q[6], q[3], q[7]);
    }
}

// Philox4x32-10 (Salmon et al., SC'11): 10 rounds of two 32x32->64 multiplies and xors.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4])
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// First coordinate of the block the random-block gradient compressor keeps of a matrix of N elements
// (k of them) at a step: floor(r (N - k + 1) / 2^64) with r the first 64 bits of the Philox call with counter
// (matrix, ~0, step), which no element draw uses (their second word is a matrix index).
__device__ __forceinline__ int64_t random_block_start(uint32_t mat, uint32_t step_lo, uint32_t step_hi, uint32_t seed_lo,
                                                      uint32_t seed_hi, int64_t N, int64_t k)
{
    uint32_t out[4];
    philox4x32_10(mat, 0xFFFFFFFFu, step_lo, step_hi, seed_lo, seed_hi, out);
    const uint64_t r = (uint64_t)out[0] | ((uint64_t)out[1] << 32);
    return (int64_t)__umul64hi(r, (uint64_t)(N - k + 1));
}

// The same for the block that the first error compressor of Algorithm 3, version 2, keeps (ke coordinates): counter
// (matrix, ~0 - 1, step), which neither the gradient compressor's block nor an element draw uses.
__device__ __forceinline__ int64_t i2_block_start(uint32_t mat, uint32_t step_lo, uint32_t step_hi, uint32_t seed_lo,
                                                  uint32_t seed_hi, int64_t N, int64_t ke)
{
    uint32_t out[4];
    philox4x32_10(mat, 0xFFFFFFFEu, step_lo, step_hi, seed_lo, seed_hi, out);
    const uint64_t r = (uint64_t)out[0] | ((uint64_t)out[1] << 32);
    return (int64_t)__umul64hi(r, (uint64_t)(N - ke + 1));
}

// Random-k gradient compressor, stratified: the flat index range of a matrix is cut into strata of g consecutive
// coordinates (the last one may be shorter) and one coordinate of every stratum is kept:
//   stratum i keeps  i g + floor(u_i len_i / 2^32),  len_i = min(g, N - i g),
//   u_i = word i % 4 of the Philox call with counter (i / 4, matrix + 2^30, step), which no other draw uses.
// N < 2^32.  strata_kept_octet looks at the 8 consecutive coordinates j0 .. j0 + 7 (those below N): bit e of the
// result is set if j0 + e is kept; the kept ones belong to consecutive strata, the first of which is *first.
__device__ __forceinline__ uint32_t stratum_of(uint32_t j, uint32_t g, uint64_t magic)
{
    return g == 1 ? j : (uint32_t)__umul64hi((uint64_t)j, magic);
}

__device__ __forceinline__ uint32_t strata_kept_octet(uint32_t j0, uint32_t N, uint32_t g, uint64_t magic, uint32_t mat,
                                                      uint32_t step_lo, uint32_t step_hi, uint32_t seed_lo, uint32_t seed_hi,
                                                      uint32_t *first)
{
    const uint32_t ia = stratum_of(j0, g, magic), ib = stratum_of(N - 1u - j0 < 7u ? N - 1u : j0 + 7u, g, magic);
    uint32_t bits = 0, first_i = 0, cached = 0xFFFFFFFFu;
    uint32_t out[4] = {0u, 0u, 0u, 0u};
    for (uint32_t i = ia; i <= ib; ++i) {
        if ((i >> 2) != cached) {
            cached = i >> 2;
            philox4x32_10(cached, mat + 0x40000000u, step_lo, step_hi, seed_lo, seed_hi, out);
        }
        const uint32_t w = i & 3u;
        const uint32_t u = w == 0 ? out[0] : (w == 1 ? out[1] : (w == 2 ? out[2] : out[3]));
        const uint32_t base = i * g;
        const uint32_t len = N - base < g ? N - base : g;
        const uint32_t rel = base + __umulhi(u, len) - j0;       // wraps to a large value if the kept one lies before j0
        if (rel < 8u) {
            if (bits == 0) first_i = i;
            bits |= 1u << rel;
        }
    }
    *first = first_i;
    return bits;
}

// Random-k gradient compressor as a uniformly drawn k-subset: a keyed bijection pi of [0, N) per matrix and step;
// coordinate j is kept iff pi(j) < k, and its value goes to slot pi(j) of the message.  pi: six alternating Feistel
// rounds on Z_a x Z_b (a = ceil(sqrt(N)), b = ceil(N / a)), walked again while the result is >= N:
//   (L, R) = (x / b, x mod b);  even round i: L = (L + floor(mix(R ^ key_i) a / 2^32)) mod a;
//   odd round i: R = (R + floor(mix(L ^ key_i) b / 2^32)) mod b;  pi_once(x) = L b + R
// keys 0..3: the Philox call with counter (matrix, ~0 - 2, step), keys 4..5: words 0..1 of the call with ~0 - 3 there.
struct RkuKeys {
    uint32_t k[6];
};

__device__ __forceinline__ RkuKeys rku_keys(uint32_t mat, uint32_t step_lo, uint32_t step_hi, uint32_t seed_lo, uint32_t seed_hi)
{
    uint32_t o0[4], o1[4];
    philox4x32_10(mat, 0xFFFFFFFDu, step_lo, step_hi, seed_lo, seed_hi, o0);
    philox4x32_10(mat, 0xFFFFFFFCu, step_lo, step_hi, seed_lo, seed_hi, o1);
    RkuKeys r;
    r.k[0] = o0[0]; r.k[1] = o0[1]; r.k[2] = o0[2]; r.k[3] = o0[3]; r.k[4] = o1[0]; r.k[5] = o1[1];
    return r;
}

__device__ __forceinline__ uint32_t rku_mix(uint32_t u)
{
    u *= 0x9E3779B1u; u ^= u >> 15; u *= 0x85EBCA77u; u ^= u >> 13;
    return u;
}

// magic_b = floor(2^64 / b) + 1: x / b = mulhi64(x, magic_b) for every x < 2^32 (see stratum_of)
// The walk leaves [0, N) at most a b - N times before it comes back (a bijection of [0, a b)): the loop is bounded by that.
__device__ __forceinline__ uint32_t rku_perm(uint32_t x, uint32_t N, uint32_t a, uint32_t b, uint64_t magic_b, const RkuKeys &key)
{
    uint32_t outside = a * b - N;          // modulo 2^32, also right for a b = 2^32
    do {
        uint32_t L = b == 1 ? x : (uint32_t)__umul64hi((uint64_t)x, magic_b);
        uint32_t R = x - L * b;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            if ((i & 1) == 0) {
                L += __umulhi(rku_mix(R ^ key.k[i]), a);
                L = L >= a ? L - a : L;
            } else {
                R += __umulhi(rku_mix(L ^ key.k[i]), b);
                R = R >= b ? R - b : R;
            }
        }
        x = L * b + R;
    } while (x >= N && outside-- > 0);
    return x;
}

// The same question for one coordinate j: is it the kept one of its stratum (*stratum)?
__device__ __forceinline__ bool strata_kept(uint32_t j, uint32_t N, uint32_t g, uint64_t magic, uint32_t mat, uint32_t step_lo,
                                            uint32_t step_hi, uint32_t seed_lo, uint32_t seed_hi, uint32_t *stratum)
{
    const uint32_t i = stratum_of(j, g, magic);
    uint32_t out[4];
    philox4x32_10(i >> 2, mat + 0x40000000u, step_lo, step_hi, seed_lo, seed_hi, out);
    const uint32_t w = i & 3u;
    const uint32_t u = w == 0 ? out[0] : (w == 1 ? out[1] : (w == 2 ? out[2] : out[3]));
    const uint32_t base = i * g;
    const uint32_t len = N - base < g ? N - base : g;
    *stratum = i;
    return j == base + __umulhi(u, len);
}

// 16-bit draw of element j from the four output words of the call that covers j>>3.
__device__ __forceinline__ uint32_t draw16(const uint32_t out[4], int j_low3)
{
    const uint32_t w = out[j_low3 >> 1];
    return (j_low3 & 1) ? (w >> 16) : (w & 0xFFFFu);
}

// The factor (s / a) * 2^16 of the rounding of a block of max-norm a, and 0 where a is 0 or so small that the factor would be
// infinite (s * 2^-112: 1.9e-34 for 2-bit codes, 1.3e-33 for 4-bit, 2.4e-32 for 8-bit): the codes of such a block are zero in
// every kernel, and its scale is a.  s / a is rounded to at least 2^112 exactly for a <= s * 2^-112.
__device__ __forceinline__ float levels_over(float a, float s)
{
    return a > s * 0x1p-112f ? (s / a) * 65536.0f : 0.0f;
}

// Stochastic rounding of one value (eq. (3) with max-norm a; inv16 = (s/a) * 2^16) in 16.16
// fixed point: the truncated product plus a uniform 16-bit draw, integer part kept.  Returns
// the b-bit two's-complement field (not yet shifted into place).
__device__ __forceinline__ uint32_t quantise_field(float x, float inv16, uint32_t r16, uint32_t mask)
{
    const uint32_t U = (uint32_t)(fabsf(x) * inv16);
    const uint32_t mag = (U + r16) >> 16;
    const uint32_t sgn = (uint32_t)((int32_t)__float_as_uint(x) >> 31);     // 0 or 0xFFFFFFFF
    return ((mag ^ sgn) - sgn) & mask;      // -mag for negative x; -0.0f gives mag 0 -> field 0
}

// Fixed-point stochastic rounding of an octet (quantise_field on each of its 8 values) straight into packed
// BITS-wide two's-complement fields: 8-bit codes give two words (elements 0..3, 4..7), 4- and 2-bit codes the low
// 32 / 16 bits of w[0].  With U the truncated |x| inv16 and d the 16-bit draw, -floor((U + d) / 2^16) is
// floor((-U + 65535 - d) / 2^16): the signed product is truncated, the draws of a negative element are complemented (one
// permute makes the sign masks of two elements, one exclusive or applies them), and bits 16 and up of the sum are the code
// with its sign.  (Magnitudes, gathered sign bits and a negation of the whole word took 6 instructions more per octet with 2-
// and 4-bit codes and 10 with 8-bit ones.)  Byte 2 of the sum is the code as a signed byte, which byte permutes gather.
// t (if asked for): the sums, for rounded_values.  They are below 2^23: |x| inv16 exceeds s * 2^16 by less than 1/2.  (A value
// that is not a number converts to zero, as does one times the 0 that the factor is for an infinite block.)
template <int BITS>
__device__ __forceinline__ void quantise_octet(const float x[8], float inv16, const uint32_t rnd[4], uint32_t w[2], int32_t t[8])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // selectors 9 and 11: the sign of the second operand's and of the first operand's top byte, in all bits
        uint32_t d = rnd[i] ^ __builtin_amdgcn_perm(__float_as_uint(x[2 * i + 1]), __float_as_uint(x[2 * i]), 0x0B0B0909u);
        asm("" : "+v"(d));          // one exclusive or for both halves, which the additions select
        t[2 * i] = (int32_t)(x[2 * i] * inv16) + (int32_t)(d & 0xFFFFu);
        t[2 * i + 1] = (int32_t)(x[2 * i + 1] * inv16) + (int32_t)(d >> 16);
    }
    // __builtin_amdgcn_perm(hi, lo, sel): result byte i is byte sel_i of {hi, lo} (0..3 lo, 4..7 hi, 12: zero)
    auto low2 = [](int32_t a, int32_t b) { return __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0C0C0602u); };     // byte 0: a's, byte 1: b's
    auto high2 = [](int32_t a, int32_t b) { return __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x06020C0Cu); };    // bytes 2 and 3
    auto fields = [](uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); };                          // one v_bfi
    if (BITS == 8) {
        w[0] = low2(t[0], t[1]) | high2(t[2], t[3]);
        w[1] = low2(t[4], t[5]) | high2(t[6], t[7]);
    } else if (BITS == 4) {
        w[0] = fields(0x0F0F0F0Fu, low2(t[0], t[2]) | high2(t[4], t[6]), (low2(t[1], t[3]) | high2(t[5], t[7])) << 4);
    } else {
        w[0] = fields(0x0303u, low2(t[0], t[4]), low2(t[1], t[5]) << 2);
        w[0] = fields(0x0F0Fu, w[0], low2(t[2], t[6]) << 4);
        w[0] = fields(0x3F3Fu, w[0], low2(t[3], t[7]) << 6) & 0xFFFFu;
    }
    if (BITS != 8) w[1] = 0;
}

template <int BITS>
__device__ __forceinline__ void quantise_octet(const float x[8], float inv16, const uint32_t rnd[4], uint32_t w[2])
{
    int32_t t[8];
    quantise_octet<BITS>(x, inv16, rnd, w, t);
}

// The codes that quantise_octet has just packed, as fp32 (code_values of them, without unpacking; not over field_unit)
__device__ __forceinline__ void rounded_values(const int32_t t[8], float q[8])
{
#pragma unroll
    for (int e = 0; e < 8; ++e) q[e] = signed_byte<2>((uint32_t)t[e]);
}

// Bit e: the sign bit of x[e].  Byte permutes make the signs of four values the bytes of a word, all ones or zero, each keeps its
// own bit, and the bytes are added up: 8 instructions for the octet (20 with a shift, a mask and an or per value).
__device__ __forceinline__ uint32_t octet_signs(const float x[8])
{
    uint32_t bits = 0;
#pragma unroll
    for (int i = 0; i < 8; i += 4) {
        // selectors 9 and 11: the sign of the second operand's and of the first operand's top byte, 12: zero
        const uint32_t lo = __builtin_amdgcn_perm(__float_as_uint(x[i + 1]), __float_as_uint(x[i]), 0x0C0C0B09u);
        const uint32_t hi = __builtin_amdgcn_perm(__float_as_uint(x[i + 3]), __float_as_uint(x[i + 2]), 0x0B090C0Cu);
        bits = __builtin_amdgcn_sad_u8((lo | hi) & (0x08040201u << i), 0u, bits);
    }
    return bits;
}

// LDS of a wave's own: its instructions are executed in order, so what is needed between one lane's write and another lane's
// read is that the compiler keeps their order.  The fences name LDS alone: a fence of all memory (an asm statement's memory
// clobber) also kept the loads of the next rows behind it, and the strip P pass on the sketch took twice as long (200000 x
// 300, rank 4: 189 against 92 us).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// The same with all memory kept in order: where loads that move across it do harm (random-k with two vectors, 1.3 G elements:
// 1778 us, 1805 with the fences of LDS).
__device__ __forceinline__ void wave_memory_sync()
{
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// max(a, |x[0]|, .. |x[7]|) for a >= 0; a value that is not a number does not count.  Written out because the compiler puts
// an instruction per value in front to quiet signalling ones, which none of the callers has, where it does not see x computed.
__device__ __forceinline__ float abs_max_octet(float a, const float x[8])
{
#pragma unroll
    for (int e = 0; e < 8; e += 2) asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(a) : "v"(x[e]), "v"(x[e + 1]));
    return a;
}

// max over the 2^lb_shift lanes of a scale block (aligned group of lanes), of values that are neither negative nor NaN: their
// bit patterns order as they do, and an integer maximum takes the lane permutation into the instruction, where the
// floating-point one needs a move and a quieting of its own.  Across rows of 16 lanes: the row swaps, without the LDS.
__device__ __forceinline__ float block_max(float a, int lb_shift)
{
    auto larger = [](uint32_t x, uint32_t y) { return x > y ? x : y; };
    uint32_t m = __float_as_uint(a);
    // quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E, row_half_mirror = 0x141, row_mirror = 0x140
    if (lb_shift >= 1) m = larger(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, true));
    if (lb_shift >= 2) m = larger(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, true));
    if (lb_shift >= 3) m = larger(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xF, 0xF, true));
    if (lb_shift >= 4) m = larger(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x140, 0xF, 0xF, true));
    if (lb_shift >= 5) {
        const auto p = __builtin_amdgcn_permlane16_swap(m, m, false, false);       // {rows 0 0 2 2, rows 1 1 3 3}
        m = larger(p[0], p[1]);
    }
    if (lb_shift >= 6) {
        const auto p = __builtin_amdgcn_permlane32_swap(m, m, false, false);
        m = larger(p[0], p[1]);
    }
    return __uint_as_float(m);
}

// Workgroups are dealt to the eight XCDs (each with its own L2) in turn: workgroup b runs on XCD
// b % 8.  This maps the grid onto work items so that every XCD takes a contiguous range of the
// item table: workgroups that are resident together on an XCD then work on neighbouring items
// and find the cache lines they share (code and scale lines that span several column blocks,
// operand tables of their matrix) in that XCD's L2.
__device__ __forceinline__ int xcd_contiguous_item(int b, int n_items)
{
    const int x = b & 7, j = b >> 3;
    const int q = n_items >> 3, rem = n_items & 7;
    return x * q + (x < rem ? x : rem) + j;
}

// Operand splits of Q+ for the matrix-core err pass: entry (k, c) of Q+ written as three bf16 parts
// (x = hi + mid + lo by truncation) in tile order [column block of 128][split][k % 8][(k / 8) % 16][32].
__device__ __forceinline__ void mfma_store_q_split(const MatDesc &d, double *ws, int k, int c, float x)
{
    const uint32_t xb = __float_as_uint(x);
    const float h = __uint_as_float(xb & 0xFFFF0000u);
    const float r1 = x - h;
    const float m = __uint_as_float(__float_as_uint(r1) & 0xFFFF0000u);
    const float l = r1 - m;
    uint16_t *o = reinterpret_cast<uint16_t *>(ws + d.qs_off) + (int64_t)(k >> 7) * (3 * 128 * 32) +
                  ((k & 7) * 16 + ((k >> 3) & 15)) * 32 + c;
    o[0 * 128 * 32] = (uint16_t)(xb >> 16);
    o[1 * 128 * 32] = (uint16_t)(__float_as_uint(m) >> 16);
    o[2 * 128 * 32] = (uint16_t)(__float_as_uint(l) >> 16);
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

}  // namespace conef
