// Device code of the octet family's three passes (see kernels_octet.hip), for its own launches and for those that carry the
// strip kernels' workgroups too (kernels_mixed.hip).
#pragma once
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace conef {

namespace {

// ------------------------------------------------------------------ octet load / decode
template <bool BF16, int BITS>
struct RawOctet {
    uint4 g0, g1;        // gradient bits (g1 only for fp32)
    uint32_t c0, c1;     // code bits: 8-bit: two words; 4-bit: c0; 2-bit: low 16 bits of c0, the others zero
    float scale;
};

// Loads one octet with its code bits and block scale; `o` must be an octet of the matrix (callers
// clamp and mask instead of loading behind a condition: a conditional load costs a branch and makes
// the waits on it conservative).
template <bool BF16, int BITS>
__device__ __forceinline__ RawOctet<BF16, BITS> load_octet_always(const MatDesc &d, const void *__restrict__ grads,
                                                                  const uint32_t *codes, const float *scales, int64_t o)
{
    RawOctet<BF16, BITS> r;
    r.g1 = make_uint4(0, 0, 0, 0); r.c1 = 0;
    if (BF16) {
        r.g0 = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(grads) + d.grad_off + o * 8);
    } else {
        const uint4 *gp = reinterpret_cast<const uint4 *>(reinterpret_cast<const float *>(grads) + d.grad_off + o * 8);
        r.g0 = gp[0];
        r.g1 = gp[1];
    }
    if (BITS == 8) {
        const uint2 c = *reinterpret_cast<const uint2 *>(codes + d.word_off + o * 2);
        r.c0 = c.x; r.c1 = c.y;
    } else if (BITS == 4) {
        r.c0 = codes[d.word_off + o];
    } else {
        r.c0 = reinterpret_cast<const uint16_t *>(codes + d.word_off)[o];
    }
    r.scale = scales[d.scale_off + (o >> d.lb_shift)];
    return r;
}

// Code bits and block scale of octet `o` of a second compressed vector laid out like the first
// (the second error vector of Algorithm 3).
template <int BITS>
struct RawCodes {
    uint32_t c0, c1;
    float scale;
};

template <int BITS>
__device__ __forceinline__ RawCodes<BITS> load_codes_always(const MatDesc &d, const uint32_t *codes, const float *scales, int64_t o)
{
    RawCodes<BITS> r;
    r.c1 = 0;
    if (BITS == 8) {
        const uint2 c = *reinterpret_cast<const uint2 *>(codes + d.word_off + o * 2);
        r.c0 = c.x; r.c1 = c.y;
    } else if (BITS == 4) {
        r.c0 = codes[d.word_off + o];
    } else {
        r.c0 = reinterpret_cast<const uint16_t *>(codes + d.word_off)[o];
    }
    r.scale = scales[d.scale_off + (o >> d.lb_shift)];
    return r;
}

// The same by a 32-bit distance `rel` from an octet that starts a scale block and a code word: the addresses are scalar bases and
// 32-bit lane offsets, which the load instructions add.
template <int BITS>
struct FlatCodes {
    uint8_t *codes, *scales;
};

template <bool BF16, int BITS>
struct FlatOctets {
    const uint8_t *grads;
    FlatCodes<BITS> c;
};

template <int BITS>
__device__ __forceinline__ FlatCodes<BITS> flat_codes(const MatDesc &d, uint32_t *codes, float *scales, int64_t o)
{
    return {reinterpret_cast<uint8_t *>(codes + d.word_off) + o * BITS, reinterpret_cast<uint8_t *>(scales + d.scale_off + (o >> d.lb_shift))};
}

template <bool BF16, int BITS>
__device__ __forceinline__ FlatOctets<BF16, BITS> flat_octets(const MatDesc &d, const void *grads, uint32_t *codes, float *scales, int64_t o)
{
    return {reinterpret_cast<const uint8_t *>(grads) + (d.grad_off + o * 8) * (BF16 ? 2 : 4), flat_codes<BITS>(d, codes, scales, o)};
}

template <int BITS>
__device__ __forceinline__ RawCodes<BITS> load_codes_rel(const FlatCodes<BITS> &b, int lb_shift, uint32_t rel)
{
    RawCodes<BITS> r;
    r.c1 = 0;
    if (BITS == 8) {
        const uint2 c = *reinterpret_cast<const uint2 *>(b.codes + rel * 8);
        r.c0 = c.x; r.c1 = c.y;
    } else if (BITS == 4) {
        r.c0 = *reinterpret_cast<const uint32_t *>(b.codes + rel * 4);
    } else {
        r.c0 = *reinterpret_cast<const uint16_t *>(b.codes + rel * 2);
    }
    r.scale = *reinterpret_cast<const float *>(b.scales + (rel >> lb_shift) * 4);
    return r;
}

template <bool BF16, int BITS>
__device__ __forceinline__ RawOctet<BF16, BITS> load_octet_rel(const FlatOctets<BF16, BITS> &b, int lb_shift, uint32_t rel)
{
    RawOctet<BF16, BITS> r;
    r.g0 = *reinterpret_cast<const uint4 *>(b.grads + rel * (BF16 ? 16 : 32));
    r.g1 = BF16 ? make_uint4(0, 0, 0, 0) : *reinterpret_cast<const uint4 *>(b.grads + rel * (BF16 ? 16 : 32) + 16);
    const RawCodes<BITS> c = load_codes_rel<BITS>(b.c, lb_shift, rel);
    r.c0 = c.c0; r.c1 = c.c1; r.scale = c.scale;
    return r;
}

template <int BITS>
__device__ __forceinline__ void store_codes_rel(const FlatCodes<BITS> &b, uint32_t rel, const uint32_t w[2])
{
    if (BITS == 8) *reinterpret_cast<uint2 *>(b.codes + rel * 8) = make_uint2(w[0], w[1]);
    else if (BITS == 4) *reinterpret_cast<uint32_t *>(b.codes + rel * 4) = w[0];
    else *reinterpret_cast<uint16_t *>(b.codes + rel * 2) = (uint16_t)w[0];
}

template <int BITS>
__device__ __forceinline__ void store_scale_rel(const FlatCodes<BITS> &b, uint32_t blk, float a)
{
    *reinterpret_cast<float *>(b.scales + blk * 4) = a;
}

// p <- p + second vector (the outer fused multiply-add of Algorithm 3's accumulation)
template <int BITS>
__device__ __forceinline__ void add_codes(const RawCodes<BITS> &r, float p[8])
{
    const float step = r.scale * (inv_levels(BITS) * field_unit(BITS));
    float q[8];
    code_values<BITS>(r.c0, r.c1, q);
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = __builtin_fmaf(step, q[e], p[e]);
}

// omb: 1 - beta of the partial update in the P and Q+ passes (Algorithm 4 line 5), 1 in the err pass
template <bool BF16, int BITS, bool NIBBLES = false>
__device__ __forceinline__ void decode_octet(const RawOctet<BF16, BITS> &r, float omb, float p[8])
{
    float g[8];
    if (BF16) {
        const uint32_t w[4] = {r.g0.x, r.g0.y, r.g0.z, r.g0.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            g[2 * i] = __uint_as_float(w[i] << 16);
            g[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    } else {
        g[0] = __uint_as_float(r.g0.x); g[1] = __uint_as_float(r.g0.y); g[2] = __uint_as_float(r.g0.z);
        g[3] = __uint_as_float(r.g0.w); g[4] = __uint_as_float(r.g1.x); g[5] = __uint_as_float(r.g1.y);
        g[6] = __uint_as_float(r.g1.z); g[7] = __uint_as_float(r.g1.w);
    }
    const float step = r.scale * (inv_levels(BITS) * field_unit(BITS)) * omb;
    float q[8];
    code_values<BITS, NIBBLES>(r.c0, r.c1, q);
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = __builtin_fmaf(step, q[e], g[e]);
}

// The last octet of a matrix that ends inside it or inside its word: nothing is stored beyond the matrix's last word, and that
// one whole.
template <int BITS>
__device__ __forceinline__ void store_code_words_end(const MatDesc &d, uint32_t *codes, int64_t o, int tail, const uint32_t w[2])
{
    if (BITS == 8) {
        codes[d.word_off + o * 2] = w[0];
        if (tail > 4) codes[d.word_off + o * 2 + 1] = w[1];
    } else if (BITS == 4) {
        codes[d.word_off + o] = w[0];
    } else {
        reinterpret_cast<uint16_t *>(codes + d.word_off)[o] = (uint16_t)w[0];
        if ((o & 1) == 0) reinterpret_cast<uint16_t *>(codes + d.word_off)[o + 1] = 0;
    }
}

template <int BITS>
__device__ __forceinline__ void store_code_words(const MatDesc &d, uint32_t *codes, int64_t o, const uint32_t w[2])
{
    if (BITS == 8) *reinterpret_cast<uint2 *>(codes + d.word_off + o * 2) = make_uint2(w[0], w[1]);
    else if (BITS == 4) codes[d.word_off + o] = w[0];
    else reinterpret_cast<uint16_t *>(codes + d.word_off)[o] = (uint16_t)w[0];
}

// the code words of the neighbouring octets o (even) and o + 1 in one store
template <int BITS>
__device__ __forceinline__ void store_code_pair(const MatDesc &d, uint32_t *codes, int64_t o, const uint32_t w0[2], const uint32_t w1[2])
{
    if (BITS == 8) *reinterpret_cast<uint4 *>(codes + d.word_off + o * 2) = make_uint4(w0[0], w0[1], w1[0], w1[1]);
    else if (BITS == 4) *reinterpret_cast<uint2 *>(codes + d.word_off + o) = make_uint2(w0[0], w1[0]);
    else codes[d.word_off + (o >> 1)] = (w0[0] & 0xFFFFu) | (w1[0] << 16);
}

// One row (RP = rank floats, 8- or 16-byte aligned) of a factor matrix; zeros if !valid.
template <int RP>
__device__ __forceinline__ void load_factor_row(const float *__restrict__ F, int64_t off, bool valid, float out[RP])
{
#pragma unroll
    for (int c = 0; c < RP; ++c) out[c] = 0.0f;
    if (!valid) return;
    if (RP == 2) {
        const float2 v = *reinterpret_cast<const float2 *>(F + off);
        out[0] = v.x; out[1] = v.y;
    } else {
#pragma unroll
        for (int c4 = 0; c4 < RP / 4; ++c4) {
            const float4 v = reinterpret_cast<const float4 *>(F + off)[c4];
            out[4 * c4] = v.x; out[4 * c4 + 1] = v.y; out[4 * c4 + 2] = v.z; out[4 * c4 + 3] = v.w;
        }
    }
}

// ------------------------------------------------------------------ err pass
// TWO (improved contractive error feedback, version 1, around this compressor): p = g + e~ + q with the first
// vector in codes_first / scales_first and the second in codes / scales; the rounded residual goes back to the
// first vector and what that rounding leaves, rounded again with random numbers of its own, to the second
// (see k_rb_octet).  Both are read by the lane that overwrites them, before it does.
template <bool BF16, int BITS, int RP, bool TWO = false>
__global__ __launch_bounds__(256) void k_err_octet(KernelPlan dp, const void *__restrict__ grads, uint32_t *codes,
                                                   float *scales, const float *__restrict__ Phat,
                                                   const float *__restrict__ Qn, uint32_t step_lo, uint32_t step_hi,
                                                   uint32_t *codes_first = nullptr, float *scales_first = nullptr)
{
    const int lane = threadIdx.x & 63;
    const int item = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (item >= dp.n_err_f) return;
    const WorkItem it = dp.err_f_items[item];
    const MatDesc d = dp.mats[it.mat];
    constexpr int r = RP;                 // this family is instantiated for the exact rank
    const int lr = 1 << d.lr_shift, rw = 64 >> d.lr_shift;
    const int sub = lane >> d.lr_shift, lc = lane & (lr - 1);
    const int oc = it.a * lr + lc;
    const float s_f = (float)((1 << (BITS - 1)) - 1);

    float q[8][RP];
#pragma unroll
    for (int e = 0; e < 8; ++e) load_factor_row<RP>(Qn, d.q_off + ((int64_t)oc * 8 + e) * r, true, q[e]);

    const int row_end = it.b + it.c;
    // One row of this lane: decode, residual, block max-norm, rounding, store.
    auto process = [&](const RawOctet<BF16, BITS> &oct, const RawCodes<BITS> &oct2, const float (&ph)[RP], int row, bool valid) {
        float x[8];
        decode_octet<BF16, BITS>(oct, 1.0f, x);
        if (TWO) add_codes<BITS>(oct2, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float acc = 0.0f;
#pragma unroll
            for (int c = 0; c < RP; ++c) acc = __builtin_fmaf(ph[c], q[e][c], acc);
            x[e] = x[e] - acc;
        }
        const float a = block_max(abs_max_octet(0.0f, x), d.lb_shift);
        const float inv16 = levels_over(a, s_f);
        const int64_t o = (int64_t)row * d.m8 + oc;
        uint32_t rnd[4];
        philox4x32_10((uint32_t)o, (uint32_t)it.mat, step_lo, step_hi, dp.seed_lo, dp.seed_hi, rnd);
        uint32_t w[2];
        int32_t t[8];
        quantise_octet<BITS>(x, inv16, rnd, w, t);
        if (valid) {
            store_code_words<BITS>(d, TWO ? codes_first : codes, o, w);
            if ((lc & ((1 << d.lb_shift) - 1)) == 0) (TWO ? scales_first : scales)[d.scale_off + (o >> d.lb_shift)] = a;
        }
        if (TWO) {
            const float dnew = a * inv_levels(BITS);
            float qn[8];
            rounded_values(t, qn);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = x[e] - dnew * qn[e];
            const float a2 = block_max(abs_max_octet(0.0f, x), d.lb_shift);
            const float inv16_2 = levels_over(a2, s_f);
            philox4x32_10((uint32_t)o, (uint32_t)it.mat | 0x80000000u, step_lo, step_hi, dp.seed_lo, dp.seed_hi, rnd);
            quantise_octet<BITS>(x, inv16_2, rnd, w);
            if (valid) {
                store_code_words<BITS>(d, codes, o, w);
                if ((lc & ((1 << d.lb_shift) - 1)) == 0) scales[d.scale_off + (o >> d.lb_shift)] = a2;
            }
        }
    };
    // Rows at or beyond the end of the item re-read its last row (nothing is stored for them), so the
    // loads are unconditional.  The next row is loaded before the current one is worked on; two
    // register sets take turns, so nothing is copied from one to the other.
    auto load_row = [&](RawOctet<BF16, BITS> &oct, RawCodes<BITS> &oct2, float (&ph)[RP], int row) {
        const int rc = row < row_end ? row : row_end - 1;
        // (gradient with the first vector; in the plain step that is the only one)
        oct = load_octet_always<BF16, BITS>(d, grads, TWO ? codes_first : codes, TWO ? scales_first : scales, (int64_t)rc * d.m8 + oc);
        if (TWO) oct2 = load_codes_always<BITS>(d, codes, scales, (int64_t)rc * d.m8 + oc);
        load_factor_row<RP>(Phat, d.p_off + (int64_t)rc * r, true, ph);
    };
    RawOctet<BF16, BITS> oa, ob;
    RawCodes<BITS> oa2 = {0u, 0u, 0.0f}, ob2 = {0u, 0u, 0.0f};
    float pa[RP], pb[RP];
    int row = it.b + sub;
    load_row(oa, oa2, pa, row);
    for (int r0 = it.b; r0 < row_end; r0 += 2 * rw) {
        load_row(ob, ob2, pb, row + rw);
        process(oa, oa2, pa, row, row < row_end);
        if (r0 + rw >= row_end) break;              // uniform
        load_row(oa, oa2, pa, row + 2 * rw);
        process(ob, ob2, pb, row + rw, row + rw < row_end);
        row += 2 * rw;
    }
}

// ------------------------------------------------------------------ err pass, residual on the fp32 matrix cores
// For rank 4 and 8, blocks of at most 256 elements and columns a multiple of 128 (of 256 for blocks of 256).  In the
// kernel above the fp32 fma chain over the rank is most of the vector work (8 of ~33 instructions per element at rank 8,
// where the vector ALU and not the memory sets the pace).  v_mfma_f32_16x16x4_f32 adds its four products one after the
// other, each fused, in ascending k (see the update kernel of the kernels for any shape): started from 0 and chained
// over the rank it gives the bits of that chain, so the results stay those of the kernel above bit for bit.
//   operand layout: lane l holds A[l%16][l/16], B[l/16][l%16] and D[4(l/16) + v][l%16], v = 0..3.
// One wave per item: a strip of 128 columns (WIDE: 256, two tiles side by side, one scale block of 256) and a range
// of rows, 16 rows per trip.  Tile t (0..7) of the matrix cores takes column 8 cc + t of every octet cc = l % 16, so
// after eight tiles lane (cc, kg = l / 16) holds rows 4 kg + v, columns 8 cc .. 8 cc + 7: the octets it loads.  The
// strip's rows of Q+ stay in registers in operand order for the whole item; a trip loads 16 rows of P^ (one or two
// floats per lane).  A scale block is 2^lb_shift <= 16 lanes of one DPP row (WIDE: the row's 16 lanes, both tiles).
// WIDE: lane cc takes the neighbouring octets 2 cc and 2 cc + 1 of the strip, one per tile, so that its two gradient
// loads are adjacent, its code bits are one load and one store, and its block scale is loaded once.
// A trip's inputs have one set of registers: as soon as a row is decoded, the same row of the next trip is requested into
// its place.  (Two sets, the next trip's loads before the whole of the present one, took 40 - 60 registers more: one wave
// per SIMD less, or 60 - 150 spilled ones with two vectors on wide strips.)
// Waves per SIMD: three where three fit without spilling more than a few registers, else two; never more, which the pass
// with one vector could do on narrow strips: it is bound by memory there, and more waves are slower.  Measured, us per step,
// two sets -> one set at 2 / 3 waves: 124 M fp32 elements at rank 4, 4-bit codes: blocks of 128 368.3 -> 365.8 / 367.5
// (370.4 at 4), of 256 403 -> 368 / 386; two vectors, of 128 477 -> 464.5 / 459.1, of 256 647 -> 459 / 765.  210 M bf16 at rank 8:
// 2-bit codes, blocks of 256 390.8 -> 390.4 / 380.8; 4-bit, of 128 414.7 -> 427 / 410.9.
#define CONEF_ERR_TILE_WAVES_N(BF16, WIDE, TWO) (((BF16) ? !((WIDE) && (TWO)) : (!(WIDE) && (TWO))) ? 3 : 2)
#define CONEF_ERR_TILE_WAVES(BF16, WIDE, TWO) \
    __attribute__((amdgpu_waves_per_eu(CONEF_ERR_TILE_WAVES_N(BF16, WIDE, TWO), CONEF_ERR_TILE_WAVES_N(BF16, WIDE, TWO))))
typedef float tile_f32x4 __attribute__((ext_vector_type(4)));

// s_bq: LDS, err_tile_lds<RP, WIDE>() floats; `block`: index of the workgroup among those of this pass
template <int RP, bool WIDE>
constexpr int err_tile_lds() { return WIDE ? 4 * 2 * 8 * (RP / 4) * 64 : 1; }

template <bool BF16, int BITS, int RP, bool WIDE, bool TWO>
__device__ __forceinline__ void err_tile(const KernelPlan &dp, int block, float *s_bq, const void *__restrict__ grads, uint32_t *codes,
                                         float *scales, const float *__restrict__ Phat, const float *__restrict__ Qn,
                                         uint32_t step_lo, uint32_t step_hi, uint32_t *codes_first, float *scales_first)
{
    constexpr int NT = WIDE ? 2 : 1, NQ = RP / 4;
    const int lane = threadIdx.x & 63;
    const int item = __builtin_amdgcn_readfirstlane(block * 4 + (int)(threadIdx.x >> 6));
    if (item >= dp.n_err_t) return;
    const WorkItem it = dp.err_t_items[item];
    const MatDesc d = dp.mats[it.mat];
    const int cc = lane & 15, kg = lane >> 4;
    // the lane's octet column in tile h: octet cc of the strip, or (WIDE) the neighbours 2 cc and 2 cc + 1
    const int oc0 = it.a * 16 * NT + (WIDE ? 2 * cc : cc);
    auto oct_col = [&](int h) { return oc0 + h; };
    const int row_end = it.b + it.c;
    const float s_f = (float)((1 << (BITS - 1)) - 1);
    const int lb = WIDE ? 4 : d.lb_shift;                   // lanes of one DPP row that share a scale block

    // B operand: Q+[column 8 oct_col(h) + t][4 q + kg].  It does not change over the strip's rows: in registers, or, for
    // the wide strips, whose two tiles need the registers for a second set of inputs, in LDS of the wave's own (one entry
    // per lane and operand: conflict-free 4-byte reads, no barrier: a lane reads back what it wrote)
    float bq[NT][8][NQ];
    float *my_bq = s_bq + (WIDE ? (threadIdx.x >> 6) * (NT * 8 * NQ * 64) + lane : 0);
#pragma unroll
    for (int h = 0; h < NT; ++h)
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const float v = Qn[d.q_off + ((int64_t)oct_col(h) * 8 + t) * RP + 4 * q + kg];
                if (WIDE) my_bq[((h * 8 + t) * NQ + q) * 64] = v;
                else bq[h][t][q] = v;
            }

    struct TripIn {
        RawOctet<BF16, BITS> o[NT][4];
        RawCodes<BITS> o2[TWO ? NT : 1][TWO ? 4 : 1];
        float a[NQ];
    };
    // Rows at or beyond the end of the item re-read its last row (nothing is stored for them): unconditional loads.
    TripIn in;
    auto load_a = [&](int r0) {
        const int ar = r0 + cc < row_end ? r0 + cc : row_end - 1;
#pragma unroll
        for (int q = 0; q < NQ; ++q) in.a[q] = Phat[d.p_off + (int64_t)ar * RP + 4 * q + kg];
    };
    auto load_row = [&](int r0, int v) {
        const int row = r0 + 4 * kg + v < row_end ? r0 + 4 * kg + v : row_end - 1;
        if (WIDE) {
            // both octets at once: o is even
            const int64_t o = (int64_t)row * d.m8 + oc0;
            const uint32_t *cw = (TWO ? codes_first : codes) + d.word_off;
            RawOctet<BF16, BITS> &a0 = in.o[0][v], &a1 = in.o[NT - 1][v];
            a0.g1 = a1.g1 = make_uint4(0, 0, 0, 0); a0.c1 = a1.c1 = 0;
            if (BF16) {
                const uint4 *gp = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(grads) + d.grad_off + o * 8);
                a0.g0 = gp[0]; a1.g0 = gp[1];
            } else {
                const uint4 *gp = reinterpret_cast<const uint4 *>(reinterpret_cast<const float *>(grads) + d.grad_off + o * 8);
                a0.g0 = gp[0]; a0.g1 = gp[1]; a1.g0 = gp[2]; a1.g1 = gp[3];
            }
            if (BITS == 8) {
                const uint4 c = *reinterpret_cast<const uint4 *>(cw + o * 2);
                a0.c0 = c.x; a0.c1 = c.y; a1.c0 = c.z; a1.c1 = c.w;
            } else if (BITS == 4) {
                const uint2 c = *reinterpret_cast<const uint2 *>(cw + o);
                a0.c0 = c.x; a1.c0 = c.y;
            } else {
                const uint32_t c = cw[o >> 1];          // the fields of the first octet are the low half
                a0.c0 = c & 0xFFFFu; a1.c0 = c >> 16;
            }
            a0.scale = a1.scale = (TWO ? scales_first : scales)[d.scale_off + (o >> d.lb_shift)];
            if (TWO) {
#pragma unroll
                for (int h = 0; h < NT; ++h) in.o2[TWO ? h : 0][TWO ? v : 0] = load_codes_always<BITS>(d, codes, scales, o + h);
            }
        } else {
            const int64_t o = (int64_t)row * d.m8 + oc0;
            in.o[0][v] = load_octet_always<BF16, BITS>(d, grads, TWO ? codes_first : codes, TWO ? scales_first : scales, o);
            if (TWO) in.o2[0][TWO ? v : 0] = load_codes_always<BITS>(d, codes, scales, o);
        }
    };
    auto process = [&](int r0) {
        tile_f32x4 acc[NT][8];
#pragma unroll
        for (int h = 0; h < NT; ++h)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                acc[h][t] = tile_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    acc[h][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(in.a[q], WIDE ? my_bq[((h * 8 + t) * NQ + q) * 64] : bq[h][t][q],
                                                                     acc[h][t], 0, 0, 0);
            }
        load_a(r0 + 16);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = r0 + 4 * kg + v;
            const bool valid = row < row_end;
            const int rowc = valid ? row : row_end - 1;
            float x[NT][8];
            float a = 0.0f;
#pragma unroll
            for (int h = 0; h < NT; ++h) {
                decode_octet<BF16, BITS>(in.o[h][v], 1.0f, x[h]);
                if (TWO) add_codes<BITS>(in.o2[TWO ? h : 0][TWO ? v : 0], x[h]);
#pragma unroll
                for (int e = 0; e < 8; ++e) x[h][e] = x[h][e] - acc[h][e][v];
                a = abs_max_octet(a, x[h]);
            }
            load_row(r0 + 16, v);
            a = block_max(a, lb);
            const float inv16 = levels_over(a, s_f);
            const float dnew = a * inv_levels(BITS);
            float a2 = 0.0f;
            uint32_t w[NT][2];
#pragma unroll
            for (int h = 0; h < NT; ++h) {
                const int64_t o = (int64_t)rowc * d.m8 + oct_col(h);
                uint32_t rnd[4];
                philox4x32_10((uint32_t)o, (uint32_t)it.mat, step_lo, step_hi, dp.seed_lo, dp.seed_hi, rnd);
                int32_t tq[8];
                quantise_octet<BITS>(x[h], inv16, rnd, w[h], tq);
                if (valid) {
                    if (!WIDE) store_code_words<BITS>(d, TWO ? codes_first : codes, o, w[h]);
                    if (h == 0 && (cc & ((1 << lb) - 1)) == 0) (TWO ? scales_first : scales)[d.scale_off + (o >> d.lb_shift)] = a;
                }
                if (TWO) {
                    float qn[8];
                    rounded_values(tq, qn);
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[h][e] = x[h][e] - dnew * qn[e];
                    a2 = abs_max_octet(a2, x[h]);
                }
            }
            if (WIDE && valid) store_code_pair<BITS>(d, TWO ? codes_first : codes, (int64_t)rowc * d.m8 + oc0, w[0], w[NT - 1]);
            if (TWO) {
                a2 = block_max(a2, lb);
                const float inv16_2 = levels_over(a2, s_f);
#pragma unroll
                for (int h = 0; h < NT; ++h) {
                    const int64_t o = (int64_t)rowc * d.m8 + oct_col(h);
                    uint32_t rnd[4];
                    philox4x32_10((uint32_t)o, (uint32_t)it.mat | 0x80000000u, step_lo, step_hi, dp.seed_lo, dp.seed_hi, rnd);
                    quantise_octet<BITS>(x[h], inv16_2, rnd, w[h]);
                    if (valid) {
                        store_code_words<BITS>(d, codes, o, w[h]);
                        if (h == 0 && (cc & ((1 << lb) - 1)) == 0) scales[d.scale_off + (o >> d.lb_shift)] = a2;
                    }
                }
            }
        }
    };
    // as soon as a row of a trip is decoded, the same row of the next trip is requested into its registers
    load_a(it.b);
#pragma unroll
    for (int v = 0; v < 4; ++v) load_row(it.b, v);
    for (int r0 = it.b; r0 < row_end; r0 += 16) process(r0);
}

// ------------------------------------------------------------------ Q+ pass
// Q+ = p^T P^ on the fp64 matrix cores (v_mfma_f64_4x4x4_4b_f64, operand layout at the P pass below):
// D[k][c] += sum_i A[k][i] B[i][c] with A[k][i] = p[row i][column k] and B[i][c] = P^[row i][c]; the four
// blocks are four groups of four columns that share B; four rows per instruction, fp64 sums throughout.
// One wave per (64 columns, row tile), independent of the other waves.  Rows are walked 32 at a
// time: octets are decoded in the coalesced load layout (8 lanes per row) into a wave-private LDS
// tile (32 rows x 64 columns of p), read back one value per lane and instruction; the rows of P^
// are converted from fp32.  Loads run one step ahead.  Partial sums per row tile go to the workspace.
// 4-bit codes of one vector are decoded by nibbles, except with bf16 gradients at rank 8: by bytes, these forms of the kernel
// spill up to 19 registers (41 M elements, bytes / nibbles: fp32 at rank 8 74 / 57 us, rank 4 39 / 39, bf16 at ranks 2 and 4
// 35 / 30 and 36 / 31; at rank 8 41 / 44).
// Occupancy target (measured): four waves per SIMD with bf16 gradients (a few spilled registers cost less
// than the fourth wave brings), three with fp32 gradients, whose octets take twice the registers.
constexpr int kQTileCols = 64;
constexpr int kQTilePitch = 80;     // floats per LDS tile row: rows 0..3 of a group fall on distinct banks
constexpr int kQStepRows = 32;

#define CONEF_Q_OCTET_WAVES(BF16, TWO) __attribute__((amdgpu_waves_per_eu((BF16 ? 4 : 3) - (TWO ? 1 : 0), (BF16 ? 4 : 3) - (TWO ? 1 : 0))))
constexpr int kQOctetLds = 4 * kQStepRows * kQTilePitch;       // floats

// TWO: p = g + e~ + q with the plan's first error vector (dp.i_codes) decoded under the codes / scales arguments.
// JOINED (dp.q_joined): the workgroup's waves are the row tiles of one strip, and Q+ is written from there.  Rank 8: kernels of their
// own, since in one with the other form the compiler no longer loads a step ahead (114 registers instead of 168; fp32 gradients, 101 M
// elements, the pass 157 us, so 123).  Lower ranks: one kernel for both (kQJoinedAtRunTime), which costs none, and of bf16 gradients
// with 8-bit codes it spills two registers less (138 M elements a step of 291 us, in kernels of their own 297).
constexpr int kQJoinedNo = 0, kQJoinedYes = 1, kQJoinedAtRunTime = 2;
// lds: kQOctetLds floats; `block`: index of the workgroup among those of this pass
template <bool BF16, int BITS, int RH, bool TWO, int JOINED>
__device__ __forceinline__ void q_octet(const KernelPlan &dp, int block, float *lds, const void *__restrict__ grads,
                                        const uint32_t *__restrict__ codes, const float *__restrict__ scales,
                                        const float *__restrict__ Phat, double *ws, float *Qout)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool joined = JOINED == kQJoinedAtRunTime ? dp.q_joined != 0 : JOINED == kQJoinedYes;
    const int item = __builtin_amdgcn_readfirstlane(joined ? block : block * 4 + (int)(threadIdx.x >> 6));
    if (item >= dp.n_q_f) return;
    float *T = lds + wave * (kQStepRows * kQTilePitch);
    const WorkItem it = dp.q_f_items[item];
    const MatDesc d = dp.mats[it.mat];
    const int r = dp.rank;
    const int col0 = it.a * kQTileCols;
    const int64_t row0 = (int64_t)(joined ? wave : it.b) * d.q_tile_rows;
    const int64_t row1 = (row0 + d.q_tile_rows < d.n) ? row0 + d.q_tile_rows : d.n;
    const int lrow = lane >> 3, loct = lane & 7;      // load layout: 8 lanes per row, rows lrow + 8 s
    const int mi = lane & 15, mk = lane >> 4;         // matrix-core roles
    // columns at or beyond m (last strip) read the last octet of the row instead: they only feed
    // rows of D that are not stored
    const int64_t oct0 = ((col0 >> 3) + loct < d.m8) ? (col0 >> 3) + loct : d.m8 - 1;

    const int mc = lane & 3;                          // factor column of this lane's B and D entries (+ 4 h)

    double acc[4][RH];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int h = 0; h < RH; ++h) acc[t][h] = 0.0;

    constexpr int kLoads = kQStepRows / 8, kGroups = kQStepRows / 4;
    struct Step {
        RawOctet<BF16, BITS> o[kLoads];
        RawCodes<BITS> o2[TWO ? kLoads : 1];
        float ph[kGroups][RH];    // P^[i0 + 4 g + mk][mc + 4 h]
    };
    auto load_step = [&](Step &st, int64_t i0) {
#pragma unroll
        for (int s = 0; s < kLoads; ++s) {
            int64_t row = i0 + lrow + 8 * s;
            row = row < row1 ? row : row1 - 1;
            st.o[s] = load_octet_always<BF16, BITS>(d, grads, TWO ? dp.i_codes : codes, TWO ? dp.i_scales : scales, row * d.m8 + oct0);
            if (TWO) st.o2[s] = load_codes_always<BITS>(d, codes, scales, row * d.m8 + oct0);
        }
        // rows at or beyond row1 re-read the last row; their P^ operand is zero
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int64_t row = i0 + 4 * g + mk;
#pragma unroll
            for (int h = 0; h < RH; ++h) {
                const int c = mc + 4 * h;
                const float v = Phat[d.p_off + (row < row1 ? row : row1 - 1) * r + (c < r ? c : r - 1)];
                st.ph[g][h] = v * ((row < row1 && c < r) ? 1.0f : 0.0f);       // a product, not a select (see the P pass)
            }
        }
    };

    Step cur;
    // (joined: a wave may have no rows; row1 is n then, and what it loads the matrix's last row)
    if (JOINED != kQJoinedAtRunTime || row0 < row1) load_step(cur, row0);           // uniform
    for (int64_t i0 = row0; i0 < row1; i0 += kQStepRows) {
        // decode into the tile
#pragma unroll
        for (int s = 0; s < kLoads; ++s) {
            float p[8];
            decode_octet<BF16, BITS, BITS == 4 && !TWO && !(BF16 && RH == 2)>(cur.o[s], dp.omb, p);
            if (TWO) add_codes<BITS>(cur.o2[s], p);
            float4 *dst = reinterpret_cast<float4 *>(T + (lrow + 8 * s) * kQTilePitch + loct * 8);
            dst[0] = make_float4(p[0], p[1], p[2], p[3]);
            dst[1] = make_float4(p[4], p[5], p[6], p[7]);
        }
        float b[kGroups][RH];
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
#pragma unroll
            for (int h = 0; h < RH; ++h) b[g][h] = cur.ph[g][h];
        load_step(cur, i0 + kQStepRows);
        wave_lds_sync();
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double a = (double)T[(4 * g + mk) * kQTilePitch + 16 * t + mi];
#pragma unroll
                for (int h = 0; h < RH; ++h)
                    acc[t][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, (double)b[g][h], acc[t][h], 0, 0, 0);
            }
        }
        wave_lds_sync();
    }
    // D of block (lane % 16) / 4, entry [lane / 16][lane % 4]: column 16 t + 4 ((lane % 16) / 4) + lane / 16 of the strip
    const int dcol = 4 * (mi >> 2) + mk;
    if (joined) {
        // the waves' sums, added in wave order
        constexpr int RC = 4 * RH;
        double *red = reinterpret_cast<double *>(lds);            // [wave][column][RC], 16 KB of the 40 KB of tiles
        __syncthreads();                              // every wave is done with its tile
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int h = 0; h < RH; ++h) red[(wave * 64 + 16 * t + dcol) * RC + mc + 4 * h] = acc[t][h];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < RH; ++u) {
            const int e = (int)threadIdx.x + 256 * u, col = col0 + e / RC, c = e % RC;
            double sum = red[e];
#pragma unroll
            for (int w = 1; w < 4; ++w) sum += red[w * 64 * RC + e];
            if (col < d.m && c < r) Qout[d.q_off + (int64_t)col * r + c] = (float)sum;
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int col = col0 + 16 * t + dcol;
#pragma unroll
        for (int h = 0; h < RH; ++h) {
            const int c = mc + 4 * h;
            if (col < d.m && c < r) ws[d.qpart_off + ((int64_t)it.b * d.m + col) * r + c] = acc[t][h];
        }
    }
}

// ------------------------------------------------------------------ P pass
// P = p Q on the fp64 matrix cores: products of fp32 values are exact in fp64 and the sum is kept in
// fp64, as in a plain fp64 loop.  v_mfma_f64_4x4x4_4b_f64 multiplies four independent 4x4 blocks:
// block b (0..3) computes D_b[i][j] += sum_k A_b[i][k] B_b[k][j]; lane l holds A_b[i][k] for i = l % 4,
// b = (l / 4) % 4, k = l / 16, B_b[k][j] for j = l % 4 (same b, k), and D_b[i][j] for i = l / 16,
// b = (l % 16) / 4, j = l % 4.  Here the four blocks are four groups of four rows that share B
// (four columns of p times four factor columns): one instruction covers 16 rows x 4 columns of p and
// 4 factor columns; rank 8 takes two instructions (RH = 2 halves), ranks 2 and 4 one.  The
// instruction runs at the rate of the fp64 vector ALU and is not overlapped with it (measured), so
// its cost is that of r fp64 FMAs per element plus nothing for the sum across lanes.
//
// One workgroup per (64 rows, column chunk).  The chunk is walked in steps of 128 columns; in a step
// wave w takes columns 32w..32w+31 (so the four waves read whole 128-byte lines of the gradient
// between them, at the same time) and adds its products to accumulators of its own; the four sets
// are added up in wave order when the chunk is done.  A wave decodes its 64 x 32 sub-tile in the
// coalesced load layout into a wave-private LDS tile (fp32); A[i][kk] = p[row i][column 4j + kk] is
// read back one value per lane (conflict-free), B[kk][c] = Q[column 4j + kk][c] is read from Q, eight
// values per lane and sub-tile; gradient and Q loads run one step ahead.
//
// Code words and block scales go through LDS a "group" at a time: the columns whose codes fill one
// 128-byte line per row (1024 / bits columns).  Fetched 32 columns at a time, a line would be pulled
// from memory again for every piece (the L2 does not hold it that long: every workgroup streams
// through it).  The group after the current one waits in registers.
constexpr int kSubCols = 32;        // columns per wave and step
constexpr int kStepCols = 128;      // columns per workgroup and step
constexpr int kTileStride = 36;     // floats per LDS tile row: 32 columns + 4 of padding
constexpr int kCodePitch = 34;      // words per row of the code stage: 128 bytes + 8 of padding
constexpr int kScalePitch = 9;      // floats per row of the scale stage: up to 8 blocks per group + 1

constexpr int kPOctetTiles = 4 * kPTileRows * kTileStride, kPOctetCodes = kPTileRows * kCodePitch, kPOctetScales = kPTileRows * kScalePitch;
constexpr int kPOctetLds = kPOctetTiles + kPOctetCodes + kPOctetScales;         // 4-byte words, one vector

// LDS of the P pass: kPOctetTiles, kPOctetCodes and kPOctetScales words (TWO: code1 and scale1 as many for the first vector).
// The pass's own kernel has an array for each: the compiler then knows them apart (two vectors, 124 M elements: 1 % of the
// pass).
struct POctetLds {
    float *tiles;
    uint32_t *code;
    float *scale;
    uint32_t *code1;
    float *scale1;
};

// TWO: p = g + e~ + q; the plan's first error vector (dp.i_codes) is staged beside the codes / scales arguments.
// (the second stage costs LDS: two workgroups per CU instead of three)
// `block`: index of the workgroup among those of this pass
#define CONEF_P_OCTET_WAVES(TWO) __attribute__((amdgpu_waves_per_eu(TWO ? 2 : 3, TWO ? 2 : 3)))
template <bool BF16, int BITS, int RH, bool TWO>
__device__ __forceinline__ void p_octet(const KernelPlan &dp, int block, const POctetLds &lds, const void *__restrict__ grads,
                                        const uint32_t *__restrict__ codes, const float *__restrict__ scales,
                                        const float *__restrict__ Q, float *P, double *ws)
{
    constexpr int kGroupCols = 1024 / BITS;                 // 512, 256, 128
    constexpr int kGroupSteps = kGroupCols / kStepCols;     // 4, 2, 1
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    uint32_t *cstage = lds.code, *cstage1 = lds.code1;
    float *sstage = lds.scale, *sstage1 = lds.scale1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    float *T = lds.tiles + wave * (kPTileRows * kTileStride);
    const WorkItem it = dp.p_f_items[xcd_contiguous_item(block, dp.n_p_f)];
    const MatDesc d = dp.mats[it.mat];
    const int r = dp.rank;
    const int64_t row0 = it.a;
    const int c_begin = it.b * d.p_chunk_cols;
    const int c_end = chunk_end(d.m, d.p_chunk_cols, c_begin);
    const int lrow = lane >> 2, loct = lane & 3;      // load layout: 4 lanes per row, 16 rows per load
    const int mi = lane & 15, mk = lane >> 4;         // matrix-core roles
    const int lb = d.lb_shift + 3;                    // log2(block)

    const int mc = lane & 3;                          // factor column of this lane's B and D entries (+ 4 h)

    double acc[4][RH];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int h = 0; h < RH; ++h) acc[t][h] = 0.0;

    // ---- group staging: 64 rows x 128 bytes of codes (two 16-byte pieces per thread) and the scales
    // of the group's blocks (up to 8 per row, two per thread).  Rows beyond the matrix re-read its last
    // row, pieces beyond the row's end its first piece of the group (neither is used).
    struct GroupRegs {
        u32x4 c0, c1;
        float s0, s1;
    };
    const int n_sc = (kGroupCols >> lb) > 0 ? (kGroupCols >> lb) : 1;       // blocks per group and row
    auto load_group = [&](GroupRegs &gr, int gcol0, const uint32_t *codes, const float *scales) {
        const uint8_t *cbase = reinterpret_cast<const uint8_t *>(codes + d.word_off);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int idx = tid + 256 * s, rr = idx >> 3, part = idx & 7;
            const int64_t row = (row0 + rr < d.n) ? row0 + rr : d.n - 1;
            const int col = (gcol0 + part * (kGroupCols / 8) < d.m) ? gcol0 + part * (kGroupCols / 8) : gcol0;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(cbase + ((row * d.m + col) * BITS >> 3));
            if (s == 0) gr.c0 = v; else gr.c1 = v;
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int idx = tid + 256 * s, rr = idx >> 3, j = idx & 7;
            const int64_t row = (row0 + rr < d.n) ? row0 + rr : d.n - 1;
            int64_t blk = (row * d.m + gcol0) >> lb;
            blk += (j < n_sc && gcol0 + (j << lb) < d.m) ? j : 0;
            const float v = scales[d.scale_off + blk];
            if (s == 0) gr.s0 = v; else gr.s1 = v;
        }
    };
    auto store_group = [&](const GroupRegs &gr, uint32_t *cstage, float *sstage) {
        {
            const int rr = tid >> 3, part = tid & 7;
            *reinterpret_cast<u32x4 *>(cstage + rr * kCodePitch + part * 4) = gr.c0;
            *reinterpret_cast<u32x4 *>(cstage + (rr + 32) * kCodePitch + part * 4) = gr.c1;
            sstage[rr * kScalePitch + part] = gr.s0;
            sstage[(rr + 32) * kScalePitch + part] = gr.s1;
        }
    };

    // B operand of a sub-tile: Q[col0 + 4 j + mk][mc + 4 h], j = 0..7; zero beyond the rank and for
    // columns at or beyond the end of the chunk (the tile holds other data of the same rows there)
    auto load_b = [&](float (&bq)[8][RH], int col0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int col = col0 + 4 * j + mk;
#pragma unroll
            for (int h = 0; h < RH; ++h) {
                const int c = mc + 4 * h;
                // (masked by a product, not a select: a select lets the compiler move the load behind a
                // branch on the condition, where it is waited for on the spot)
                const float v = Q[d.q_off + (int64_t)(col < c_end ? col : c_end - 1) * r + (c < r ? c : r - 1)];
                bq[j][h] = v * ((col < c_end && c < r) ? 1.0f : 0.0f);
            }
        }
    };
    // gradient octets of a sub-tile.  Rows at or beyond n re-read the last row (their rows of D are
    // not stored); octets at or beyond the end of the chunk re-read its last octet (their B operand is zero)
    struct GradRegs {
        uint4 g0, g1;
    };
    const int oct_end = c_end >> 3;
    auto load_grads = [&](GradRegs (&o)[4], int col0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            int64_t row = row0 + s * 16 + lrow;
            row = row < d.n ? row : d.n - 1;
            int oc = (col0 >> 3) + loct;
            oc = oc < oct_end ? oc : oct_end - 1;
            const int64_t e = (row * d.m8 + oc) * 8;
            if (BF16) {
                o[s].g0 = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(grads) + d.grad_off + e);
                o[s].g1 = make_uint4(0, 0, 0, 0);
            } else {
                const uint4 *gp = reinterpret_cast<const uint4 *>(reinterpret_cast<const float *>(grads) + d.grad_off + e);
                o[s].g0 = gp[0];
                o[s].g1 = gp[1];
            }
        }
    };

    const int n_steps = (c_end - c_begin + kStepCols - 1) / kStepCols;
    GroupRegs gr, gr1;
    GradRegs cur[4];
    float bq[8][RH], bn[8][RH];
    load_group(gr, c_begin, codes, scales);
    if (TWO) load_group(gr1, c_begin, dp.i_codes, dp.i_scales);
    load_grads(cur, c_begin + kSubCols * wave);
    load_b(bq, c_begin + kSubCols * wave);
    for (int step = 0; step < n_steps; ++step) {
        const int col0 = c_begin + step * kStepCols + kSubCols * wave;       // this wave's sub-tile
        const int gcol0 = c_begin + (step / kGroupSteps) * kGroupCols;        // its code group
        if (step % kGroupSteps == 0) {
            __syncthreads();            // every wave is done with the previous group's stage
            store_group(gr, cstage, sstage);
            if (TWO) store_group(gr1, cstage1, sstage1);
            const int gnext = gcol0 + kGroupCols;
            load_group(gr, gnext < c_end ? gnext : gcol0, codes, scales);
            if (TWO) load_group(gr1, gnext < c_end ? gnext : gcol0, dp.i_codes, dp.i_scales);
            __syncthreads();
        }
        // decode the loaded sub-tile into the wave's LDS tile (row-major, padded)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int rr = s * 16 + lrow;
            int oc = ((col0 - gcol0) >> 3) + loct;                       // octet of the group
            oc = oc < (kGroupCols >> 3) ? oc : (kGroupCols >> 3) - 1;    // (columns beyond the chunk: unused)
            // code bits and block scale of the octet from a stage
            auto staged = [&](const uint32_t *cs, const float *ss) {
                RawCodes<BITS> k;
                k.c1 = 0;
                if (BITS == 8) {
                    const uint2 c = *reinterpret_cast<const uint2 *>(cs + rr * kCodePitch + oc * 2);
                    k.c0 = c.x; k.c1 = c.y;
                } else if (BITS == 4) {
                    k.c0 = cs[rr * kCodePitch + oc];
                } else {
                    k.c0 = reinterpret_cast<const uint16_t *>(cs + rr * kCodePitch)[oc];
                }
                k.scale = ss[rr * kScalePitch + ((oc << 3) >> lb)];
                return k;
            };
            const RawCodes<BITS> k0 = TWO ? staged(cstage1, sstage1) : staged(cstage, sstage);
            RawOctet<BF16, BITS> o;
            o.g0 = cur[s].g0; o.g1 = cur[s].g1; o.c0 = k0.c0; o.c1 = k0.c1; o.scale = k0.scale;
            float p[8];
            decode_octet<BF16, BITS>(o, dp.omb, p);
            if (TWO) add_codes<BITS>(staged(cstage, sstage), p);
            float4 *dst = reinterpret_cast<float4 *>(T + rr * kTileStride + loct * 8);
            dst[0] = make_float4(p[0], p[1], p[2], p[3]);
            dst[1] = make_float4(p[4], p[5], p[6], p[7]);
        }
        // issue the loads of this wave's next sub-tile
        load_b(bn, col0 + kStepCols);
        load_grads(cur, col0 + kStepCols);
        wave_lds_sync();
        if (col0 < c_end) {             // a ragged last step leaves the upper waves without columns
#pragma unroll
            for (int j = 0; j < 8; ++j) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const double a = (double)T[(16 * t + mi) * kTileStride + 4 * j + mk];
#pragma unroll
                    for (int h = 0; h < RH; ++h)
                        acc[t][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, (double)bq[j][h], acc[t][h], 0, 0, 0);
                }
            }
        }
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int h = 0; h < RH; ++h) bq[j][h] = bn[j][h];
    }
    // ---- the four waves' sums, added in wave order.  D of block (lane % 16) / 4, entry [lane / 16][lane % 4]:
    // row 16 t + 4 ((lane % 16) / 4) + lane / 16 of the tile, factor column lane % 4 + 4 h
    __syncthreads();
    double *red = reinterpret_cast<double *>(lds.tiles);      // [wave][row][8], 16 KB of the 36 KB of tiles
    const int drow = 4 * (mi >> 2) + mk;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int h = 0; h < RH; ++h) red[(wave * kPTileRows + 16 * t + drow) * 8 + mc + 4 * h] = acc[t][h];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int idx = tid + 256 * s, rr = idx >> 3, c = idx & 7;
        const int64_t row = row0 + rr;
        if (c < r && row < d.n) {
            double sum = red[rr * 8 + c];
#pragma unroll
            for (int w = 1; w < 4; ++w) sum += red[(w * kPTileRows + rr) * 8 + c];
            if (d.n_p_chunks == 1) P[d.p_off + row * r + c] = (float)sum;
            else ws[d.ppart_off + ((int64_t)it.b * d.n + row) * r + c] = sum;
        }
    }
}

}  // namespace

}  // namespace conef
