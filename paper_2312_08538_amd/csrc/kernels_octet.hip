// Octet kernel family: the streaming passes for matrices whose rows hold whole scale blocks
// (cols % block == 0, block a power of two from 64 to 512, cols % 64 == 0) and rank 2, 4 or 8.
//
// A lane owns an "octet": 8 consecutive elements of a row -- one 16-byte (bf16) or two 16-byte
// (fp32) gradient loads, 16/32/64 bits of codes, one Philox call in the error pass.  `lr` lanes
// (8..64, a power of two) cover a row segment; 64/lr rows share a wave.
//
//   P pass    one workgroup per 64-row x column-chunk item on the fp64 matrix cores (rank padded to
//             16 columns).  Octets are decoded in the coalesced load layout, p goes through a
//             wave-private LDS tile and comes back in the operand layout; codes and scales are staged
//             through LDS in whole 128-byte lines.  Products of fp32 values are exact in fp64, the
//             sum stays in fp64, one rounding at the end.
//   Q+ pass   one wave per 64-column x row-tile item, same instruction with the roles of rows and
//             columns exchanged; per-tile fp64 partial sums go to the workspace and are added in
//             tile order by the reduction kernel.
//   err pass  one wave per strip x row range, Q+ tile (8 x r) in registers, residual as the fp32
//             fma chain, block max-norm by DPP, fixed-point stochastic rounding, pack, in place.
//             Ranks 4 and 8 with blocks up to 256: the same chain on the fp32 matrix cores (k_err_tile).
//
// All sums are combined in a fixed order: results do not depend on scheduling.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "octet_device.h"

namespace conef {

namespace {

// ------------------------------------------------------------------ the three passes (device code: octet_device.h)
template <bool BF16, int BITS, int RH, bool TWO = false>
__global__ __launch_bounds__(256) CONEF_P_OCTET_WAVES(TWO)
void k_p_octet(KernelPlan dp, const void *__restrict__ grads, const uint32_t *__restrict__ codes,
               const float *__restrict__ scales, const float *__restrict__ Q, float *P, double *ws)
{
    __shared__ __attribute__((aligned(16))) float tiles[kPOctetTiles];
    __shared__ __attribute__((aligned(16))) uint32_t code[kPOctetCodes];
    __shared__ float scale[kPOctetScales];
    __shared__ __attribute__((aligned(16))) uint32_t code1[TWO ? kPOctetCodes : 4];
    __shared__ float scale1[TWO ? kPOctetScales : 1];
    const POctetLds lds = {tiles, code, scale, code1, scale1};
    p_octet<BF16, BITS, RH, TWO>(dp, blockIdx.x, lds, grads, codes, scales, Q, P, ws);
}

template <bool BF16, int BITS, int RH, bool TWO, int JOINED>
__global__ __launch_bounds__(256) CONEF_Q_OCTET_WAVES(BF16, TWO)
void k_q_octet(KernelPlan dp, const void *__restrict__ grads, const uint32_t *__restrict__ codes,
               const float *__restrict__ scales, const float *__restrict__ Phat, double *ws, float *Qout)
{
    __shared__ __attribute__((aligned(16))) float lds[kQOctetLds];
    q_octet<BF16, BITS, RH, TWO, JOINED>(dp, blockIdx.x, lds, grads, codes, scales, Phat, ws, Qout);
}

template <bool BF16, int BITS, int RP, bool WIDE, bool TWO>
__global__ __launch_bounds__(256) CONEF_ERR_TILE_WAVES(BF16, WIDE, TWO)
void k_err_tile(KernelPlan dp, const void *__restrict__ grads, uint32_t *codes, float *scales,
                                                  const float *__restrict__ Phat, const float *__restrict__ Qn,
                                                  uint32_t step_lo, uint32_t step_hi, uint32_t *codes_first, float *scales_first)
{
    __shared__ float s_bq[err_tile_lds<RP, WIDE>()];
    err_tile<BF16, BITS, RP, WIDE, TWO>(dp, blockIdx.x, s_bq, grads, codes, scales, Phat, Qn, step_lo, step_hi, codes_first,
                                        scales_first);
}

// ------------------------------------------------------------------ element-wise gradient compressors
// MODE 0, random block (Section 5.3): Delta keeps the k consecutive coordinates [start, start + k) of p = g + (1 - beta) e and nothing
// else; the error compressor then takes beta e + p - Delta: g + e outside the block (the fma of the other
// passes), beta e inside it.  One streaming pass: a wave walks runs of 64 octets (512 elements) of the flat
// index; scale blocks of 8 * 2^j elements never straddle a run.  Decode, select, block max-norm by DPP,
// stochastic rounding, pack, in place; the kept values go to the Delta buffer.
// Scaled sign (Section 5.1), Delta = c sign(p) with c = ||p||_1 / N per matrix, takes two passes of the same walk:
// MODE 1 adds up |p| in fp64, one partial sum per wave in a fixed order (the scale kernel adds the partials in
// item order); MODE 2 reads c, writes one sign byte per octet (bit e set if element e is negative) and
// compresses (g + e) - Delta.
// TWO: improved contractive error feedback, version 1 (Algorithm 3, no beta): a second compressed vector q of the
// same layout (codes2, scales2) is added in the accumulation, p = g + e~ + q; the first vector becomes
// e~+ = C(p - Delta) as before and the second q+ = C(p - Delta - e~+): the decoded e~+ (rounded to fp32) is
// subtracted, the block maximum taken again and the difference rounded with random numbers of its own (matrix
// word of the Philox counter + 2^31), all in registers.
// MODE 3, random-k (stratified: one coordinate kept per stratum of rk_g consecutive ones, see strata_kept):
// as MODE 0 with the kept coordinates scattered; the kept values go to the Delta buffer in stratum order.
// MODE 4, random-k as a uniformly drawn subset (see rku_perm): the same; coordinate j is kept iff pi(j) < rk_uk and its value
// goes to slot pi(j).  Eight evaluations of the keyed permutation per octet: several times the arithmetic of MODE 3.

// V2: improved contractive error feedback, version 2 (Algorithm 3, no beta), for MODE 0 and 3: the first error vector
// is a random block of every matrix kept as it is (i2_k values, dp.i2_in; taken from the block drawn one step ago), the
// compressed vector is q: p = g + q, + e~ on that block; Delta = p on the kept coordinates; e~+ = p - Delta on the block
// drawn now (to dp.i2_out, another buffer: other waves still read the old one); q+ = C(p - Delta - e~+).
template <bool BF16, int BITS, int MODE, bool TWO, bool V2>
__global__ __launch_bounds__(256) void k_rb_octet(KernelPlan dp, const void *__restrict__ grads, uint32_t *codes, float *scales,
                                                  float *__restrict__ delta, uint32_t step_lo, uint32_t step_hi,
                                                  uint32_t *__restrict__ sign_words, const float *__restrict__ c_scale, double *ws,
                                                  uint32_t *codes2, float *scales2)
{
    constexpr bool BACK = TWO || V2;
    constexpr bool SPARSE = MODE == kModeBlock || MODE == kModeStrata || MODE == kModeUniform;      // Delta keeps a few coordinates as they are
    const int lane = threadIdx.x & 63;
    const int block = MODE == kModeNorm && dp.norm_back ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x;     // (see Plan::norm_back)
    const int item = __builtin_amdgcn_readfirstlane(block * 4 + (int)(threadIdx.x >> 6));
    if (item >= dp.n_rb) return;
    const WorkItem it = dp.rb_items[item];
    const MatDesc d = dp.mats[it.mat];
    const int64_t start = MODE == kModeBlock ? random_block_start((uint32_t)it.mat, step_lo, step_hi, dp.seed_lo, dp.seed_hi, d.N, d.rb_k) : 0;
    const int64_t stop = MODE == kModeBlock ? start + d.rb_k : 0;
    const float c = MODE == kModeSign ? c_scale[it.mat] : 0.0f;
    int64_t e_from = 0, e_to = 0;
    if (V2) {
        const uint64_t prev = (((uint64_t)step_hi << 32) | step_lo) - 1;
        e_from = i2_block_start((uint32_t)it.mat, (uint32_t)prev, (uint32_t)(prev >> 32), dp.seed_lo, dp.seed_hi, d.N, d.i2_k);
        e_to = i2_block_start((uint32_t)it.mat, step_lo, step_hi, dp.seed_lo, dp.seed_hi, d.N, d.i2_k);
    }
    RkuKeys ku = {};
    if (MODE == kModeUniform) ku = rku_keys((uint32_t)it.mat, step_lo, step_hi, dp.seed_lo, dp.seed_hi);
    __shared__ __attribute__((aligned(16))) float s_val[MODE == kModeStrata ? 4 : 1][MODE == kModeStrata ? 512 : 4];
    __shared__ uint32_t s_kept[MODE == kModeStrata && !BACK ? 4 : 1][64];
    __shared__ __attribute__((aligned(16))) uint32_t s_pos[MODE == kModeStrata ? 4 : 1][MODE == kModeStrata ? 256 : 4];
    uint32_t win = 0xFFFFFFFFu;        // MODE 3: first Philox call of the window of strata in s_pos (none yet)
    double l1 = 0.0;
    const float s_f = (float)((1 << (BITS - 1)) - 1);
    // The last run of a matrix may be short: octets beyond the end re-read the last octet and store nothing (where they share
    // its block, they repeat what it brings to the block's maximum).  The last octet may hold fewer than eight elements (tail):
    // the rest of it is read from the padding behind the matrix and counts as zero.
    const int64_t n_oct = (d.N + 7) >> 3;
    const int tail = (int)(d.N - ((n_oct - 1) << 3));
    // does the last octet end its code word and (sign mode) its sign word?
    const bool ends = tail != 8 || (BITS == 2 && (n_oct & 1) != 0) || (MODE == kModeSign && (n_oct & 3) != 0);
    // An octet of the item is a 32-bit distance from its first one, and an address a scalar base and such a distance (in 64 bits per
    // lane: 12 to 15 instructions more per octet).  The passes that round are bound by their vector instructions: random-k with two
    // vectors, 1.3 G elements, 1591 -> 1460 us with this and the kept coordinates' zeros read back below; the scaled sign, 210 M
    // elements of 2-bit codes, 227 -> 218 us for both passes with this, the signs of an octet at once, and p formed beside g + e only
    // where beta is not 0.
    const int64_t o_first = (int64_t)it.a * 64;             // (whole blocks)
    const uint32_t n_rel = (uint32_t)((n_oct - o_first < (int64_t)it.b * 64) ? n_oct - o_first : (int64_t)it.b * 64);
    const FlatOctets<BF16, BITS> base = flat_octets<BF16, BITS>(d, grads, codes, scales, o_first);
    const FlatCodes<BITS> base2 = TWO ? flat_codes<BITS>(d, codes2, scales2, o_first) : base.c;
    auto clamp = [&](uint32_t o) { return o < n_rel ? o : n_rel - 1; };
    RawOctet<BF16, BITS> cur = load_octet_rel<BF16, BITS>(base, d.lb_shift, clamp(lane));
    RawCodes<BITS> cur2 = {0u, 0u, 0.0f};
    if (TWO) cur2 = load_codes_rel<BITS>(base2, d.lb_shift, clamp(lane));
    // TAIL: the run that holds the last octet of a matrix that ends inside that octet or inside its word
    auto run = [&](int rr, auto tail_tag) {
        constexpr bool TAIL = decltype(tail_tag)::value;
        const uint32_t rel_raw = (uint32_t)(rr * 64 + lane);
        const bool valid = rel_raw < n_rel;
        const uint32_t rel = clamp(rel_raw);
        const int64_t o = o_first + rel;
        RawOctet<BF16, BITS> r = cur;
        RawCodes<BITS> r2 = cur2;
        const bool cut = TAIL && rel == n_rel - 1;
        // the next run is requested before this one is worked on (the last one re-reads itself)
        cur = load_octet_rel<BF16, BITS>(base, d.lb_shift, clamp(rel_raw + 64));
        if (TWO) cur2 = load_codes_rel<BITS>(base2, d.lb_shift, clamp(rel_raw + 64));
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
        if (TAIL) {
            // the code fields of a full octet (here because its word ends a code or sign word) all count: no shift by a word's width
            const uint64_t fields = tail < 8 ? (1ull << (BITS * tail)) - 1ull : ~0ull;
            const uint32_t lo = (uint32_t)fields, hi = (uint32_t)(fields >> 32);
            if (cut) {
                r.c0 &= lo; r.c1 &= hi; r2.c0 &= lo; r2.c1 &= hi;
#pragma unroll
                for (int e = 1; e < 8; ++e) g[e] = e < tail ? g[e] : 0.0f;
            }
        }
        const float dstep = r.scale * (inv_levels(BITS) * field_unit(BITS));
        const float dpart = TWO ? dstep : dstep * dp.omb;
        const float dstep2 = r2.scale * (inv_levels(BITS) * field_unit(BITS));
        float qf[8], qf2[8];
        code_values<BITS>(r.c0, r.c1, qf);
        if (TWO) code_values<BITS>(r2.c0, r2.c1, qf2);
        // Which of the octet's coordinates does the gradient compressor keep as they are (bit e of kbits), and where
        // does the first of them go in the Delta buffer (the others follow it)?  Most octets of a random block keep none.
        uint32_t kbits = 0;
        int64_t kslot = 0;
        if (MODE == kModeBlock) {
            const int64_t lo = start - o * 8, hi = stop - o * 8;       // the block in the octet's own coordinates
            if (hi > 0 && lo < 8) {
                const int l8 = lo > 0 ? (int)lo : 0, h8 = hi < 8 ? (int)hi : 8;
                kbits = ((1u << h8) - 1u) & ~((1u << l8) - 1u);
                kslot = d.rb_delta_off + (l8 - lo);
            }
        }
        uint32_t kpos[8];                                               // MODE 4: pi of the octet's coordinates
        if (MODE == kModeUniform) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                kpos[e] = rku_perm((uint32_t)(o * 8 + (cut && e >= tail ? 0 : e)), (uint32_t)d.N, d.rk_ua, d.rk_ub, d.rk_umagic, ku);
                kbits |= (kpos[e] < d.rk_uk ? 1u : 0u) << e;
            }
            if (cut) kbits &= (1u << tail) - 1u;
            kslot = d.rk_delta_off;
        }
        // x: the argument of the error compressor.  First as if nothing were kept: g + e (= beta e + p), or p = g + e~ + q
        float x[8];
        uint32_t neg_bits = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[e] = __builtin_fmaf(dstep, qf[e], g[e]);
            if (TWO) x[e] = __builtin_fmaf(dstep2, qf2[e], x[e]);
        }
        if (MODE == kModeNorm || MODE == kModeSign) {
            // |p| and its sign, p = g + (1 - beta) e: x itself where beta is 0 (the empty statement keeps the compiler from forming
            // both)
            float v[8];
            auto take = [&](int e, float pv) { v[e] = MODE == kModeNorm ? fabsf(pv) : __builtin_copysignf(c, pv); };
            if (TWO || dp.omb == 1.0f) {                            // uniform
#pragma unroll
                for (int e = 0; e < 8; ++e) take(e, x[e]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float pv = __builtin_fmaf(dpart, qf[e], g[e]);
                    asm volatile("" : "+v"(pv));
                    take(e, pv);
                }
            }
            if (MODE == kModeNorm) {
#pragma unroll
                for (int e = 0; e < 8; ++e) l1 += (double)(valid ? v[e] : 0.0f);
            } else {
                neg_bits = octet_signs(v);
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = x[e] - v[e];
            }
        }
        if (MODE == kModeNorm) return;
        if (MODE == kModeSign && TAIL && cut) {
            neg_bits &= (1u << tail) - 1u;
#pragma unroll
            for (int e = 1; e < 8; ++e) x[e] = e < tail ? x[e] : 0.0f;
        }
        if (V2) {
            // + e~ where it was taken from
            const int64_t lo = e_from - o * 8, hi = lo + d.i2_k;
            if (hi > 0 && lo < 8) {
                const float *src = dp.i2_in + d.i2_off - lo;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e >= lo && e < hi) x[e] = x[e] + src[e];
            }
        }
        // ... then the kept coordinates: Delta = p there, and beta e (plain) or nothing (two vectors) is left
        if (MODE == kModeStrata) {
            // The run's values of p go through LDS, and the lanes take the run's strata: each looks up its stratum's coordinate,
            // passes the value on and, where nothing stays behind (two vectors, version 2), leaves zero for the octet to read back,
            // else marks it in the octet's word.  (An octet looking for its strata's coordinates evaluated
            // two Philox calls and a branch per element: half of the pass.)
            // Strata of 8 or more: the coordinates are drawn a window at a time, 64 calls, one per lane, all four words of
            // each: 256 strata, that is four runs of the shortest.  (A call per lane and run used one word of its four: two vectors,
            // 1.3 G elements in strata of ten 1702 us, so 1591.)  Of shorter ones a run has more than a window would serve: a lane takes
            // the four of a call.
            float *sp = s_val[threadIdx.x >> 6];
            uint32_t *sk = s_kept[BACK ? 0 : threadIdx.x >> 6];
            uint32_t *su = s_pos[threadIdx.x >> 6];
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = (TWO || V2) ? x[e] : __builtin_fmaf(dpart, qf[e], g[e]);
            reinterpret_cast<float4 *>(sp + lane * 8)[0] = make_float4(p[0], p[1], p[2], p[3]);
            reinterpret_cast<float4 *>(sp + lane * 8)[1] = make_float4(p[4], p[5], p[6], p[7]);
            if (!BACK) sk[lane] = 0;
            const uint32_t N = (uint32_t)d.N, j0 = (uint32_t)(((int64_t)it.a + rr) << 9);
            const uint32_t s0 = stratum_of(j0, d.rk_g, d.rk_magic), s1 = stratum_of(N - 1u - j0 < 511u ? N - 1u : j0 + 511u, d.rk_g, d.rk_magic);
            uint32_t out[4];
            auto position = [&](uint32_t s, uint32_t u) {
                const uint32_t base = s * d.rk_g;
                const uint32_t len = N - base < d.rk_g ? N - base : d.rk_g;
                return base + __umulhi(u, len);
            };
            auto take = [&](uint32_t s, uint32_t pos) {
                const uint32_t rel = pos - j0;                                // wraps to a large value before the run
                if (rel < 512u) {
                    delta[d.rk_delta_off + s] = sp[rel];
                    if (BACK) sp[rel] = 0.0f;
                    else __hip_atomic_fetch_or(sk + (rel >> 3), 1u << (rel & 7u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            };
            if (d.rk_g >= 8) {
                if (win == 0xFFFFFFFFu || (s1 >> 2) - win >= 64u) {          // uniform
                    win = s0 >> 2;
                    philox4x32_10(win + lane, (uint32_t)it.mat + 0x40000000u, step_lo, step_hi, dp.seed_lo, dp.seed_hi, out);
                    const uint32_t s = (win + lane) * 4;                      // (strata behind the last one are never looked up)
                    *reinterpret_cast<uint4 *>(su + lane * 4) =
                        make_uint4(position(s, out[0]), position(s + 1, out[1]), position(s + 2, out[2]), position(s + 3, out[3]));
                }
                wave_memory_sync();
                for (uint32_t s = s0 + lane; s <= s1; s += 64) take(s, su[s - win * 4]);
            } else {
                wave_memory_sync();
                for (uint32_t q = (s0 >> 2) + lane; q <= (s1 >> 2); q += 64) {
                    philox4x32_10(q, (uint32_t)it.mat + 0x40000000u, step_lo, step_hi, dp.seed_lo, dp.seed_hi, out);
#pragma unroll
                    for (uint32_t w = 0; w < 4; ++w)
                        if (q * 4 + w >= s0 && q * 4 + w <= s1) take(q * 4 + w, position(q * 4 + w, out[w]));
                }
            }
            wave_memory_sync();
            // (an octet beyond the end must not bring the last octet's coordinates to the maximum)
            if (BACK) {
                const float4 lo = reinterpret_cast<const float4 *>(sp + lane * 8)[0], hi = reinterpret_cast<const float4 *>(sp + lane * 8)[1];
                x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w; x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
                if ((uint32_t)(rr * 64 + 64) > n_rel) {             // uniform
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = valid ? x[e] : 0.0f;
                }
            } else {
                const uint32_t left = valid ? ~sk[lane] : 0u;
                const float back = valid ? dp.beta : 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const bool keep = (left >> e) & 1u;             // nothing was taken
                    x[e] = keep ? x[e] : back * (dstep * qf[e]);
                }
            }
            wave_memory_sync();                // the next run's values may not overtake these reads
        } else if (SPARSE && kbits != 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if ((kbits >> e) & 1u) {
                    const int64_t slot = kslot + (MODE == kModeUniform ? kpos[e] : (uint32_t)__popc(kbits & ((1u << e) - 1u)));
                    if (TWO || V2) {
                        if (valid) delta[slot] = x[e];
                        x[e] = 0.0f;
                    } else {
                        if (valid) delta[slot] = __builtin_fmaf(dpart, qf[e], g[e]);
                        x[e] = dp.beta * (dstep * qf[e]);
                    }
                }
            }
        }
        if (V2) {
            // e~+: what is left on the block drawn now, as it is (0 where Delta has taken it)
            const int64_t lo = e_to - o * 8, hi = lo + d.i2_k;
            if (hi > 0 && lo < 8) {
                float *dst = dp.i2_out + d.i2_off - lo;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (e >= lo && e < hi) {
                        if (valid) dst[e] = x[e];
                        x[e] = 0.0f;
                    }
                }
            }
        }
        if (MODE == kModeSign && valid) {
            uint8_t *sb = reinterpret_cast<uint8_t *>(sign_words + d.sign_off) + o_first;
            sb[rel] = (uint8_t)neg_bits;
            if (TAIL && cut)
                for (uint32_t b = rel + 1; (b & 3) != 0; ++b) sb[b] = 0;       // the rest of the last word (o_first is a whole one)
        }
        const float a = block_max(abs_max_octet(0.0f, x), d.lb_shift);
        const float inv16 = levels_over(a, s_f);
        uint32_t rnd[4], w[2];
        int32_t t[8];
        philox4x32_10((uint32_t)o, (uint32_t)it.mat, step_lo, step_hi, dp.seed_lo, dp.seed_hi, rnd);
        quantise_octet<BITS>(x, inv16, rnd, w, t);
        if (valid) {
            if (cut) store_code_words_end<BITS>(d, codes, o, tail, w);
            else store_codes_rel<BITS>(base.c, rel, w);
            if ((lane & ((1 << d.lb_shift) - 1)) == 0) store_scale_rel(base.c, rel >> d.lb_shift, a);
        }
        if (TWO) {
            // q+ = C(x - e~+): what the first rounding left, one level finer
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
                if (cut) store_code_words_end<BITS>(d, codes2, o, tail, w);
                else store_codes_rel<BITS>(base2, rel, w);
                if ((lane & ((1 << d.lb_shift) - 1)) == 0) store_scale_rel(base2, rel >> d.lb_shift, a2);
            }
        }
    };
    const int whole = ends && (((int64_t)it.a + it.b) << 6) >= n_oct ? it.b - 1 : it.b;
    for (int rr = 0; rr < whole; ++rr) run(rr, std::false_type{});
    if (whole < it.b) run(whole, std::true_type{});
    if (MODE == kModeNorm) {
        l1 = wave_sum(l1);
        if (lane == 0) ws[d.st_part_off + (item - d.st_first)] = l1;
    }
}

}  // namespace

// mode: 0 random block, 1 l1-norm partials of the scaled sign, 2 scaled sign, 3 and 4 random-k; codes2 / scales2: the second error
// vector of Algorithm 3, or null for plain contractive error feedback
void octet_stream_step(const DevicePlan &dp, int mode, const void *grads, uint32_t *codes, float *scales, float *delta,
                       uint64_t step, uint32_t *sign_words, const float *c_scale, double *ws, uint32_t *codes2,
                       float *scales2, hipStream_t st)
{
    if (dp.n_rb <= 0) return;
    const dim3 grid((dp.n_rb + 3) / 4);
    const uint32_t lo = (uint32_t)step, hi = (uint32_t)(step >> 32);
    const bool two = codes2 != nullptr, v2 = dp.i2_out != nullptr;
    KernelPlan kp = dp;
    kp.norm_back = two ? dp.norm_back_two : dp.norm_back_one;
#define CONEF_STREAM_LAUNCH(BF, B, M, T, V)                                                                                        \
    hipLaunchKernelGGL((k_rb_octet<BF, B, M, T, V>), grid, dim3(256), 0, st, kp, grads, codes, scales, delta, lo, hi, sign_words,  \
                       c_scale, ws, codes2, scales2)
#define CONEF_STREAM_MODE(BF, B, M)                                                                                                \
    do {                                                                                                                           \
        if (two) CONEF_STREAM_LAUNCH(BF, B, M, true, false);                                                                       \
        else CONEF_STREAM_LAUNCH(BF, B, M, false, false);                                                                          \
    } while (0)
#define CONEF_STREAM_MODE_V2(BF, B, M)                                                                                             \
    do {                                                                                                                           \
        if (v2 && !two) CONEF_STREAM_LAUNCH(BF, B, M, false, true);                                                                \
        else CONEF_STREAM_MODE(BF, B, M);                                                                                          \
    } while (0)
#define CONEF_STREAM_CASE(BF, B)                                                                                                   \
    case ((BF ? 1 : 0) << 8) | B:                                                                                                  \
        if (mode == kModeBlock) CONEF_STREAM_MODE_V2(BF, B, kModeBlock);                                                           \
        else if (mode == kModeStrata) CONEF_STREAM_MODE_V2(BF, B, kModeStrata);                                                    \
        else if (mode == kModeUniform) CONEF_STREAM_MODE_V2(BF, B, kModeUniform);                                                  \
        else if (mode == kModeNorm) CONEF_STREAM_MODE(BF, B, kModeNorm);                                                           \
        else CONEF_STREAM_MODE(BF, B, kModeSign);                                                                                  \
        break;
    switch ((dp.dtype << 8) | dp.bits) {
        CONEF_STREAM_CASE(false, 2)
        CONEF_STREAM_CASE(false, 4)
        CONEF_STREAM_CASE(false, 8)
        CONEF_STREAM_CASE(true, 2)
        CONEF_STREAM_CASE(true, 4)
        CONEF_STREAM_CASE(true, 8)
    default: break;
    }
#undef CONEF_STREAM_LAUNCH
#undef CONEF_STREAM_MODE
#undef CONEF_STREAM_MODE_V2
#undef CONEF_STREAM_CASE
}

#define CONEF_OCTET_CASE(KERNEL, BF, B, R, GRID, ST, ...) \
    case ((BF ? 1 : 0) << 8) | (B << 4) | R: hipLaunchKernelGGL((KERNEL<BF, B, R>), GRID, dim3(256), 0, ST, __VA_ARGS__); break;

#define CONEF_OCTET_DISPATCH(KERNEL, GRID, ST, ...)                                  \
    do {                                                                             \
        switch ((dp.dtype << 8) | (dp.bits << 4) | dp.rank) {                        \
            CONEF_OCTET_CASE(KERNEL, false, 2, 2, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, false, 2, 4, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, false, 2, 8, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, false, 4, 2, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, false, 4, 4, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, false, 4, 8, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, false, 8, 2, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, false, 8, 4, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, false, 8, 8, GRID, ST, __VA_ARGS__)             \
            CONEF_OCTET_CASE(KERNEL, true, 2, 2, GRID, ST, __VA_ARGS__)              \
            CONEF_OCTET_CASE(KERNEL, true, 2, 4, GRID, ST, __VA_ARGS__)              \
            CONEF_OCTET_CASE(KERNEL, true, 2, 8, GRID, ST, __VA_ARGS__)              \
            CONEF_OCTET_CASE(KERNEL, true, 4, 2, GRID, ST, __VA_ARGS__)              \
            CONEF_OCTET_CASE(KERNEL, true, 4, 4, GRID, ST, __VA_ARGS__)              \
            CONEF_OCTET_CASE(KERNEL, true, 4, 8, GRID, ST, __VA_ARGS__)              \
            CONEF_OCTET_CASE(KERNEL, true, 8, 2, GRID, ST, __VA_ARGS__)              \
            CONEF_OCTET_CASE(KERNEL, true, 8, 4, GRID, ST, __VA_ARGS__)              \
            CONEF_OCTET_CASE(KERNEL, true, 8, 8, GRID, ST, __VA_ARGS__)              \
        default: break; /* the plan selects this family for ranks 2, 4, 8 only */    \
        }                                                                            \
    } while (0)

#define CONEF_OCTET2_CASE(KERNEL, BF, B, GRID, ST, ...)                                                         \
    case ((BF ? 1 : 0) << 8) | B:                                                                              \
        if (dp.rank > 4) hipLaunchKernelGGL((KERNEL<BF, B, 2>), GRID, dim3(256), 0, ST, __VA_ARGS__);          \
        else hipLaunchKernelGGL((KERNEL<BF, B, 1>), GRID, dim3(256), 0, ST, __VA_ARGS__);                      \
        break;

#define CONEF_OCTET2_DISPATCH(KERNEL, GRID, ST, ...)                     \
    do {                                                                 \
        switch ((dp.dtype << 8) | dp.bits) {                             \
            CONEF_OCTET2_CASE(KERNEL, false, 2, GRID, ST, __VA_ARGS__)   \
            CONEF_OCTET2_CASE(KERNEL, false, 4, GRID, ST, __VA_ARGS__)   \
            CONEF_OCTET2_CASE(KERNEL, false, 8, GRID, ST, __VA_ARGS__)   \
            CONEF_OCTET2_CASE(KERNEL, true, 2, GRID, ST, __VA_ARGS__)    \
            CONEF_OCTET2_CASE(KERNEL, true, 4, GRID, ST, __VA_ARGS__)    \
            CONEF_OCTET2_CASE(KERNEL, true, 8, GRID, ST, __VA_ARGS__)    \
        default: break;                                                  \
        }                                                                \
    } while (0)

// the two-vector instances (a plan that carries a first error vector, see DevicePlan::i_codes)
#define CONEF_OCTET2T_CASE(KERNEL, BF, B, GRID, ST, ...)                                                           \
    case ((BF ? 1 : 0) << 8) | B:                                                                                  \
        if (dp.rank > 4) hipLaunchKernelGGL((KERNEL<BF, B, 2, true>), GRID, dim3(256), 0, ST, __VA_ARGS__);        \
        else hipLaunchKernelGGL((KERNEL<BF, B, 1, true>), GRID, dim3(256), 0, ST, __VA_ARGS__);                    \
        break;

#define CONEF_OCTET2T_DISPATCH(KERNEL, GRID, ST, ...)                     \
    do {                                                                  \
        switch ((dp.dtype << 8) | dp.bits) {                              \
            CONEF_OCTET2T_CASE(KERNEL, false, 2, GRID, ST, __VA_ARGS__)   \
            CONEF_OCTET2T_CASE(KERNEL, false, 4, GRID, ST, __VA_ARGS__)   \
            CONEF_OCTET2T_CASE(KERNEL, false, 8, GRID, ST, __VA_ARGS__)   \
            CONEF_OCTET2T_CASE(KERNEL, true, 2, GRID, ST, __VA_ARGS__)    \
            CONEF_OCTET2T_CASE(KERNEL, true, 4, GRID, ST, __VA_ARGS__)    \
            CONEF_OCTET2T_CASE(KERNEL, true, 8, GRID, ST, __VA_ARGS__)    \
        default: break;                                                   \
        }                                                                 \
    } while (0)

void octet_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales,
                  const float *Q, float *P, double *ws, hipStream_t st)
{
    if (dp.n_p_f <= 0) return;
    if (dp.i_codes) CONEF_OCTET2T_DISPATCH(k_p_octet, dim3(dp.n_p_f), st, dp, grads, codes, scales, Q, P, ws);
    else CONEF_OCTET2_DISPATCH(k_p_octet, dim3(dp.n_p_f), st, dp, grads, codes, scales, Q, P, ws);
}

void octet_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales,
                  const float *Phat, double *ws, float *Qout, hipStream_t st)
{
    if (dp.n_q_f <= 0) return;
    auto go = [&](auto bf, auto bits, auto half, auto two, auto joined) {
        hipLaunchKernelGGL((k_q_octet<decltype(bf)::value, decltype(bits)::value, decltype(half)::value, decltype(two)::value,
                                      decltype(joined)::value>),
                           dim3(q_octet_groups(dp)), dim3(256), 0, st, dp, grads, codes, scales, Phat, ws, Qout);
    };
    auto form = [&](auto bf, auto bits, auto half, auto two) {
        if constexpr (decltype(half)::value == 1) go(bf, bits, half, two, std::integral_constant<int, kQJoinedAtRunTime>{});
        else if (dp.q_joined) go(bf, bits, half, two, std::integral_constant<int, kQJoinedYes>{});
        else go(bf, bits, half, two, std::integral_constant<int, kQJoinedNo>{});
    };
    auto vectors = [&](auto bf, auto bits, auto half) {
        if (dp.i_codes) form(bf, bits, half, std::true_type{});
        else form(bf, bits, half, std::false_type{});
    };
    auto rank = [&](auto bf, auto bits) {
        if (dp.rank > 4) vectors(bf, bits, std::integral_constant<int, 2>{});
        else vectors(bf, bits, std::integral_constant<int, 1>{});
    };
    auto width = [&](auto bf) {
        if (dp.bits == 2) rank(bf, std::integral_constant<int, 2>{});
        else if (dp.bits == 4) rank(bf, std::integral_constant<int, 4>{});
        else rank(bf, std::integral_constant<int, 8>{});
    };
    if (dp.dtype == 1) width(std::true_type{});
    else width(std::false_type{});
}

// The strip kernel for the plan's err_t_items (rank 4 or 8; `first`: the first vector of Algorithm 3, or null)
template <bool TWO>
static void launch_err_tile(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat,
                            const float *Qn, uint64_t step, uint32_t *codes_first, float *scales_first, hipStream_t st)
{
    if (dp.n_err_t <= 0) return;
    const dim3 grid((dp.n_err_t + 3) / 4);
    const uint32_t lo = (uint32_t)step, hi = (uint32_t)(step >> 32);
#define CONEF_ERR_TILE_CASE(BF, B, R)                                                                                             \
    case ((BF ? 1 : 0) << 8) | (B << 4) | R:                                                                                      \
        if (dp.block == 256)                                                                                                      \
            hipLaunchKernelGGL((k_err_tile<BF, B, R, true, TWO>), grid, dim3(256), 0, st, dp, grads, codes, scales, Phat, Qn, lo, \
                               hi, codes_first, scales_first);                                                                    \
        else                                                                                                                      \
            hipLaunchKernelGGL((k_err_tile<BF, B, R, false, TWO>), grid, dim3(256), 0, st, dp, grads, codes, scales, Phat, Qn,    \
                               lo, hi, codes_first, scales_first);                                                                \
        break;
#define CONEF_ERR_TILE_DTYPE(BF)                                                                    \
    CONEF_ERR_TILE_CASE(BF, 2, 4) CONEF_ERR_TILE_CASE(BF, 2, 8) CONEF_ERR_TILE_CASE(BF, 4, 4)       \
    CONEF_ERR_TILE_CASE(BF, 4, 8) CONEF_ERR_TILE_CASE(BF, 8, 4) CONEF_ERR_TILE_CASE(BF, 8, 8)
    switch ((dp.dtype << 8) | (dp.bits << 4) | dp.rank) {
        CONEF_ERR_TILE_DTYPE(false)
        CONEF_ERR_TILE_DTYPE(true)
    default: break;
    }
#undef CONEF_ERR_TILE_CASE
#undef CONEF_ERR_TILE_DTYPE
}

void octet_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat,
                    const float *Qn, uint64_t step, hipStream_t st)
{
    launch_err_tile<false>(dp, grads, codes, scales, Phat, Qn, step, nullptr, nullptr, st);
    if (dp.n_err_f <= 0) return;
    CONEF_OCTET_DISPATCH(k_err_octet, dim3((dp.n_err_f + 3) / 4), st, dp, grads, codes, scales, Phat, Qn,
                         (uint32_t)step, (uint32_t)(step >> 32), (uint32_t *)nullptr, (float *)nullptr);
}

// The err pass of improved contractive error feedback: codes / scales hold the first vector, codes2 / scales2 the
// second; both are decoded and both replaced.
void octet_pass_err_two(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2,
                        float *scales2, const float *Phat, const float *Qn, uint64_t step, hipStream_t st)
{
    launch_err_tile<true>(dp, grads, codes2, scales2, Phat, Qn, step, codes, scales, st);
    if (dp.n_err_f <= 0) return;
    const dim3 grid((dp.n_err_f + 3) / 4);
#define CONEF_ERR_TWO_CASE(BF, B, R)                                                                                    \
    case ((BF ? 1 : 0) << 8) | (B << 4) | R:                                                                            \
        hipLaunchKernelGGL((k_err_octet<BF, B, R, true>), grid, dim3(256), 0, st, dp, grads, codes2, scales2, Phat,     \
                           Qn, (uint32_t)step, (uint32_t)(step >> 32), codes, scales);                                  \
        break;
#define CONEF_ERR_TWO_DTYPE(BF)                                                                   \
    CONEF_ERR_TWO_CASE(BF, 2, 2) CONEF_ERR_TWO_CASE(BF, 2, 4) CONEF_ERR_TWO_CASE(BF, 2, 8)        \
    CONEF_ERR_TWO_CASE(BF, 4, 2) CONEF_ERR_TWO_CASE(BF, 4, 4) CONEF_ERR_TWO_CASE(BF, 4, 8)        \
    CONEF_ERR_TWO_CASE(BF, 8, 2) CONEF_ERR_TWO_CASE(BF, 8, 4) CONEF_ERR_TWO_CASE(BF, 8, 8)
    switch ((dp.dtype << 8) | (dp.bits << 4) | dp.rank) {
        CONEF_ERR_TWO_DTYPE(false)
        CONEF_ERR_TWO_DTYPE(true)
    default: break;
    }
#undef CONEF_ERR_TWO_DTYPE
#undef CONEF_ERR_TWO_CASE
}

}  // namespace conef
