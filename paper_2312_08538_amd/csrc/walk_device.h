// Device code of the strip family's err pass for matrices whose Q+ fits into LDS (see kernels_walk.hip), for its own launches and
// for those that carry the octet family's workgroups too (kernels_mixed.hip).
#pragma once
#include "device_common.h"
#include "kernels.h"
#include "octet_device.h"

namespace conef {

namespace {

// A workgroup walks runs of 64 octets (512 elements) of the flat index, four waves in turn; a lane keeps its octet in registers
// from load to store, as in the stream kernels.  The octet's columns are wherever the row length puts them: its eight rows of Q+
// are read from LDS, where the whole factor stands (with its first rows once more behind the last one, for octets that reach into
// the next row of the matrix), and the one or two rows of P^ from memory.
// In LDS the rows of Q+ stand in groups of eight with 16 bytes between the groups: neighbouring lanes are eight columns apart, and
// without the gap their reads of 16 bytes fall on the same banks.
// R: the rank or the next of 1, 2, 4, 8 (both factors are zero beyond the rank: such terms leave the fp32 chain as it is).
// TWO: both error vectors are decoded and replaced (codes / scales: the first); see k_rb_octet.
template <bool BF16, int BITS, int R, bool TWO>
__device__ __forceinline__ void err_walk(const KernelPlan &dp, int block, float *tab, const void *__restrict__ grads, uint32_t *codes,
                                         float *scales, uint32_t *codes2, float *scales2, const float *__restrict__ Phat,
                                         const float *__restrict__ Qn, uint32_t step_lo, uint32_t step_hi)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WorkItem it = dp.err_w_items[block];
    const MatDesc d = dp.mats[it.mat];
    const int r = dp.rank, lb = dp.lb_shift;
    const uint32_t m = (uint32_t)d.m;
    const float s_f = (float)((1 << (BITS - 1)) - 1);
    // octets by their 32-bit distance from the item's first one; those beyond the matrix re-read its last one and store nothing
    // (where they share its block, they repeat what it brings to the block's maximum)
    const int64_t o_first = (int64_t)it.a * 64, n_oct = (d.N + 7) >> 3;
    const uint32_t n_rel = (uint32_t)((n_oct - o_first < (int64_t)it.b * 64) ? n_oct - o_first : (int64_t)it.b * 64);
    const int tail = (int)(d.N - ((n_oct - 1) << 3));               // elements of the matrix's last octet
    const bool at_end = o_first + n_rel == n_oct;                   // the item's last octet is that one
    const FlatOctets<BF16, BITS> base = flat_octets<BF16, BITS>(d, grads, codes, scales, o_first);
    const FlatCodes<BITS> base2 = TWO ? flat_codes<BITS>(d, codes2, scales2, o_first) : base.c;
    auto clamp = [&](uint32_t o) { return o < n_rel ? o : n_rel - 1; };
    RawOctet<BF16, BITS> cur;
    RawCodes<BITS> cur2 = {0u, 0u, 0.0f};
    auto load = [&](int run) {
        const uint32_t rel = clamp((uint32_t)(run * 64 + lane));
        cur = load_octet_rel<BF16, BITS>(base, lb, rel);
        if (TWO) cur2 = load_codes_rel<BITS>(base2, lb, rel);
    };
    // an octet's first row, relative to the item's (it.c), and column: element 8 rel + off of that row's flat index, divided by m
    // (exact: m times an item's elements is below 2^32)
    const uint32_t off = (uint32_t)(o_first * 8 - (int64_t)it.c * d.m);
    const uint32_t magic = m == 1 ? 0u : 0xFFFFFFFFu / m + 1;
    const float *prun = Phat + d.p_off + (int64_t)it.c * r;
    const uint32_t last_row = (uint32_t)(d.n - 1 - it.c < 0x7FFFFFFF ? d.n - 1 - it.c : 0x7FFFFFFF);
    float ph[2][R];
    uint32_t col = 0;
    auto load_rows = [&](int run) {
        const uint32_t at = clamp((uint32_t)(run * 64 + lane)) * 8 + off;
        const uint32_t row = __umulhi(at, magic);
        col = at - row * m;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t rw = row + h < last_row ? row + h : last_row;
            const float *src = prun + rw * (uint32_t)r;
            if (R >= 4 && r == R) {                                 // uniform
#pragma unroll
                for (int c4 = 0; c4 < R / 4; ++c4) {
                    const float4 v = reinterpret_cast<const float4 *>(src)[c4];
                    ph[h][4 * c4] = v.x; ph[h][4 * c4 + 1] = v.y; ph[h][4 * c4 + 2] = v.z; ph[h][4 * c4 + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int c = 0; c < R; ++c) {
                    const float v = src[c < r ? c : r - 1];
                    ph[h][c] = c < r ? v : 0.0f;
                }
            }
        }
    };
    load(wave);
    load_rows(wave);
    {
        const float *src = Qn + d.q_off;
        if (R >= 4 && r == R) {                                     // uniform; a row of Q+ or half of one per access, four in flight
            constexpr int V = R >= 4 ? R / 4 : 1;
            const int n_vec = (int)(m + 8) * V;
            for (int e0 = tid; e0 < n_vec; e0 += 4 * 256) {
                float4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = e0 + 256 * u < n_vec ? e0 + 256 * u : tid;
                    v[u] = reinterpret_cast<const float4 *>(src)[e < (int)m * V ? e : e - (int)m * V];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = e0 + 256 * u;
                    if (e < n_vec) reinterpret_cast<float4 *>(tab)[e + e / (8 * V)] = v[u];
                }
            }
        } else {
#pragma unroll 4
            for (int e = tid; e < (int)(m + 8) * R; e += 256) {
                const int k = e / R, c = e % R;
                const float v = src[(k < (int)m ? k : k - (int)m) * r + (c < r ? c : r - 1)];
                tab[k * R + (k >> 3) * 4 + c] = c < r ? v : 0.0f;
            }
        }
    }
    __syncthreads();
    for (int run = wave; run < it.b; run += 4) {
        const uint32_t rel_raw = (uint32_t)(run * 64 + lane);
        const bool valid = rel_raw < n_rel;
        const uint32_t rel = clamp(rel_raw);
        const bool cut = at_end && rel == n_rel - 1;
        float x[8], acc[8];
        decode_octet<BF16, BITS>(cur, 1.0f, x);
        if (TWO) add_codes<BITS>(cur2, x);
        load(run + 4 < it.b ? run + 4 : run);
        // rows of Q+ from column `col` on: the gap between groups of eight comes in where the octet passes into the next one
        const float *q = tab + col * R + (col >> 3) * 4;
        const uint32_t gaps = 0xFF00u >> (col & 7u);    // bit e: column col + e is in the next group
        const uint32_t in_row = m - col;                            // elements of the octet in its first row
        const bool two_rows = in_row < 8u;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
        auto chain = [&](auto both_tag) {
            constexpr bool BOTH = decltype(both_tag)::value;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float *qe = q + e * R + ((gaps >> e) & 1u) * 4;
                float qv[R];
                if constexpr (R >= 4) {
#pragma unroll
                    for (int c4 = 0; c4 < R / 4; ++c4) {
                        const float4 v = reinterpret_cast<const float4 *>(qe)[c4];
                        qv[4 * c4] = v.x; qv[4 * c4 + 1] = v.y; qv[4 * c4 + 2] = v.z; qv[4 * c4 + 3] = v.w;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < R; ++c) qv[c] = qe[c];
                }
#pragma unroll
                for (int c = 0; c < R; ++c) {
                    const float p = BOTH && (uint32_t)e >= in_row ? ph[1][c] : ph[0][c];
                    acc[e] = __builtin_fmaf(p, qv[c], acc[e]);
                }
            }
        };
        if (__any(two_rows)) chain(std::true_type{});
        else chain(std::false_type{});
        load_rows(run + 4 < it.b ? run + 4 : run);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = x[e] - acc[e];
        if (at_end && (uint32_t)(run * 64 + 64) >= n_rel && tail < 8) {     // uniform
#pragma unroll
            for (int e = 1; e < 8; ++e) x[e] = cut && e >= tail ? 0.0f : x[e];
        }
        const uint32_t o = (uint32_t)o_first + rel;
        auto round_octet = [&](uint32_t mat_word, const FlatCodes<BITS> &to, uint32_t *to_codes, int32_t (&t)[8]) {
            const float a = block_max(abs_max_octet(0.0f, x), lb);
            const float inv16 = levels_over(a, s_f);
            uint32_t rnd[4], w[2];
            philox4x32_10(o, mat_word, step_lo, step_hi, dp.seed_lo, dp.seed_hi, rnd);
            quantise_octet<BITS>(x, inv16, rnd, w, t);
            if (valid) {
                if (cut) store_code_words_end<BITS>(d, to_codes, o_first + rel, tail, w);
                else store_codes_rel<BITS>(to, rel, w);
                if ((lane & ((1 << lb) - 1)) == 0) store_scale_rel(to, rel >> lb, a);
            }
            return a;
        };
        int32_t t[8];
        const float a = round_octet((uint32_t)it.mat, base.c, codes, t);
        if (TWO) {
            const float dnew = a * inv_levels(BITS);
            float qn[8];
            rounded_values(t, qn);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = x[e] - dnew * qn[e];
            round_octet((uint32_t)it.mat | 0x80000000u, base2, codes2, t);
        }
    }
}

}  // namespace

}  // namespace conef
