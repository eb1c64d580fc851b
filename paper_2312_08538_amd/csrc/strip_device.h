// Device code of the strip family's three passes (see kernels_strip.hip), for its own launches and for those that carry the
// octet family's workgroups too (kernels_mixed.hip).
#pragma once
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "ragged_device.h"

namespace conef {

namespace {

constexpr int kSrcOne = 0, kSrcTwo = 1, kSrcRow = 2, kSrcCol = 3;      // quantiser with one / two vectors, sketch by rows / columns

typedef double f64x4 __attribute__((ext_vector_type(4)));

// What a lane loads for one element.
template <int SRC>
struct Raw {
    uint32_t g;                 // gradient bits (fp32, or bf16 in the low half)
    uint32_t c, c2;             // code words (c2: the second vector), or the table entry's bits in c
    float s, s2;                // block scales, or (sketch) the signed 1 - beta in s
};

struct Source {
    const void *grads;
    const uint32_t *codes;      // kSrcTwo: the second vector (the first is in the plan)
    const float *scales;
    const void *table;
};

// (1 - beta) with the sign of a hashed row or column folded in
__device__ __forceinline__ float signed_omb(float omb, int32_t hv) { return hv < 0 ? -omb : omb; }

// Where a wave's elements lie: the arrays from the scale block on that holds the element the wave starts from, so that a
// lane needs only its 32-bit distance `rel` from that block's first element: code word rel >> wshift, bit rel * bits mod
// 32, block rel / block, and every load is a scalar base plus a 32-bit offset.  (Per-row 64-bit addresses and divisions on
// the scalar side, a quarter of the vector issue rate, took twice as long as everything else in these kernels.)  The plan
// keeps a workgroup's rows within 2^29 elements.
template <int SRC>
struct Base {
    const void *g;
    const uint32_t *c, *c2;     // first (or only) and second vector
    const float *s, *s2;
    int64_t j;                  // the element the arrays start at (sketch: the starting element itself)
};

template <int SRC>
__device__ __forceinline__ Base<SRC> make_base(const KernelPlan &dp, const MatDesc &d, const Source &src, int64_t start, uint32_t *rel0)
{
    Base<SRC> b;
    int64_t blk = 0;
    b.j = start;
    if (SRC == kSrcOne || SRC == kSrcTwo) {
        blk = (int64_t)__umul64hi((uint64_t)start, dp.bmagic);
        b.j = blk * dp.block;
        const int64_t w = d.word_off + (b.j >> dp.wshift);
        b.c = (SRC == kSrcTwo ? dp.i_codes : src.codes) + w;
        b.s = (SRC == kSrcTwo ? dp.i_scales : src.scales) + d.scale_off + blk;
        b.c2 = src.codes + w;
        b.s2 = src.scales + d.scale_off + blk;
    } else {
        b.c = b.c2 = nullptr;
        b.s = b.s2 = nullptr;
    }
    b.g = dp.dtype == 0 ? (const void *)(reinterpret_cast<const float *>(src.grads) + d.grad_off + b.j)
                        : (const void *)(reinterpret_cast<const uint16_t *>(src.grads) + d.grad_off + b.j);
    *rel0 = (uint32_t)(start - b.j);
    return b;
}

// Loads U elements of a lane, at distances rel[u] from the base; row[u] / col are their matrix row (uniform) and first
// column of the strip (lc: the lane's offset from it), hv_col the lane's column hash: used by the sketch forms only.
template <int SRC, int U>
__device__ __forceinline__ void load_rows(const KernelPlan &dp, const MatDesc &d, const Source &src, const Base<SRC> &b,
                                          const uint32_t (&rel)[U], const int64_t (&row)[U], int64_t col, uint32_t lc, int32_t hv_col,
                                          Raw<SRC> (&o)[U])
{
    if (dp.dtype == 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) o[u].g = reinterpret_cast<const uint32_t *>(b.g)[rel[u]];
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) o[u].g = reinterpret_cast<const uint16_t *>(b.g)[rel[u]];
    }
    if (SRC == kSrcOne || SRC == kSrcTwo) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            o[u].c = b.c[rel[u] >> dp.wshift];
            if (SRC == kSrcTwo) o[u].c2 = b.c2[rel[u] >> dp.wshift];
        }
        if (dp.block_shift >= 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                o[u].s = b.s[rel[u] >> dp.block_shift];
                if (SRC == kSrcTwo) o[u].s2 = b.s2[rel[u] >> dp.block_shift];
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t blk = rel[u] / (uint32_t)dp.block;
                o[u].s = b.s[blk];
                if (SRC == kSrcTwo) o[u].s2 = b.s2[blk];
            }
        }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // row form: the row's bucket; column form: the column's
            const int32_t hv = SRC == kSrcRow ? dp.row_hash[d.hash_off + row[u]] : hv_col;
            const int64_t base = SRC == kSrcRow ? d.table_off + (int64_t)(hv & INT32_MAX) * d.m + col : d.table_off + row[u] * d.w;
            const uint32_t off = SRC == kSrcRow ? lc : (uint32_t)(hv & INT32_MAX);
            if (dp.table_dtype == 1) o[u].c = (reinterpret_cast<const uint16_t *>(src.table) + base)[off];
            else o[u].c = (reinterpret_cast<const uint32_t *>(src.table) + base)[off];
            o[u].s = signed_omb(dp.omb, hv);
        }
    }
}

// p of a loaded element at distance rel.
template <int SRC>
__device__ __forceinline__ float form_p(const KernelPlan &dp, const Raw<SRC> &o, uint32_t rel, float omb)
{
    const float g = dp.dtype == 0 ? __uint_as_float(o.g) : bf16_bits_to_f32(o.g);
    if (SRC == kSrcOne || SRC == kSrcTwo) {
        const uint32_t sh = (rel * (uint32_t)dp.bits) & 31u;
        const int q = __builtin_amdgcn_sbfe((int)o.c, sh, (uint32_t)dp.bits);
        const float step = o.s * dp.inv_s * omb;
        const float p1 = __builtin_fmaf(step, (float)q, g);
        if (SRC == kSrcOne) return p1;
        const int q2 = __builtin_amdgcn_sbfe((int)o.c2, sh, (uint32_t)dp.bits);
        return __builtin_fmaf(o.s2 * dp.inv_s, (float)q2, p1);
    }
    const float t = dp.table_dtype == 1 ? (float)__builtin_bit_cast(_Float16, (uint16_t)o.c) : __uint_as_float(o.c);
    return __builtin_fmaf(o.s, t, g);
}

// ------------------------------------------------------------------ P pass
// v_mfma_f64_4x4x4_4b_f64 for ranks up to 8 (RH = 1, 2 instructions per 16 x 4 operand) and v_mfma_f64_16x16x4_f64 above
// (RH = 4: one, RH = 8: two); the operand layouts are those of the octet family.  A[i][k] comes from the LDS tile of 32
// rows x 64 columns (pitch 68: the 64 lanes of a read fall on 64 banks), B[k][c] = Q[column k][c] straight from memory.
// Factor columns at or beyond the rank read a valid entry and are not stored; columns beyond the chunk are zero in the
// tile.
constexpr int kPPitch = 68;

constexpr int kPStripLds = 4 * kStripRows * kPPitch;      // floats

// lds: kPStripLds floats; `block`: index of the workgroup among those of this pass (in the other passes too)
template <int SRC, int RH>
__device__ __forceinline__ void p_strip(const KernelPlan &dp, int block, float *lds, const Source &src, const float *__restrict__ Q,
                                        float *P, double *ws)
{
    constexpr bool WIDE = RH >= 4;
    constexpr int BN = WIDE ? RH / 4 : RH, RC = 4 * RH;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *T = lds + wave * (kStripRows * kPPitch);
    const WorkItem it = dp.p_items[block];
    const MatDesc d = dp.mats[it.mat];
    const int r = dp.rank;
    const int64_t row0 = it.a;
    const int c_begin = it.b * d.p_chunk_cols;
    const int c_end = chunk_end(d.m, d.p_chunk_cols, c_begin);
    const int mi = lane & 15, mk = lane >> 4, mc = lane & 3;
    double acc[2][WIDE ? 1 : RH];
    f64x4 accw[2][WIDE ? BN : 1];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int h = 0; h < (WIDE ? 1 : RH); ++h) acc[t][h] = 0.0;
#pragma unroll
        for (int h = 0; h < (WIDE ? BN : 1); ++h) accw[t][h] = f64x4{0.0, 0.0, 0.0, 0.0};
    }
    // factor columns of this lane's B entries
    int bc[BN];
#pragma unroll
    for (int h = 0; h < BN; ++h) {
        const int c = WIDE ? mi + 16 * h : mc + 4 * h;
        bc[h] = c < r ? c : r - 1;
    }
    const int n_strips = (c_end - c_begin + 63) >> 6;
    const int rows = it.c;
    uint32_t rel0;
    const Base<SRC> base = make_base<SRC>(dp, d, src, row0 * d.m + c_begin, &rel0);
    for (int s = wave; s < n_strips; s += 4) {
        const int col0 = c_begin + 64 * s;
        const int ncol = (c_end - col0 < 64) ? c_end - col0 : 64;
        const uint32_t lc = (uint32_t)(lane < ncol ? lane : ncol - 1);
        const int32_t hv_col = SRC == kSrcCol ? dp.row_hash[d.hash_off + col0 + lc] : 0;
        float bq[16][BN];
        const float *qbase = Q + d.q_off + (int64_t)col0 * r;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int k = 4 * j + mk < ncol ? 4 * j + mk : ncol - 1;
#pragma unroll
            for (int h = 0; h < BN; ++h) bq[j][h] = qbase[(uint32_t)(k * r + bc[h])];
        }
        if (ncol & 3) {                                         // uniform; zero, so that 0 x inf does not reach a sum
#pragma unroll
            for (int j = 0; j < 16; ++j)
#pragma unroll
                for (int h = 0; h < BN; ++h) bq[j][h] = 4 * j + mk < ncol ? bq[j][h] : 0.0f;
        }
        const uint32_t rel_s = rel0 + 64u * (uint32_t)s + lc;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint32_t rel[16];
            int64_t row[16];
            Raw<SRC> o[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {                      // rows beyond the item re-read its last one (not stored)
                const int rr = 16 * half + u < rows ? 16 * half + u : rows - 1;
                rel[u] = rel_s + (uint32_t)rr * (uint32_t)d.m;
                row[u] = row0 + rr;
            }
            load_rows<SRC, 16>(dp, d, src, base, rel, row, col0, lc, hv_col, o);
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const float p = form_p<SRC>(dp, o[u], rel[u], dp.omb);
                T[(16 * half + u) * kPPitch + lane] = lane < ncol ? p : 0.0f;
            }
        }
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if (4 * j < ncol) {                                 // uniform
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const double a = (double)T[(16 * t + mi) * kPPitch + 4 * j + mk];
#pragma unroll
                    for (int h = 0; h < BN; ++h) {
                        if (WIDE) accw[t][h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)bq[j][h], accw[t][h], 0, 0, 0);
                        else acc[t][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, (double)bq[j][h], acc[t][h], 0, 0, 0);
                    }
                }
            }
        }
        wave_lds_sync();
    }
    __syncthreads();
    double *red = reinterpret_cast<double *>(lds);      // [wave][row][factor column]
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        if (WIDE) {
#pragma unroll
            for (int h = 0; h < BN; ++h)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[(wave * kStripRows + 16 * t + 4 * v + mk) * RC + 16 * h + mi] = accw[t][h][v];
        } else {
#pragma unroll
            for (int h = 0; h < BN; ++h) red[(wave * kStripRows + 16 * t + 4 * (mi >> 2) + mk) * RC + mc + 4 * h] = acc[t][h];
        }
    }
    __syncthreads();
    for (int idx = tid; idx < kStripRows * RC; idx += 256) {
        const int rr = idx / RC, c = idx % RC;
        const int64_t row = row0 + rr;
        if (c < r && rr < rows) {
            double sum = red[idx];
#pragma unroll
            for (int w = 1; w < 4; ++w) sum += red[w * kStripRows * RC + idx];
            if (d.n_p_chunks == 1) P[d.p_off + row * r + c] = (float)sum;
            else ws[d.ppart_off + ((int64_t)it.b * d.n + row) * r + c] = sum;
        }
    }
}

// A factor row at a wave-uniform address (scalar loads); entries at or beyond the rank are zero.  A rank that is not R takes its
// whole groups of four as one load each: entry by entry they were most of the err pass (10000 x 650 at rank 24: 102 -> 54 us, 600 x
// 5000 at rank 12 36 -> 25).
template <int R, bool EXACT>
__device__ __forceinline__ void uniform_row(const float *__restrict__ F, int r, float (&out)[R])
{
#pragma unroll
    for (int c0 = 0; c0 < R; c0 += 4) {
        constexpr int G = R < 4 ? R : 4;
        if (EXACT || c0 + G <= r) {                     // uniform: four entries in one load
#pragma unroll
            for (int c = c0; c < c0 + G; ++c) out[c] = F[c];
        } else {
#pragma unroll
            for (int c = c0; c < c0 + G; ++c) out[c] = c < r ? F[c < r ? c : r - 1] : 0.0f;
        }
    }
}

// ------------------------------------------------------------------ Q+ pass
// R: the rank (EXACT) or the next of 4, 8, 16, 32 (the sums beyond the rank stay zero).  Eight rows per trip, the next
// trip's loads ahead of the current one's arithmetic.  The four waves' sums are added as (0 + 2) + (1 + 3); a matrix with
// a single row tile gets its Q+ from here.
// red: LDS, 2 * R * 64 doubles
template <int SRC, int R, bool EXACT>
__device__ __forceinline__ void q_strip(const KernelPlan &dp, int block, double *red, const Source &src, const float *__restrict__ Phat,
                                        double *ws, float *Qout)
{
    constexpr int U = 8, kHalf = R * 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WorkItem it = dp.q_items[block];
    const MatDesc d = dp.mats[it.mat];
    const int r = EXACT ? R : dp.rank;
    const int64_t col0 = (int64_t)it.a * 64;
    const int ncol = (int)((d.m - col0 < 64) ? d.m - col0 : 64);
    const uint32_t lc = (uint32_t)(lane < ncol ? lane : ncol - 1);
    const int64_t t0 = (int64_t)it.b * d.q_tile_rows + (int64_t)wave * (d.q_tile_rows >> 2);
    const int64_t t1 = (t0 + (d.q_tile_rows >> 2) < d.n) ? t0 + (d.q_tile_rows >> 2) : d.n;
    const int32_t hv_col = SRC == kSrcCol ? dp.row_hash[d.hash_off + col0 + lc] : 0;
    double acc[R];
#pragma unroll
    for (int c = 0; c < R; ++c) acc[c] = 0.0;
    if (t0 < t1) {
        uint32_t rel0;
        const Base<SRC> base = make_base<SRC>(dp, d, src, t0 * d.m + col0, &rel0);
        rel0 += lc;
        Raw<SRC> cur[U];
        const int rows = (int)(t1 - t0);
        auto rel_of = [&](int i) { return rel0 + (uint32_t)(i < rows ? i : rows - 1) * (uint32_t)d.m; };
        auto load_trip = [&](Raw<SRC> (&o)[U], int i0) {
            uint32_t rel[U];
            int64_t row[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                rel[u] = rel_of(i0 + u);
                row[u] = t0 + (i0 + u < rows ? i0 + u : rows - 1);
            }
            load_rows<SRC, U>(dp, d, src, base, rel, row, col0, lc, hv_col, o);
        };
        load_trip(cur, 0);
        for (int i0 = 0; i0 < rows; i0 += U) {
            float p[U];
#pragma unroll
            for (int u = 0; u < U; ++u) p[u] = form_p<SRC>(dp, cur[u], rel_of(i0 + u), dp.omb);
            load_trip(cur, i0 + U < rows ? i0 + U : i0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u < rows) {                            // uniform
                    float ph[R];
                    uniform_row<R, EXACT>(Phat + d.p_off + (t0 + i0 + u) * r, r, ph);
                    const double pd = (double)p[u];
#pragma unroll
                    for (int c = 0; c < R; ++c) acc[c] = __builtin_fma(pd, (double)ph[c], acc[c]);
                }
            }
        }
    }
    if (wave >= 2) {
#pragma unroll
        for (int c = 0; c < R; ++c) red[(wave - 2) * kHalf + c * 64 + lane] = acc[c];
    }
    __syncthreads();
    if (wave < 2) {
#pragma unroll
        for (int c = 0; c < R; ++c) acc[c] += red[wave * kHalf + c * 64 + lane];
    }
    if (wave == 1) {
#pragma unroll
        for (int c = 0; c < R; ++c) red[kHalf + c * 64 + lane] = acc[c];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int c = 0; c < R; ++c) red[c * 64 + lane] = acc[c] + red[kHalf + c * 64 + lane];
    }
    __syncthreads();
    // the strip's rows of Q+ are contiguous
    const int64_t e0 = col0 * r;
    for (int e = tid; e < ncol * r; e += 256) {
        const double v = red[(e % r) * 64 + e / r];
        if (d.n_q_tiles == 1) Qout[d.q_off + e0 + e] = (float)v;
        else ws[d.qpart_off + (int64_t)it.b * d.m * r + e0 + e] = v;
    }
}

// Matrices of up to kFlatRows rows: a strip per wave, which has all rows (item: four strips).  In q_strip three waves of four
// have no rows then, and a trip repeats what rows there are: 1 x 1000000, rank 1, 16.7 us (31 with two vectors) against 7.5
// here; a thread per column without strips took 11.9.
template <int SRC, int R, bool EXACT>
__device__ __forceinline__ void q_flat(const KernelPlan &dp, int block, const Source &src, const float *__restrict__ Phat, float *Qout)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const WorkItem it = dp.q_flat_items[block];
    const MatDesc d = dp.mats[it.mat];
    const int r = EXACT ? R : dp.rank;
    const int64_t col0 = ((int64_t)it.a * 4 + wave) * 64;
    if (col0 >= d.m) return;
    const int ncol = (int)((d.m - col0 < 64) ? d.m - col0 : 64);
    const uint32_t lc = (uint32_t)(lane < ncol ? lane : ncol - 1);
    const int32_t hv_col = SRC == kSrcCol ? dp.row_hash[d.hash_off + col0 + lc] : 0;
    uint32_t rel0;
    const Base<SRC> base = make_base<SRC>(dp, d, src, col0, &rel0);
    const int rows = (int)d.n;
    double acc[R];
#pragma unroll
    for (int c = 0; c < R; ++c) acc[c] = 0.0;
    for (int i0 = 0; i0 < rows; i0 += 2) {
        uint32_t rel[2];
        int64_t row[2];
        Raw<SRC> o[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            row[u] = i0 + u < rows ? i0 + u : rows - 1;
            rel[u] = rel0 + lc + (uint32_t)row[u] * (uint32_t)d.m;
        }
        load_rows<SRC, 2>(dp, d, src, base, rel, row, col0, lc, hv_col, o);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (i0 + u < rows) {                                // uniform
                float ph[R];
                uniform_row<R, EXACT>(Phat + d.p_off + (i0 + u) * r, r, ph);
                const double pd = (double)form_p<SRC>(dp, o[u], rel[u], dp.omb);
#pragma unroll
                for (int c = 0; c < R; ++c) acc[c] = __builtin_fma(pd, (double)ph[c], acc[c]);
            }
        }
    }
    if (lane < ncol) {
        float *out = Qout + d.q_off + (col0 + lane) * r;
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (EXACT || c < r) out[c] = (float)acc[c];
    }
}

// ------------------------------------------------------------------ err pass
// The workgroup's run of scale blocks is either a piece of the flat index (d.es_seg == 0: es_tile elements from
// it.a * es_tile on, spanning it.c rows from row it.b), or, for matrices too wide for several rows to fit into LDS, for
// each of it.c rows from row it.a the blocks that START in the columns of segment it.b; these may reach past the segment
// by less than a block, into the next row after the last segment ("virtual" columns m, m + 1, ...).  Either way a row
// has a window [lo, hi) of (virtual) columns and its residuals lie in LDS in the order of the flat index.
// A matrix of up to 32 columns (GROUP) is walked in groups of es_rows rows that fill a wave, as if a group were a row; a lane
// then has a row of P^ of its own.  One row per access left the lanes empty: 4096 x 9 at rank 4 21 us, 100000 x 1 140; 7.6 and
// 7.6 in groups (7.5 and 7.3 with the kernel for any block, a lane per element, which needs 84 for 200000 x 12 where groups
// take 11).  Launched apart from the other strips: both in one kernel cost those 5 - 10 %.
//
// Three parts with barriers between them: p into LDS in octets; the reconstruction subtracted there; octets rounded and packed
// (every code of the run has been read by then).
template <int BITS, bool TWO>
__device__ __forceinline__ void quantise_run(const KernelPlan &dp, const MatDesc &d, int mat, uint32_t step_lo, uint32_t step_hi,
                                             const float *X, int64_t flat0, int count, int slots, int first, int stride,
                                             uint32_t *codes, float *scales, uint32_t *codes2, float *scales2)
{
    const int lane = threadIdx.x & 63;
    const int lb = dp.lb_shift;
    const float s_f = (float)((1 << (BITS - 1)) - 1);
    // octet `id` of the run: elements flat0 + 8 id .. + 7 of the matrix, `count` elements in all
    for (int base = first; base < slots; base += stride) {          // uniform
        const int id = base + lane, pos = 8 * id;
        float x[8];
        const bool any = pos < count;
        {
            const float4 *xp = reinterpret_cast<const float4 *>(X + (any ? pos : 0));
            const float4 a = xp[0], b = xp[1];
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        }
        if (pos + 8 > count) {                                      // the short last block of the matrix, or nothing
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = pos + e < count ? x[e] : 0.0f;
        }
        const int64_t o = (flat0 >> 3) + id;
        auto round_octet = [&](uint32_t mat_word, uint32_t *cw, float *sc, int32_t (&t)[8]) {
            const float a = block_max(abs_max_octet(0.0f, x), lb);
            const float inv16 = levels_over(a, s_f);
            uint32_t rnd[4];
            philox4x32_10((uint32_t)o, mat_word, step_lo, step_hi, dp.seed_lo, dp.seed_hi, rnd);
            uint32_t w[2];
            quantise_octet<BITS>(x, inv16, rnd, w, t);
            if (any) {
                uint32_t *wp = cw + d.word_off;
                if (BITS == 8) {
                    wp[2 * o] = w[0];
                    if (pos + 4 < count) wp[2 * o + 1] = w[1];
                } else if (BITS == 4) {
                    wp[o] = w[0];
                } else {
                    if (pos + 8 >= count && (o & 1) == 0) wp[o >> 1] = w[0];      // the last word of the run is half used
                    else reinterpret_cast<uint16_t *>(wp)[o] = (uint16_t)w[0];
                }
                if ((id & ((1 << lb) - 1)) == 0) sc[d.scale_off + (o >> lb)] = a;
            }
            return a;
        };
        int32_t t[8];
        const float a = round_octet((uint32_t)mat, codes, scales, t);
        if (TWO) {
            const float dnew = a * inv_levels(BITS);
            float qn[8];
            rounded_values(t, qn);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = x[e] - dnew * qn[e];
            round_octet((uint32_t)mat | 0x80000000u, codes2, scales2, t);
        }
    }
}

// codes / scales: the error vector that is replaced (TWO: the first one, also in the plan); codes2 / scales2: TWO only,
// the second
// X: LDS, dp.es_lds floats
// GROUP: the matrix is walked in groups of rows (it has no segments)
template <int R, bool EXACT, bool TWO, bool GROUP>
__device__ __forceinline__ void err_strip(const KernelPlan &dp, int block, float *X, const void *__restrict__ grads, uint32_t *codes,
                                          float *scales, uint32_t *codes2, float *scales2, const float *__restrict__ Phat,
                                          const float *__restrict__ Qn, uint32_t step_lo, uint32_t step_hi)
{
    constexpr int U = 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WorkItem it = GROUP ? dp.err_g_items[block] : dp.err_s_items[block];
    const MatDesc d = dp.mats[it.mat];
    const int r = EXACT ? R : dp.rank;
    const int64_t B = dp.block;
    const bool seg = !GROUP && d.es_seg != 0;
    const int64_t j0 = seg ? 0 : (int64_t)it.a * d.es_tile;
    const int64_t j1 = seg ? 0 : (j0 + d.es_tile < d.N ? j0 + d.es_tile : d.N);
    const int64_t i_first = seg ? it.a : it.b;
    const int n_rows = it.c;
    const int64_t M = GROUP ? d.m * d.es_rows : d.m;            // GROUP: below, a row is a group of them
    const int lane_row = GROUP ? lane / (int)d.m : 0, lane_col = GROUP ? lane - lane_row * (int)d.m : lane;
    const int64_t c0 = seg ? (int64_t)it.b * d.es_seg : 0;
    const int64_t c1 = seg ? (c0 + d.es_seg < d.m ? c0 + d.es_seg : d.m) : M;
    // (virtual) columns: [c0, c0 + width)
    const int width = (int)(c1 - c0) + (seg ? d.es_over : 0);

    // All indices are relative to the first owned block of the run (its first element: jb); row rl of the run owns the
    // elements [ws, we) and its (virtual) column 64 st + lane is element rel_row(rl) + 64 st + lane.
    const int64_t f0 = i_first * M + c0;
    const int64_t jb = seg ? ((f0 + B - 1) & ~(B - 1)) : j0;
    const int rel_f0 = (int)(f0 - jb);                          // (negative: the run's first row starts before its first block)
    auto rel_row = [&](int rl) { return rel_f0 + rl * (int)M; };
    const int last = (int)(seg ? (d.N - jb < INT32_MAX ? d.N - jb : INT32_MAX) : j1 - jb);
    auto window = [&](int rl, int &ws, int &we) {
        const int f = rel_row(rl);
        if (seg) {
            ws = (f + (int)B - 1) & ~((int)B - 1);
            we = (f + (int)(c1 - c0) + (int)B - 1) & ~((int)B - 1);
        } else {
            ws = f > 0 ? f : 0;
            we = f + (int)M;
        }
        we = we < last ? we : last;
    };
    // First part: p of the run, octet by octet (the run's pieces start at scale blocks, so these are aligned and whole, up to
    // the last one of the matrix).
    auto fill = [&](auto bf_tag, auto bits_tag) {
        constexpr bool BF16 = decltype(bf_tag)::value;
        constexpr int BITS = decltype(bits_tag)::value, NB = 4;
        const OctetBase<BF16, BITS, TWO> base = octet_base<BF16, BITS, TWO>(dp, d, grads, TWO ? codes2 : codes, TWO ? scales2 : scales, jb >> 3);
        // groups of 64 octets from first, first + stride, ... on below n_oct of the piece that starts at the base's octet o0 and goes to
        // `to`.  A group that is not there is not asked for: rows of a segment are one to three groups, and repeating the last octet
        // in their place cost 40 x 1300 at rank 4 7.6 us for the pass, 6.6 so, and 600 x 5000 14.3, 13.2.
        auto piece = [&](int o0, int n_oct, float *to, int first, int stride) {
            for (int at = first; at < n_oct; at += NB * stride) {        // uniform
                OctetRegs<BF16, BITS, TWO> o[NB];
                int id[NB];
#pragma unroll
                for (int u = 0; u < NB; ++u) {                  // (beyond the piece: its last one again, with what it holds)
                    id[u] = at + u * stride + lane < n_oct ? at + u * stride + lane : n_oct - 1;
                    if (u == 0 || at + u * stride < n_oct) load_octet_at<BF16, BITS, TWO>(base, (uint32_t)(o0 + id[u]), o[u]);
                }
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    if (u > 0 && at + u * stride >= n_oct) break;
                    float x[8];
                    decode_octet_at<BF16, BITS, TWO>(o[u], 1.0f, x);
                    float4 *dst = reinterpret_cast<float4 *>(to + 8 * id[u]);
                    dst[0] = make_float4(x[0], x[1], x[2], x[3]);
                    dst[1] = make_float4(x[4], x[5], x[6], x[7]);
                }
            }
        };
        if (!seg) {
            piece(0, ((int)(j1 - j0) + 7) >> 3, X, 64 * wave, 256);
        } else {
            for (int rl = wave; rl < n_rows; rl += 4) {
                int ws, we;
                window(rl, ws, we);
                piece(ws >> 3, (we - ws + 7) >> 3, X + rl * d.es_pitch, 0, 64);
            }
        }
    };
    auto fill_bits = [&](auto bf_tag) {
        if (dp.bits == 4) fill(bf_tag, std::integral_constant<int, 4>{});
        else if (dp.bits == 2) fill(bf_tag, std::integral_constant<int, 2>{});
        else fill(bf_tag, std::integral_constant<int, 8>{});
    };
    if (dp.dtype == 0) fill_bits(std::false_type{});
    else fill_bits(std::true_type{});
    __syncthreads();

    // Second part: the reconstruction is subtracted, in units of four rows x one strip, each wave a contiguous quarter of the
    // units in strip-major order.  Per row of the run: own are the lanes lo <= 64 st + lane < hi, and that lane's residual lies
    // at X[base + 64 st + lane].
    struct Row {
        int lo, hi, base;
    };
    const int n_strips = (width + 63) >> 6, n_groups = (n_rows + U - 1) / U;
    const int n_units = n_strips * n_groups;
    const int u_begin = (int)((int64_t)n_units * wave / 4), u_end = (int)((int64_t)n_units * (wave + 1) / 4);
    const float *prun = Phat + d.p_off + (GROUP ? 0 : i_first * r);
    auto subtract = [&](auto seg_tag) {
        constexpr bool SEG = decltype(seg_tag)::value;
        auto row_at = [&](int rl) {
            Row w;
            const int f = rel_row(rl);
            if (SEG) {
                const int ws = (f + (int)B - 1) & ~((int)B - 1), we = (f + (int)(c1 - c0) + (int)B - 1) & ~((int)B - 1);
                w.lo = ws - f;
                w.hi = (we < last ? we : last) - f;
                w.base = rl * d.es_pitch - w.lo;
            } else {
                w.lo = f < 0 ? -f : 0;
                w.hi = last - f < (int)M ? last - f : (int)M;
                w.base = f;
            }
            return w;
        };
        int strip = n_groups > 0 ? u_begin / n_groups : 0, group = u_begin - strip * n_groups;
        float q[R];
#pragma unroll
        for (int c = 0; c < R; ++c) q[c] = 0.0f;
        int q_strip = -1;
        for (int un = u_begin; un < u_end; ++un) {
            const int v0 = 64 * strip, v = v0 + lane;               // the lane's column in the run (SEG: from c0 on)
            if (strip != q_strip) {                                 // uniform
                q_strip = strip;
                const uint32_t k = virtual_column((uint32_t)d.m, (uint32_t)c0, (uint32_t)(GROUP ? lane_col : v));
                const float *qrow = Qn + d.q_off + (int64_t)k * r;
                if (EXACT && R >= 4) {
#pragma unroll
                    for (int c4 = 0; c4 < R / 4; ++c4) {
                        const float4 w = reinterpret_cast<const float4 *>(qrow)[c4];
                        q[4 * c4] = w.x; q[4 * c4 + 1] = w.y; q[4 * c4 + 2] = w.z; q[4 * c4 + 3] = w.w;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < R; ++c)
                        if (EXACT || c < r) q[c] = qrow[c];
                }
            }
            const int rl0 = group * U;
            // UB rows at a time: their rows of P^ and their p are asked for together, so that a group costs one round trip to
            // LDS and the scalar cache
            constexpr int UB = R <= 8 ? U : R <= 16 ? 2 : 1;
#pragma unroll
            for (int u0 = 0; u0 < U; u0 += UB) {
                if (rl0 + u0 >= n_rows) break;                      // uniform
                const bool wraps = SEG && c0 + v0 + 63 >= d.m;      // uniform: some lanes may belong to the next row
                const int f0 = rel_row(rl0 + u0);
                Row w[UB];
                bool whole = !GROUP && !wraps && rl0 + u0 + UB <= n_rows;      // uniform: every lane of every row is its owner
                if (SEG) {
#pragma unroll
                    for (int u = 0; u < UB; ++u) {
                        w[u] = row_at(rl0 + u0 + u);
                        whole = whole && w[u].lo <= v0 && v0 + 64 <= w[u].hi;
                    }
                } else {
                    whole = whole && f0 >= 0 && f0 + UB * (int)M <= last && v0 + 64 <= (int)M;
                }
                float x[UB], acc[UB];
                if (whole) {
                    int at[UB];
#pragma unroll
                    for (int u = 0; u < UB; ++u) at[u] = (SEG ? w[u].base : f0 + u * (int)M) + v;
                    float ph[UB][R];
                    const float *prow = prun + (uint32_t)((rl0 + u0) * r);
#pragma unroll
                    for (int u = 0; u < UB; ++u) uniform_row<R, EXACT>(prow + u * r, r, ph[u]);
#pragma unroll
                    for (int u = 0; u < UB; ++u) {
                        x[u] = X[(uint32_t)at[u]];
                        acc[u] = 0.0f;
                    }
#pragma unroll
                    for (int c = 0; c < R; ++c)
#pragma unroll
                        for (int u = 0; u < UB; ++u) acc[u] = __builtin_fmaf(ph[u][c], q[c], acc[u]);
#pragma unroll
                    for (int u = 0; u < UB; ++u) X[(uint32_t)at[u]] = x[u] - acc[u];
                    continue;
                }
                // rows beyond the run repeat its last one and store nothing
                constexpr int RL = GROUP && R <= 8 ? R : 1;
                float pl[UB][RL];                                   // GROUP: the lanes' rows of P^
                bool own[UB];
                auto lane_p = [&](int u) {
                    const int rl = rl0 + u0 + u < n_rows ? rl0 + u0 + u : n_rows - 1;
                    const int64_t i = (i_first + rl) * d.es_rows + lane_row;
                    return prun + (i < d.n ? i : d.n - 1) * r;
                };
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    if (!SEG) w[u] = row_at(rl0 + u0 + u);
                    own[u] = rl0 + u0 + u < n_rows && v >= w[u].lo && v < w[u].hi;
                    x[u] = X[own[u] ? (uint32_t)(w[u].base + v) : 0u];
                    acc[u] = 0.0f;
                    if (GROUP && R <= 8) {
                        const float *prow = lane_p(u);
#pragma unroll
                        for (int c = 0; c < RL; ++c) pl[u][c] = prow[EXACT ? c : (c < r ? c : r - 1)];
                    }
                }
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    if (GROUP) {
                        const float *prow = lane_p(u);
#pragma unroll
                        for (int c = 0; c < R; ++c)
                            if (EXACT || c < r) acc[u] = __builtin_fmaf(R <= 8 ? pl[u][R <= 8 && GROUP ? c : 0] : prow[c], q[c], acc[u]);
                    } else {
                        const int rl = rl0 + u0 + u < n_rows ? rl0 + u0 + u : n_rows - 1;
                        float ph[R];
                        uniform_row<R, EXACT>(prun + (uint32_t)(rl * r), r, ph);
                        if (!wraps) {
#pragma unroll
                            for (int c = 0; c < R; ++c) acc[u] = __builtin_fmaf(ph[c], q[c], acc[u]);
                        } else {
                            float pn[R];
                            uniform_row<R, EXACT>(prun + (uint32_t)((i_first + rl + 1 < d.n ? rl + 1 : rl) * r), r, pn);
#pragma unroll
                            for (int c = 0; c < R; ++c) acc[u] = __builtin_fmaf(c0 + v < d.m ? ph[c] : pn[c], q[c], acc[u]);
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < UB; ++u)
                    if (own[u]) X[(uint32_t)(w[u].base + v)] = x[u] - acc[u];
            }
            if (++group == n_groups) { group = 0; ++strip; }
        }
    };
    if (!GROUP && seg) subtract(std::integral_constant<bool, !GROUP>{});
    else subtract(std::false_type{});
    __syncthreads();
    auto quantise = [&](auto bits_tag) {
        constexpr int BITS = decltype(bits_tag)::value;
        if (!seg) {
            const int count = (int)(j1 - j0);
            quantise_run<BITS, TWO>(dp, d, it.mat, step_lo, step_hi, X, j0, count, (count + 7) >> 3, 64 * wave, 256, codes, scales,
                                    codes2, scales2);
        } else {
            for (int rl = wave; rl < n_rows; rl += 4) {
                int ws, we;
                window(rl, ws, we);
                const int count = we - ws;
                quantise_run<BITS, TWO>(dp, d, it.mat, step_lo, step_hi, X + rl * d.es_pitch, jb + ws, count,
                                        (count + 7) >> 3, 0, 64, codes, scales, codes2, scales2);
            }
        }
    };
    if (dp.bits == 4) quantise(std::integral_constant<int, 4>{});
    else if (dp.bits == 2) quantise(std::integral_constant<int, 2>{});
    else quantise(std::integral_constant<int, 8>{});
}

}  // namespace

}  // namespace conef
