// Device code of the strip family's P and Q+ passes on octets (see kernels_ragged.hip), for its own launches and for those
// that carry the octet family's workgroups too (kernels_mixed.hip); and the octets' loads, which its err pass shares.
#pragma once
#include "device_common.h"
#include "kernels.h"
#include "octet_device.h"

namespace conef {

namespace {

// A scalar base at an octet of a matrix, and octets by their 32-bit distance from it (a byte offset stays below 2^32: the
// plan keeps the rows that share a base within 2^29 elements).  TWO: codes / scales are the second vector, the first is the
// plan's; octets are decoded in that order.
template <bool BF16, int BITS, bool TWO>
struct OctetBase {
    const uint8_t *g, *c, *c2;
    const float *s, *s2;
    uint32_t rem;               // octets between the start of the base's scale block and the base
    int lb;                     // log2(octets per scale block)
};

template <bool BF16, int BITS, bool TWO>
struct OctetRegs {
    RawOctet<BF16, BITS> o;
    RawCodes<BITS> o2;          // TWO
};

template <bool BF16, int BITS, bool TWO>
__device__ __forceinline__ OctetBase<BF16, BITS, TWO> octet_base(const KernelPlan &dp, const MatDesc &d, const void *grads,
                                                                 const uint32_t *codes, const float *scales, int64_t oct)
{
    OctetBase<BF16, BITS, TWO> b;
    b.lb = dp.lb_shift;
    b.rem = (uint32_t)oct & ((1u << b.lb) - 1u);
    b.g = reinterpret_cast<const uint8_t *>(grads) + (d.grad_off + oct * 8) * (BF16 ? 2 : 4);
    b.c = reinterpret_cast<const uint8_t *>((TWO ? dp.i_codes : codes) + d.word_off) + oct * BITS;
    b.s = (TWO ? dp.i_scales : scales) + d.scale_off + (oct >> b.lb);
    b.c2 = TWO ? reinterpret_cast<const uint8_t *>(codes + d.word_off) + oct * BITS : nullptr;
    b.s2 = TWO ? scales + d.scale_off + (oct >> b.lb) : nullptr;
    return b;
}

template <int BITS>
__device__ __forceinline__ void load_octet_codes(const uint8_t *c, uint32_t o, uint32_t &c0, uint32_t &c1)
{
    c1 = 0;
    if (BITS == 8) {
        const uint2 v = *reinterpret_cast<const uint2 *>(c + o * 8u);
        c0 = v.x; c1 = v.y;
    } else if (BITS == 4) {
        c0 = *reinterpret_cast<const uint32_t *>(c + o * 4u);
    } else {
        c0 = *reinterpret_cast<const uint16_t *>(c + o * 2u);
    }
}

template <bool BF16, int BITS, bool TWO>
__device__ __forceinline__ void load_octet_at(const OctetBase<BF16, BITS, TWO> &b, uint32_t o, OctetRegs<BF16, BITS, TWO> &r)
{
    r.o.g1 = make_uint4(0, 0, 0, 0);
    if (BF16) {
        r.o.g0 = *reinterpret_cast<const uint4 *>(b.g + o * 16u);
    } else {
        const uint4 *gp = reinterpret_cast<const uint4 *>(b.g + o * 32u);
        r.o.g0 = gp[0];
        r.o.g1 = gp[1];
    }
    load_octet_codes<BITS>(b.c, o, r.o.c0, r.o.c1);
    r.o.scale = b.s[(b.rem + o) >> b.lb];
    if (TWO) {
        load_octet_codes<BITS>(b.c2, o, r.o2.c0, r.o2.c1);
        r.o2.scale = b.s2[(b.rem + o) >> b.lb];
    }
}

template <bool BF16, int BITS, bool TWO>
__device__ __forceinline__ void decode_octet_at(const OctetRegs<BF16, BITS, TWO> &r, float omb, float p[8])
{
    decode_octet<BF16, BITS>(r.o, omb, p);
    if (TWO) add_codes<BITS>(r.o2, p);
}

// ------------------------------------------------------------------ a wave's tile
// 32 rows x 64 columns of p in LDS, for rows that start anywhere in an octet.  Row i of the tile holds the (up to) nine whole
// octets that its 64 columns lie in, so that loads and stores are aligned pieces of 16 bytes whatever the row length; its first
// column stands sh = (flat index of that element) mod 8 floats into the row.  The 32 x 9 octets are dealt to the lanes in
// turn, five to a lane; which ones does not change along the rows or (for steps of a multiple of 8 rows) down the columns.
// Pitch 76: without the shifts the 16 rows x 4 columns of an operand read fall on 64 banks.  Row 32 takes the octets dealt
// to nobody.
constexpr int kRagPitch = 76, kRagOcts = 5;
constexpr int kRagTile = (kStripRows + 1) * kRagPitch;      // floats
constexpr int kRagLds = 4 * kRagTile;

struct RagLanes {
    uint32_t oct[kRagOcts];     // the lane's octets, from the octet of the tile's first element on
    uint32_t dst[kRagOcts];     // where they go (floats)
    uint32_t row[kRagOcts];
};

// sh0: the first element's place in its octet; rows: of the tile; ncol: columns of the widest strip
__device__ __forceinline__ RagLanes rag_lanes(int lane, uint32_t sh0, int rows, int64_t m, int ncol)
{
    RagLanes r;
    const uint32_t so = (uint32_t)(ncol + 14) >> 3;             // octets per row: at most 9
#pragma unroll
    for (int p = 0; p < kRagOcts; ++p) {
        const uint32_t idx = (uint32_t)(lane + 64 * p);
        const uint32_t row = idx / so, oc = idx - row * so;
        const uint32_t rc = row < (uint32_t)rows ? row : (uint32_t)rows - 1;
        r.row[p] = row;
        r.oct[p] = ((sh0 + rc * (uint32_t)m) >> 3) + oc;
        r.dst[p] = (row < (uint32_t)kStripRows ? row : (uint32_t)kStripRows) * kRagPitch + 8u * (row < (uint32_t)kStripRows ? oc : 0u);
    }
    return r;
}

// ------------------------------------------------------------------ P pass
// As p_strip: a workgroup per (32 rows, column chunk), its waves take the chunk's strips of 64 columns in turn, fp64 matrix
// cores, the four waves' sums added in wave order.  Bound by the loads in flight and the vector ALU together: an element costs
// an eighth of an octet's loads, addresses and decode, where p_strip loads a gradient, a code word and a scale for each.
// lds: kRagLds floats; `block`: index of the workgroup among those of this pass
template <bool BF16, int BITS, int RH, bool TWO>
__device__ __forceinline__ void p_ragged(const KernelPlan &dp, int block, float *lds, const void *__restrict__ grads,
                                         const uint32_t *__restrict__ codes, const float *__restrict__ scales,
                                         const float *__restrict__ Q, float *P, double *ws)
{
    typedef double dx4 __attribute__((ext_vector_type(4)));
    constexpr bool WIDE = RH >= 4;
    constexpr int BN = WIDE ? RH / 4 : RH, RC = 4 * RH;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *T = lds + wave * kRagTile;
    const WorkItem it = dp.p_items[block];
    const MatDesc d = dp.mats[it.mat];
    const int r = dp.rank;
    const int64_t row0 = it.a;
    const int rows = it.c;
    const int c_begin = it.b * d.p_chunk_cols;
    const int c_end = chunk_end(d.m, d.p_chunk_cols, c_begin);
    const int mi = lane & 15, mk = lane >> 4, mc = lane & 3;
    double acc[2][WIDE ? 1 : RH];
    dx4 accw[2][WIDE ? BN : 1];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int h = 0; h < (WIDE ? 1 : RH); ++h) acc[t][h] = 0.0;
#pragma unroll
        for (int h = 0; h < (WIDE ? BN : 1); ++h) accw[t][h] = dx4{0.0, 0.0, 0.0, 0.0};
    }
    // factor columns of this lane's B entries (at or beyond the rank: a valid entry, whose results are not stored)
    int bc[BN];
#pragma unroll
    for (int h = 0; h < BN; ++h) {
        const int c = WIDE ? mi + 16 * h : mc + 4 * h;
        bc[h] = c < r ? c : r - 1;
    }
    const int n_strips = (c_end - c_begin + 63) >> 6;
    const int64_t f0 = row0 * d.m + c_begin;
    const uint32_t sh0 = (uint32_t)f0 & 7u;
    const OctetBase<BF16, BITS, TWO> base = octet_base<BF16, BITS, TWO>(dp, d, grads, codes, scales, f0 >> 3);
    const int64_t left = ((d.N - 1) >> 3) - (f0 >> 3);
    const uint32_t last = left < 0x0FFFFFFF ? (uint32_t)left : 0x0FFFFFFFu;        // octets beyond the matrix: its last one
    const RagLanes lanes = rag_lanes(lane, sh0, rows, d.m, c_end - c_begin < 64 ? c_end - c_begin : 64);
    uint32_t abase[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int rr = 16 * t + mi;
        abase[t] = (uint32_t)rr * kRagPitch + ((sh0 + (uint32_t)(rr < rows ? rr : rows - 1) * (uint32_t)d.m) & 7u) + (uint32_t)mk;
    }
    OctetRegs<BF16, BITS, TWO> o[kRagOcts];
    // (two values per lane and column group: no second set, whose registers cost a wave per SIMD)
    constexpr bool AHEAD = BN == 1;
    float bq[16][BN], bn[AHEAD ? 16 : 1][BN];
    auto load_data = [&](int s) {
#pragma unroll
        for (int p = 0; p < kRagOcts; ++p) {
            const uint32_t at = lanes.oct[p] + 8u * (uint32_t)s;
            load_octet_at<BF16, BITS, TWO>(base, at < last ? at : last, o[p]);
        }
    };
    // B operand: Q[column 4 j + mk of the strip][bc]; columns beyond the chunk re-read its last one (their A entries are zero)
    auto load_b = [&](auto &b, int s) {
        const int col0 = c_begin + 64 * s;
        const int ncol = c_end - col0 < 64 ? c_end - col0 : 64;
        const float *qbase = Q + d.q_off + (int64_t)col0 * r;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int k = 4 * j + mk < ncol ? 4 * j + mk : ncol - 1;
#pragma unroll
            for (int h = 0; h < BN; ++h) b[j][h] = qbase[(uint32_t)(k * r + bc[h])];
        }
    };
    if (wave < n_strips) {
        if (AHEAD) load_b(bq, wave);
        load_data(wave);
    }
    for (int s = wave; s < n_strips; s += 4) {
        const int ncol = c_end - (c_begin + 64 * s) < 64 ? c_end - (c_begin + 64 * s) : 64;
#pragma unroll
        for (int p = 0; p < kRagOcts; ++p) {
            float x[8];
            decode_octet_at<BF16, BITS, TWO>(o[p], dp.omb, x);
            float4 *dst = reinterpret_cast<float4 *>(T + lanes.dst[p]);
            dst[0] = make_float4(x[0], x[1], x[2], x[3]);
            dst[1] = make_float4(x[4], x[5], x[6], x[7]);
        }
        const int next = s + 4 < n_strips ? s + 4 : s;
        if constexpr (AHEAD) load_b(bn, next);
        else load_b(bq, s);
        load_data(next);
        wave_lds_sync();
        auto multiply = [&](auto ragged) {
            constexpr bool RAGGED = decltype(ragged)::value;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                if (!RAGGED || 4 * j < ncol) {                      // uniform
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        float v = T[abase[t] + 4 * j];
                        if (RAGGED) v = 4 * j + mk < ncol ? v : 0.0f;      // (what stands there belongs to the next row)
                        const double a = (double)v;
#pragma unroll
                        for (int h = 0; h < BN; ++h) {
                            const float bv = !RAGGED || 4 * j + mk < ncol ? bq[j][h] : 0.0f;
                            if (WIDE) accw[t][h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)bv, accw[t][h], 0, 0, 0);
                            else acc[t][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, (double)bv, acc[t][h], 0, 0, 0);
                        }
                    }
                }
            }
        };
        if (ncol == 64) multiply(std::false_type{});
        else multiply(std::true_type{});
        wave_lds_sync();
        if constexpr (AHEAD) {
#pragma unroll
            for (int j = 0; j < 16; ++j)
#pragma unroll
                for (int h = 0; h < BN; ++h) bq[j][h] = bn[j][h];
        }
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

// ------------------------------------------------------------------ Q+ pass
// A workgroup per (strip of 64 columns, row tile); its waves take the tile's 32-row steps in turn.  D[column][c] +=
// p[row][column] P^[row][c] on the fp64 matrix cores, whose A operand is read from the same tile of p as in the P pass; the
// four waves' sums are added as (0 + 2) + (1 + 3).  A matrix with a single row tile gets its Q+ from here.
// lds: kRagLds floats
template <bool BF16, int BITS, int RH, bool TWO>
__device__ __forceinline__ void q_ragged(const KernelPlan &dp, int block, float *lds, const void *__restrict__ grads,
                                         const uint32_t *__restrict__ codes, const float *__restrict__ scales,
                                         const float *__restrict__ Phat, double *ws, float *Qout)
{
    typedef double dx4 __attribute__((ext_vector_type(4)));
    constexpr bool WIDE = RH >= 4;
    constexpr int BN = WIDE ? RH / 4 : RH, RC = 4 * RH, kHalf = RC * 64, kGroups = kStripRows / 4;
    static_assert(2 * kHalf * 2 <= kRagLds, "two waves' sums fit into the tiles");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *T = lds + wave * kRagTile;
    const WorkItem it = dp.q_items[xcd_contiguous_item(block, dp.n_q)];
    const MatDesc d = dp.mats[it.mat];
    const int r = dp.rank;
    const int64_t col0 = (int64_t)it.a * 64;
    const int ncol = (int)((d.m - col0 < 64) ? d.m - col0 : 64);
    const int64_t t0 = (int64_t)it.b * d.q_tile_rows;
    const int64_t t1 = t0 + d.q_tile_rows < d.n ? t0 + d.q_tile_rows : d.n;
    const int mi = lane & 15, mk = lane >> 4, mc = lane & 3;
    double acc[4][WIDE ? 1 : RH];
    dx4 accw[4][WIDE ? BN : 1];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int h = 0; h < (WIDE ? 1 : RH); ++h) acc[t][h] = 0.0;
#pragma unroll
        for (int h = 0; h < (WIDE ? BN : 1); ++h) accw[t][h] = dx4{0.0, 0.0, 0.0, 0.0};
    }
    int bc[BN];
#pragma unroll
    for (int h = 0; h < BN; ++h) {
        const int c = WIDE ? mi + 16 * h : mc + 4 * h;
        bc[h] = c < r ? c : r - 1;
    }
    // steps start 32 rows apart: all of them have the first element at the same place of its octet
    const uint32_t sh0 = (uint32_t)(t0 * d.m + col0) & 7u;
    const RagLanes lanes = rag_lanes(lane, sh0, kStripRows, d.m, ncol);
    uint32_t abase[2];              // row 4 g + mk of the tile for even and odd g: rows 8 apart have the same shift
#pragma unroll
    for (int g = 0; g < 2; ++g) abase[g] = (uint32_t)(4 * g + mk) * kRagPitch + ((sh0 + (uint32_t)(4 * g + mk) * (uint32_t)d.m) & 7u) + (uint32_t)mi;
    struct Step {
        OctetRegs<BF16, BITS, TWO> o[kRagOcts];
        float ph[kGroups][BN];
    };
    // rows at or beyond the tile's end: some octet before it, and its last row of P^ (both replaced by zero)
    auto load_step = [&](Step &st, int64_t r0) {
        const OctetBase<BF16, BITS, TWO> base = octet_base<BF16, BITS, TWO>(dp, d, grads, codes, scales, (r0 * d.m + col0) >> 3);
        const int left = (int)(t1 - r0 < kStripRows ? t1 - r0 : kStripRows);
        const uint32_t last = (sh0 + (uint32_t)(left - 1) * (uint32_t)d.m + (uint32_t)ncol - 1u) >> 3;
#pragma unroll
        for (int p = 0; p < kRagOcts; ++p) load_octet_at<BF16, BITS, TWO>(base, lanes.oct[p] < last ? lanes.oct[p] : last, st.o[p]);
        const float *pbase = Phat + d.p_off + r0 * r;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int row = 4 * g + mk < left ? 4 * g + mk : left - 1;
#pragma unroll
            for (int h = 0; h < BN; ++h) st.ph[g][h] = pbase[(uint32_t)(row * r + bc[h])];
        }
    };
    Step cur;
    if (t0 + 32 * wave < t1) load_step(cur, t0 + 32 * wave);
    for (int64_t r0 = t0 + 32 * wave; r0 < t1; r0 += 128) {
        const int left = (int)(t1 - r0 < kStripRows ? t1 - r0 : kStripRows);
#pragma unroll
        for (int p = 0; p < kRagOcts; ++p) {
            float x[8];
            decode_octet_at<BF16, BITS, TWO>(cur.o[p], dp.omb, x);
            if (left < kStripRows) {                                // uniform
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = lanes.row[p] < (uint32_t)left ? x[e] : 0.0f;
            }
            float4 *dst = reinterpret_cast<float4 *>(T + lanes.dst[p]);
            dst[0] = make_float4(x[0], x[1], x[2], x[3]);
            dst[1] = make_float4(x[4], x[5], x[6], x[7]);
        }
        float b[kGroups][BN];
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
#pragma unroll
            for (int h = 0; h < BN; ++h) b[g][h] = left == kStripRows || 4 * g + mk < left ? cur.ph[g][h] : 0.0f;
        load_step(cur, r0 + 128 < t1 ? r0 + 128 : r0);
        wave_lds_sync();
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double a = (double)T[abase[g & 1] + (uint32_t)((g >> 1) * 8 * kRagPitch + 16 * t)];
#pragma unroll
                for (int h = 0; h < BN; ++h) {
                    if (WIDE) accw[t][h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)b[g][h], accw[t][h], 0, 0, 0);
                    else acc[t][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, (double)b[g][h], acc[t][h], 0, 0, 0);
                }
            }
        }
        wave_lds_sync();
    }
    // the lane's entries of D: column, factor column
    double *red = reinterpret_cast<double *>(lds);                  // [2][factor column][64]
    auto each = [&](auto &&f) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (WIDE) {
#pragma unroll
                for (int h = 0; h < BN; ++h)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        double x = accw[t][h][v];
                        f(x, (16 * h + mi) * 64 + 16 * t + 4 * v + mk);
                        accw[t][h][v] = x;
                    }
            } else {
#pragma unroll
                for (int h = 0; h < BN; ++h) f(acc[t][h], (mc + 4 * h) * 64 + 16 * t + 4 * (mi >> 2) + mk);
            }
        }
    };
    __syncthreads();
    if (wave >= 2) each([&](double &x, int at) { red[(wave - 2) * kHalf + at] = x; });
    __syncthreads();
    if (wave < 2) each([&](double &x, int at) { x += red[wave * kHalf + at]; });
    if (wave == 1) each([&](double &x, int at) { red[kHalf + at] = x; });
    __syncthreads();
    if (wave == 0) each([&](double &x, int at) { red[at] = x + red[kHalf + at]; });
    __syncthreads();
    // the strip's rows of Q+ are contiguous
    const int64_t e0 = col0 * r;
    for (int e = tid; e < ncol * r; e += 256) {
        const double v = red[(e % r) * 64 + e / r];
        if (d.n_q_tiles == 1) Qout[d.q_off + e0 + e] = (float)v;
        else ws[d.qpart_off + (int64_t)it.b * d.m * r + e0 + e] = v;
    }
}

}  // namespace

}  // namespace conef
