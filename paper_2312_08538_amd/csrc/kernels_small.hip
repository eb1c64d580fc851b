// The whole step of models whose matrices are all small, in one launch: a workgroup per matrix.
//
// Such a step is a chain of six launches of a workgroup or two, each 2 - 6 us of launch and of round trips to memory.  Here a
// matrix is fetched once: a thread keeps its octets as they came (gradient, codes, scale), p = g + (1 - beta) e goes to LDS, and P,
// the Gram matrix, its factor, P^, Q+ and the residual follow one another across workgroup barriers.  Bound by that chain on
// one CU.  One matrix of 256 x 128 at rank 2, fp32, 8-bit codes: 23 - 28 us a step in six launches, 14.8 so, of which in the kernel
// fetch and decode 2.1, P 2.2 and Q+ 3.2 (LDS reads, conversions to fp64), Gram matrix and factor 1.4, P^ 0.3, residual and
// rounding 2.4.
// The sums are the octet family's: fp64 matrix cores for P and Q+ (v_mfma_f64_4x4x4_4b_f64, layout at the octet P pass; in an order
// of their own, so that an entry in some 10^8 rounds to the other side of its last fp32 bit than in the stages' launches), the
// Gram matrix in the order of k_gram_small and k_cholesky_apply, the residual as the fp32 fma chain.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "octet_device.h"
#include "orth_device.h"

namespace conef {

namespace {

constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / 64;
constexpr int kSmallOctets = (int)(kSmallMaxElems / 8 / kSmallThreads);     // per thread

// Entry (i, c) of a factor as an operand of the fp64 matrix cores, and row `col` of Q+ in fp32: the rows of an octet are neighbours,
// and those of the octets that a wave's lanes read together fall on distinct banks.
__device__ __forceinline__ int small_factor_at(int i, int c, int rp) { return ((i >> 2) * rp + c) * 4 + (i & 3); }
__device__ __forceinline__ int small_q_at(int col, int rp) { return col * rp + (col >> 3) * 4; }

template <bool BF16, int BITS, int RP>
__global__ __launch_bounds__(kSmallThreads) void k_step_small(SmallPlan sp, const void *__restrict__ grads, uint32_t *codes, float *scales,
                                                              const float *Q_in, float *P_out, float *Q_out, uint32_t step_lo,
                                                              uint32_t step_hi)
{
    constexpr int H = RP / 4, E = RP * RP;
    extern __shared__ __attribute__((aligned(16))) double small_lds[];
    __shared__ CholeskyLds<RP> chol;
    __shared__ double rinv[E];
    const MatDesc d = sp.mats[blockIdx.x];
    const int r = sp.rank;
    const int n = (int)d.n, m = (int)d.m, m8 = d.m8;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int mi = lane & 15, mk = lane >> 4, mc = lane & 3;
    const int n16 = (n + 15) & ~15, m16 = (m + 15) & ~15, mp = m16 + kSmallPad;
    // LDS; the factors as operands of the fp64 matrix cores are doubles, converted once
    double *part = small_lds;                               // kSmallWaves x 16 x RP: partial sums of a split contraction, Gram tiles
    double *dq = part + kSmallWaves * 16 * RP;              // Q, columns up to m16
    double *dp = dq + m16 * RP;                             // P^, rows up to n16
    float *fp = reinterpret_cast<float *>(dp + n16 * RP);   // P, then P^
    float *T = fp + n16 * RP;                               // p: [row][mp], rows up to n16, columns up to m16
    float *fq = reinterpret_cast<float *>(dq);              // Q+, in the place of Q

    // ---- fetch: the thread's octets, and Q (columns of the rank's padding and rows up to n16 are zero)
    const int n_oct = n * m8;
    const int row_0 = t / m8, oct_0 = t - row_0 * m8;       // the thread's first octet; the others are kSmallThreads apart
    const int row_step = kSmallThreads / m8, oct_step = kSmallThreads - row_step * m8;
    auto advance = [&](int &row, int &oc) {
        row += row_step;
        oc += oct_step;
        if (oc >= m8) { oc -= m8; ++row; }
    };
    RawOctet<BF16, BITS> oct[kSmallOctets];
#pragma unroll
    for (int u = 0; u < kSmallOctets; ++u) {
        const int o = t + kSmallThreads * u;
        oct[u] = load_octet_always<BF16, BITS>(d, grads, codes, scales, o < n_oct ? o : n_oct - 1);
    }
    for (int e = t; e < m16 * RP; e += kSmallThreads) {
        const int k = e / RP, c = e % RP;
        const float v = Q_in[d.q_off + (int64_t)(k < m ? k : m - 1) * r + (c < r ? c : r - 1)];
        dq[small_factor_at(k, c, RP)] = k < m && c < r ? (double)v : 0.0;
    }
    for (int e = n * RP + t; e < n16 * RP; e += kSmallThreads) {
        fp[e] = 0.0f;
        dp[small_factor_at(e / RP, e % RP, RP)] = 0.0;
    }
    for (int e = n * mp + t; e < n16 * mp; e += kSmallThreads) T[e] = 0.0f;
    if (m16 != m)
        for (int e = t; e < 8 * n; e += kSmallThreads) T[(e >> 3) * mp + m + (e & 7)] = 0.0f;
    {
        int row = row_0, oc = oct_0;
#pragma unroll
        for (int u = 0; u < kSmallOctets; ++u) {
            if (t + kSmallThreads * u < n_oct) {
                float p[8];
                decode_octet<BF16, BITS>(oct[u], sp.omb, p);
                float4 *dst = reinterpret_cast<float4 *>(T + row * mp + oc * 8);
                dst[0] = make_float4(p[0], p[1], p[2], p[3]);
                dst[1] = make_float4(p[4], p[5], p[6], p[7]);
            }
            advance(row, oc);
        }
    }
    __syncthreads();

    // Where entry (i, c) of a factor stands in dq and dp: a lane's operands of four steps, i = 16 S + 4 mk + 0..3, are neighbours.
    // (Which four rows or columns a step of a contraction takes is free as long as both operands agree; LDS reads of 16 bytes,
    // a third as many, are what the two contractions are bound by.)
    auto load_b = [&](const double *f, int S, double (&b)[H][4]) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const double2 *src = reinterpret_cast<const double2 *>(f + ((4 * S + mk) * RP + mc + 4 * h) * 4);
            const double2 lo = src[0], hi = src[1];
            b[h][0] = lo.x; b[h][1] = lo.y; b[h][2] = hi.x; b[h][3] = hi.y;
        }
    };
    const int drow = 4 * (mi >> 2) + mk;                    // D of block (lane % 16) / 4, entry [lane / 16][lane % 4]

    // ---- P = p Q: 16 rows per wave and trip; fewer than 16 such tiles are shared by several waves, a range of columns each, and
    // the ranges' sums added in order
    {
        const int units = n16 >> 4, steps = (m + 15) >> 4;
        const int split = units >= kSmallWaves ? 1 : kSmallWaves / units;
        for (int w = wave; w < units * split; w += kSmallWaves) {           // (one trip where it is split)
            const int tile = split == 1 ? w : w % units, q = split == 1 ? 0 : w / units;
            const int s1 = steps * (q + 1) / split;
            const float *ap = T + (16 * tile + mi) * mp + 4 * mk;
            double acc[H] = {};
#pragma unroll 1
            for (int s = steps * q / split; s < s1; ++s) {
                const float4 a4 = *reinterpret_cast<const float4 *>(ap + 16 * s);
                double b[H][4];
                load_b(dq, s, b);
                const double av[4] = {(double)a4.x, (double)a4.y, (double)a4.z, (double)a4.w};
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int h = 0; h < H; ++h) acc[h] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[k], b[h][k], acc[h], 0, 0, 0);
            }
#pragma unroll
            for (int h = 0; h < H; ++h) {
                if (split == 1) fp[(16 * tile + drow) * RP + mc + 4 * h] = (float)acc[h];
                else part[(w * 16 + drow) * RP + mc + 4 * h] = acc[h];
            }
        }
        __syncthreads();
        if (split > 1) {
            for (int e = t; e < n16 * RP; e += kSmallThreads) {
                double s = part[e];
                for (int q = 1; q < split; ++q) s += part[q * n16 * RP + e];
                fp[e] = (float)s;
            }
            __syncthreads();
        }
    }

    // ---- partial Gram matrices: 64 rows per wave, groups of 16 added in order
    const int tiles = (n + 63) >> 6;
    if (wave < tiles) gram_tile<RP>(fp, n, wave, lane, part);
    __syncthreads();
    if (t < 64) factor_tiles<RP>(chol, part, tiles, t, r, rinv);
    __syncthreads();

    // ---- P^ = P R^-1, a row per thread
    if (t < n) {
        float in[RP];
#pragma unroll
        for (int c4 = 0; c4 < H; ++c4) {
            const float4 v = reinterpret_cast<const float4 *>(fp + t * RP)[c4];
            in[4 * c4] = v.x; in[4 * c4 + 1] = v.y; in[4 * c4 + 2] = v.z; in[4 * c4 + 3] = v.w;
        }
#pragma unroll
        for (int c = 0; c < RP; ++c) {
            if (c < r) {                                    // uniform
                double a = 0.0;
#pragma unroll
                for (int k = 0; k <= c; ++k) a = __builtin_fma((double)in[k], rinv[k * r + c], a);
                fp[t * RP + c] = (float)a;
                dp[small_factor_at(t, c, RP)] = (double)(float)a;
                P_out[d.p_off + (int64_t)t * r + c] = (float)a;
            } else {
                dp[small_factor_at(t, c, RP)] = 0.0;
            }
        }
    }
    __syncthreads();

    // ---- Q+ = p^T P^: 64 columns per wave and trip, a lane's four tiles are four neighbouring columns; ranges of rows as above, whose
    // sums take the place of p once all waves are done with it
    {
        const int units = (m + 63) >> 6, steps = n16 >> 4;
        const int split = units >= kSmallWaves ? 1 : kSmallWaves / units < steps ? kSmallWaves / units : steps;      // (so the sums fit)
        double *sums = reinterpret_cast<double *>(T);
        auto put = [&](int col, int c, double v) {
            if (col < m) fq[small_q_at(col, RP) + c] = (float)v;
            if (col < m && c < r) Q_out[d.q_off + (int64_t)col * r + c] = (float)v;
        };
        for (int w0 = 0; w0 < units * split; w0 += kSmallWaves) {           // (one trip where it is split)
            const int w = w0 + wave;
            const int tile = split == 1 ? w : w % units, q = split == 1 ? 0 : w / units;
            double acc[4][H] = {};
            if (w < units * split) {
                const int s1 = steps * (q + 1) / split;
                const int col = 64 * tile + 4 * mi;
                const float *ap = T + 4 * mk * mp + (col < m ? col : m - 4);        // (columns beyond the matrix are not stored)
#pragma unroll 1
                for (int s = steps * q / split; s < s1; ++s) {
                    float4 a4[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) a4[k] = *reinterpret_cast<const float4 *>(ap + (16 * s + k) * mp);
                    double b[H][4];
                    load_b(dp, s, b);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const double av[4] = {(double)a4[k].x, (double)a4[k].y, (double)a4[k].z, (double)a4[k].w};
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int h = 0; h < H; ++h)
                                acc[i][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[i], b[h][k], acc[i][h], 0, 0, 0);
                    }
                }
            }
            if (split == 1) {
                if (w < units) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int h = 0; h < H; ++h) put(64 * tile + 4 * drow + i, mc + 4 * h, acc[i][h]);
                }
                continue;
            }
            __syncthreads();
            if (w < units * split) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        const int col = 64 * tile + 4 * drow + i;
                        if (col < m) sums[(q * m + col) * RP + mc + 4 * h] = acc[i][h];
                    }
            }
        }
        __syncthreads();
        if (split > 1) {
            for (int e = t; e < m * RP; e += kSmallThreads) {
                double s = sums[e];
                for (int q = 1; q < split; ++q) s += sums[q * m * RP + e];
                put(e / RP, e % RP, s);
            }
            __syncthreads();
        }
    }

    // ---- residual, block maximum, rounding
    const float s_f = (float)((1 << (BITS - 1)) - 1);
    int row = row_0, oc = oct_0;
#pragma unroll
    for (int u = 0; u < kSmallOctets; ++u) {
        if (kSmallThreads * u >= n_oct) break;              // uniform
        const int o = t + kSmallThreads * u;
        const bool valid = o < n_oct;
        const float *ph = fp + (valid ? row : 0) * RP, *q = fq + small_q_at(8 * oc, RP);
        float x[8], acc[8];
        decode_octet<BF16, BITS>(oct[u], 1.0f, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const float4 p4 = reinterpret_cast<const float4 *>(ph)[h];
            float4 q4[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                q4[e] = *reinterpret_cast<const float4 *>(q + e * RP + 4 * h);
                acc[e] = __builtin_fmaf(p4.x, q4[e].x, acc[e]);
                acc[e] = __builtin_fmaf(p4.y, q4[e].y, acc[e]);
            }
            if (4 * h + 2 < r) {                            // uniform; an odd rank's padding is zero
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    acc[e] = __builtin_fmaf(p4.z, q4[e].z, acc[e]);
                    acc[e] = __builtin_fmaf(p4.w, q4[e].w, acc[e]);
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = x[e] - acc[e];
        const float a = block_max(valid ? abs_max_octet(0.0f, x) : 0.0f, d.lb_shift);
        const float inv16 = levels_over(a, s_f);
        uint32_t rnd[4], w[2];
        philox4x32_10((uint32_t)o, (uint32_t)blockIdx.x, step_lo, step_hi, sp.seed_lo, sp.seed_hi, rnd);
        quantise_octet<BITS>(x, inv16, rnd, w);
        if (valid) {
            if (BITS == 2 && o == n_oct - 1) store_code_words_end<BITS>(d, codes, o, 8, w);
            else store_code_words<BITS>(d, codes, o, w);
            if ((o & ((1 << d.lb_shift) - 1)) == 0) scales[d.scale_off + (o >> d.lb_shift)] = a;
        }
        advance(row, oc);
    }
}

}  // namespace

hipError_t launch_step_small(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Q_in, float *P_out,
                             float *Q_out, uint64_t step, hipStream_t st)
{
    const SmallPlan sp = {dp.mats, dp.rank, dp.omb, dp.seed_lo, dp.seed_hi};
    const uint32_t lo = (uint32_t)step, hi = (uint32_t)(step >> 32);
    auto go = [&](auto bf, auto bits, auto rp) {
        hipLaunchKernelGGL((k_step_small<decltype(bf)::value, decltype(bits)::value, decltype(rp)::value>), dim3(dp.n_mats), dim3(kSmallThreads),
                           dp.small_lds, st, sp, grads, codes, scales, Q_in, P_out, Q_out, lo, hi);
    };
    auto rank = [&](auto bf, auto bits) {
        if (dp.rpad == 4) go(bf, bits, std::integral_constant<int, 4>{});
        else go(bf, bits, std::integral_constant<int, 8>{});
    };
    auto width = [&](auto bf) {
        if (dp.bits == 2) rank(bf, std::integral_constant<int, 2>{});
        else if (dp.bits == 4) rank(bf, std::integral_constant<int, 4>{});
        else rank(bf, std::integral_constant<int, 8>{});
    };
    if (dp.dtype == 1) width(std::true_type{});
    else width(std::false_type{});
    return hipGetLastError();
}

}  // namespace conef
