// Device code of the Cholesky factorisation of a Gram matrix, for the orthonormalisation's launches (kernels_orth.hip) and the
// step of small matrices in one launch (kernels_small.hip).
#pragma once
#include "device_common.h"

namespace conef {

namespace {

// 1 / sqrt(x) in fp64: the hardware's approximation and two Newton steps (a few units in the last place)
__device__ __forceinline__ double rsqrt_f64(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    y = __builtin_fma(y, __builtin_fma(-h * y, y, 0.5), y);
    y = __builtin_fma(y, __builtin_fma(-h * y, y, 0.5), y);
    return y;
}

// Factors G = R^T R (r x r, in LDS with row pitch RP) and writes R^-1 (row-major, r x r).  THREADS threads of the workgroup,
// t = 0 .. THREADS - 1, take part: one wave, or all.  Forward elimination of the rows of [G | I], a row per trip: row c times
// 1 / R[c][c] is row c of R and of (R^T)^-1, and a thread has its entries of both halves in registers.  A column whose squared
// norm after projection is not above 1e-12 of its squared norm is linearly dependent on the earlier ones: its column of R^-1
// (and so of P^) is zero.  So it is for a column with an entry that is not finite, and nothing of it reaches the others: P^ then
// has NaN in that entry's row and nowhere else.
// The loop is not unrolled: a launch that runs its code once fetches every line of it from memory, and with all trips and lane
// indices written out (61 KB at rank 32) that was most of its time (the stage's four launches for three matrices of 64 x 64
// at rank 32: 40.0 -> 28.9 us).  A trip is a chain of LDS reads, the reciprocal root and the products: with a branch around a
// dead pivot's the reads wait for the comparison (600 x 300, the stage at ranks 8 / 16 / 32 9.4 / 18.4 / 28.5 us, so 9.1 / 17.5 /
// 27.7).
template <int RP>
struct CholeskyLds {
    double G[RP * RP];
    double row_g[2][RP], row_y[2][RP];
};

template <int RP, int THREADS>
__device__ __forceinline__ void cholesky_inverse(CholeskyLds<RP> &lds, int t, int r, double *rinv)
{
    constexpr int V = RP * RP > THREADS ? RP * RP / THREADS : 1, kRows = THREADS / RP;
    const int j = t % RP, i0 = t / RP;
    double g[V], y[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int i = i0 + v * kRows;
        g[v] = i < r && j < r ? lds.G[i * RP + j] : 0.0;
        y[v] = i == j ? 1.0 : 0.0;
    }
#pragma unroll 1
    for (int c = 0; c < r; ++c) {
        double *row_g = lds.row_g[c & 1], *row_y = lds.row_y[c & 1];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (i0 + v * kRows == c) {
                row_g[j] = g[v];
                row_y[j] = y[v];
            }
        }
        if (THREADS > 64) __syncthreads();
        else wave_lds_sync();
        // all that the trip reads is asked for at once
        const double dcc = row_g[c], gcc = lds.G[c * RP + c];
        double gj = row_g[j], yj = row_y[j], gi[V];
#pragma unroll
        for (int v = 0; v < V; ++v) gi[v] = row_g[i0 + v * kRows < RP ? i0 + v * kRows : 0];
        // a dead pivot's row counts as zero before it is multiplied: that of a column of P that is not finite is not finite either
        const bool live = dcc > 1e-12 * gcc;            // uniform
        const double ri = rsqrt_f64(live ? dcc : 1.0);  // 1 / R[c][c]
        gj = live ? gj * ri : 0.0;
        yj = live ? yj * ri : 0.0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int i = i0 + v * kRows;
            if (i == c) y[v] = yj;
            if (i > c && i < RP) {
                const double rci = live ? gi[v] * ri : 0.0;
                g[v] = __builtin_fma(-rci, gj, g[v]);
                y[v] = __builtin_fma(-rci, yj, y[v]);
            }
        }
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int i = i0 + v * kRows;
        if (i < r && j < r) rinv[j * r + i] = y[v];
    }
}

// Partial Gram matrices of a factor that stands in LDS ([row][RP], n rows, zero beyond the rank): 64 rows per wave, groups of 16
// (v_mfma_f64_4x4x4_4b_f64, see k_gram_small) added in order; tile w's blocks 00, 01, 11 to part[w][.][16].
template <int RP>
__device__ __forceinline__ void gram_tile(const float *rows, int n, int wave, int lane, double *part)
{
    constexpr int H = RP / 4, NG = H * (H + 1) / 2;
    const int mc = lane & 3;
    double sum[NG];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int row = 64 * wave + 16 * g + (lane >> 2);
        double a[H];
#pragma unroll
        for (int h = 0; h < H; ++h) a[h] = row < n ? (double)rows[row * RP + mc + 4 * h] : 0.0;
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            double acc = __builtin_amdgcn_mfma_f64_4x4x4f64(a[q == 2 ? H - 1 : 0], a[q == 0 ? 0 : H - 1], 0.0, 0, 0, 0);
            acc += __shfl_xor(acc, 4, 64);
            acc += __shfl_xor(acc, 8, 64);
            sum[q] = g == 0 ? acc : sum[q] + acc;
        }
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
        if ((lane & 12) == 0) part[(wave * NG + q) * 16 + (lane >> 4) * 4 + mc] = sum[q];
}

// The sum of up to 16 such tiles, in the order of k_cholesky_apply, and its factorisation, by one wave (t = 0 .. 63).
template <int RP>
__device__ __forceinline__ void factor_tiles(CholeskyLds<RP> &chol, const double *part, int tiles, int t, int r, double *rinv)
{
    constexpr int H = RP / 4, NG = H * (H + 1) / 2, PARTS = orth_threads(RP) / (RP * RP);
    if (t < r * r) {
        const int i = t / r, j = t - i * r;
        const int lo = i < j ? i : j, hi = i < j ? j : i;
        const double *src = part + ((lo >> 2) + (hi >> 2)) * 16 + (lo & 3) * 4 + (hi & 3);
        double v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = k < tiles ? src[k * NG * 16] : 0.0;
        double all = 0.0;
#pragma unroll
        for (int k = 0; k < PARTS; ++k) all += PARTS < 16 ? v[k] + v[(k + PARTS) & 15] : v[k];
        chol.G[i * RP + j] = all;
    }
    wave_lds_sync();
    cholesky_inverse<RP, 64>(chol, t, r, rinv);
}

}  // namespace

}  // namespace conef
