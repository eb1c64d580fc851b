// Strip kernel family: the three passes for any layout (any number of columns, any rank up to 32, blocks that straddle
// rows).  Most P and Q+ passes of the quantiser for blocks of whole octets are in kernels_ragged.hip; here are the others and the
// err pass.  A wave works on strips of 64 neighbouring columns, a lane owns a column of the strip and the row is uniform over
// the wave: a row of the strip is one coalesced access of the gradient (one element per lane, whatever the alignment of
// the row).  The 64-bit addresses of a workgroup's first block are formed once, on the scalar side; an element is a 32-bit
// distance from there, from which each lane takes its code word and block by shifts (a division where the block is not a
// power of two).  The row of a factor is a scalar operand.
//
// The element source is a template parameter: the quantiser's codes and scales (one or two error vectors) or the count
// sketch's table in its row or column form.
//
//   P pass    a workgroup per (32 rows, column chunk); its waves take the chunk's strips in turn.  p goes through a
//             wave-private LDS tile into the operand layout of the fp64 matrix cores; the four waves' sums are added in
//             wave order.  Products of fp32 values are exact in fp64, the sum stays in fp64, one rounding.
//   Q+ pass   a workgroup per (strip, row tile), a quarter of the rows per wave; a lane adds up its column's r sums in
//             fp64 registers, the row of P^ being a scalar operand.  Matrices of a few rows: a strip per wave (k_q_flat).
//   err pass  (ranks above 8 and matrices too wide for their Q+ to stand in LDS; the others: kernels_walk.hip)  a workgroup per run
//             of whole scale blocks: p is loaded and decoded in octets and goes to LDS in the order of
//             the flat index; there the reconstruction (the fp32 fma chain over c = 0..r-1, a lane's row of Q+ in registers,
//             the row of P^ on the scalar side) is subtracted a row of a strip at a time; then the workgroup walks the run in
//             octets as the octet family does: block max-norm by DPP, one Philox call per eight elements, rounding, pack, in
//             place.  Matrices of a few columns: groups of rows that fill a wave.
//
// All sums are combined in a fixed order: results do not depend on scheduling.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "strip_device.h"

namespace conef {

namespace {

template <int SRC, int RH>
__global__ __launch_bounds__(256) void k_p_strip(KernelPlan dp, Source src, const float *__restrict__ Q, float *P, double *ws)
{
    __shared__ __attribute__((aligned(16))) float lds[kPStripLds];
    p_strip<SRC, RH>(dp, blockIdx.x, lds, src, Q, P, ws);
}

template <int SRC, int R, bool EXACT>
__global__ __launch_bounds__(256) void k_q_strip(KernelPlan dp, Source src, const float *__restrict__ Phat, double *ws, float *Qout)
{
    __shared__ double red[2 * R * 64];
    q_strip<SRC, R, EXACT>(dp, blockIdx.x, red, src, Phat, ws, Qout);
}

template <int SRC, int R, bool EXACT>
__global__ __launch_bounds__(256) void k_q_flat(KernelPlan dp, Source src, const float *__restrict__ Phat, float *Qout)
{
    q_flat<SRC, R, EXACT>(dp, blockIdx.x, src, Phat, Qout);
}

template <int R, bool EXACT, bool TWO, bool GROUP>
__global__ __launch_bounds__(256) void k_err_strip(KernelPlan dp, const void *__restrict__ grads, uint32_t *codes, float *scales,
                                                   uint32_t *codes2, float *scales2, const float *__restrict__ Phat,
                                                   const float *__restrict__ Qn, uint32_t step_lo, uint32_t step_hi)
{
    extern __shared__ __attribute__((aligned(16))) float X[];
    err_strip<R, EXACT, TWO, GROUP>(dp, blockIdx.x, X, grads, codes, scales, codes2, scales2, Phat, Qn, step_lo, step_hi);
}

template <int SRC>
void pass_p(const DevicePlan &dp, const Source &src, const float *Q, float *P, double *ws, hipStream_t st)
{
    const dim3 grid(dp.n_p), block(256);
    switch (dp.rpad) {
    case 4: hipLaunchKernelGGL((k_p_strip<SRC, 1>), grid, block, 0, st, dp, src, Q, P, ws); break;
    case 8: hipLaunchKernelGGL((k_p_strip<SRC, 2>), grid, block, 0, st, dp, src, Q, P, ws); break;
    case 16: hipLaunchKernelGGL((k_p_strip<SRC, 4>), grid, block, 0, st, dp, src, Q, P, ws); break;
    default: hipLaunchKernelGGL((k_p_strip<SRC, 8>), grid, block, 0, st, dp, src, Q, P, ws); break;
    }
}

// go(rank or the next of 4, 8, 16, 32 as a constant, is it the rank itself)
template <typename F>
void by_rank(int rank, F &&go)
{
    switch (rank) {
    case 1: go(std::integral_constant<int, 1>{}, std::true_type{}); break;
    case 2: go(std::integral_constant<int, 2>{}, std::true_type{}); break;
    case 4: go(std::integral_constant<int, 4>{}, std::true_type{}); break;
    case 8: go(std::integral_constant<int, 8>{}, std::true_type{}); break;
    case 16: go(std::integral_constant<int, 16>{}, std::true_type{}); break;
    case 32: go(std::integral_constant<int, 32>{}, std::true_type{}); break;
    default:
        if (rank < 4) go(std::integral_constant<int, 4>{}, std::false_type{});
        else if (rank < 8) go(std::integral_constant<int, 8>{}, std::false_type{});
        else if (rank < 16) go(std::integral_constant<int, 16>{}, std::false_type{});
        else go(std::integral_constant<int, 32>{}, std::false_type{});
    }
}

template <int SRC>
void pass_q(const DevicePlan &dp, const Source &src, const float *Phat, double *ws, float *Qout, hipStream_t st)
{
    if (dp.n_q > 0)
        by_rank(dp.rank, [&](auto rank, auto exact) {
            hipLaunchKernelGGL((k_q_strip<SRC, decltype(rank)::value, decltype(exact)::value>), dim3(dp.n_q), dim3(256), 0, st, dp, src,
                               Phat, ws, Qout);
        });
}

// the matrices of up to kFlatRows rows (ranks up to 8: a matrix has at least as many rows)
template <int SRC>
void pass_q_flat(const DevicePlan &dp, const Source &src, const float *Phat, float *Qout, hipStream_t st)
{
    if (dp.n_q_flat > 0)
        by_rank(dp.rank, [&](auto rank, auto exact) {
            constexpr int R = decltype(rank)::value;
            if constexpr (R <= kFlatRows)
                hipLaunchKernelGGL((k_q_flat<SRC, R, decltype(exact)::value>), dim3(dp.n_q_flat), dim3(256), 0, st, dp, src, Phat, Qout);
        });
}

template <bool TWO, bool GROUP>
void pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2, float *scales2,
              const float *Phat, const float *Qn, uint64_t step, hipStream_t st)
{
    const int n = GROUP ? dp.n_err_g : dp.n_err_s;
    if (n <= 0) return;
    const uint32_t lo = (uint32_t)step, hi = (uint32_t)(step >> 32);
    by_rank(dp.rank, [&](auto rank, auto exact) {
        hipLaunchKernelGGL((k_err_strip<decltype(rank)::value, decltype(exact)::value, TWO, GROUP>), dim3(n), dim3(256),
                           (size_t)dp.es_lds * 4, st, dp, grads, codes, scales, codes2, scales2, Phat, Qn, lo, hi);
    });
}

}  // namespace

void strip_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Q, float *P,
                  double *ws, hipStream_t st)
{
    if (dp.n_p <= 0) return;
    const Source src = {grads, codes, scales, nullptr};
    if (dp.i_codes) pass_p<kSrcTwo>(dp, src, Q, P, ws, st);
    else pass_p<kSrcOne>(dp, src, Q, P, ws, st);
}

void strip_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat, double *ws,
                  float *Qout, hipStream_t st)
{
    const Source src = {grads, codes, scales, nullptr};
    if (dp.i_codes) pass_q<kSrcTwo>(dp, src, Phat, ws, Qout, st);
    else pass_q<kSrcOne>(dp, src, Phat, ws, Qout, st);
}

void strip_pass_q_flat(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat,
                       float *Qout, hipStream_t st)
{
    const Source src = {grads, codes, scales, nullptr};
    if (dp.i_codes) pass_q_flat<kSrcTwo>(dp, src, Phat, Qout, st);
    else pass_q_flat<kSrcOne>(dp, src, Phat, Qout, st);
}

void strip_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat, const float *Qn,
                    uint64_t step, hipStream_t st)
{
    pass_err<false, false>(dp, grads, codes, scales, nullptr, nullptr, Phat, Qn, step, st);
    pass_err<false, true>(dp, grads, codes, scales, nullptr, nullptr, Phat, Qn, step, st);
}

void strip_pass_err_two(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2, float *scales2,
                        const float *Phat, const float *Qn, uint64_t step, hipStream_t st)
{
    pass_err<true, false>(dp, grads, codes, scales, codes2, scales2, Phat, Qn, step, st);
    pass_err<true, true>(dp, grads, codes, scales, codes2, scales2, Phat, Qn, step, st);
}

void strip_cs_pass_p(const DevicePlan &dp, const void *grads, const void *table, const float *Q, float *P, double *ws, hipStream_t st)
{
    if (dp.n_p <= 0) return;
    const Source src = {grads, nullptr, nullptr, table};
    if (dp.cs_cols_mode) pass_p<kSrcCol>(dp, src, Q, P, ws, st);
    else pass_p<kSrcRow>(dp, src, Q, P, ws, st);
}

void strip_cs_pass_q(const DevicePlan &dp, const void *grads, const void *table, const float *Phat, double *ws, float *Qout,
                     hipStream_t st)
{
    const Source src = {grads, nullptr, nullptr, table};
    if (dp.cs_cols_mode) {
        pass_q<kSrcCol>(dp, src, Phat, ws, Qout, st);
        pass_q_flat<kSrcCol>(dp, src, Phat, Qout, st);
    } else {
        pass_q<kSrcRow>(dp, src, Phat, ws, Qout, st);
        pass_q_flat<kSrcRow>(dp, src, Phat, Qout, st);
    }
}

}  // namespace conef
