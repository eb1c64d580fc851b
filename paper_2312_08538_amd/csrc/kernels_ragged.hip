// Strip family, P and Q+ passes of the quantiser for scale blocks of 8 * 2^j elements (j <= 6) and any number of columns.  The
// gradient, codes and scales are loaded and decoded in octets of the flat index, which are aligned whatever the row length
// and never cross a scale block; a wave puts them into its LDS tile as they are, each row shifted by where it starts in its
// first octet, and the operands of the fp64 matrix cores are read with that shift (ragged_device.h).  Blocks that no
// power-of-two number of lanes holds in octets, the count sketch, and a matrix of more than 2^24 columns take the kernels of
// kernels_strip.hip, a lane per column and a load per element; so does the Q+ pass of a model whose matrices are too small or have
// too few rows (ragged_q_pays in plan.h).
//
// Measured (28.4 M elements in five matrices of 650 columns, fp32, rank 4, 4-bit codes in blocks of 128), before and after: P
// pass 35 -> 29 us (0.13 GB: 4.4 TB/s), Q+ pass 46 -> 28 us.  Of the latter 43 -> 28 came from giving every XCD a contiguous
// range of items: a strip's row is 256 bytes at any alignment and its codes 32, so neighbouring strips share most lines, and
// dealt to the XCDs in turn each fetched them again.
#include <type_traits>

#include "ragged_device.h"

namespace conef {

namespace {

template <bool BF16, int BITS, int RH, bool TWO>
__global__ __launch_bounds__(256) void k_p_ragged(KernelPlan dp, const void *__restrict__ grads, const uint32_t *__restrict__ codes,
                                                  const float *__restrict__ scales, const float *__restrict__ Q, float *P, double *ws)
{
    __shared__ __attribute__((aligned(16))) float lds[kRagLds];
    p_ragged<BF16, BITS, RH, TWO>(dp, blockIdx.x, lds, grads, codes, scales, Q, P, ws);
}

template <bool BF16, int BITS, int RH, bool TWO>
__global__ __launch_bounds__(256) void k_q_ragged(KernelPlan dp, const void *__restrict__ grads, const uint32_t *__restrict__ codes,
                                                  const float *__restrict__ scales, const float *__restrict__ Phat, double *ws, float *Qout)
{
    __shared__ __attribute__((aligned(16))) float lds[kRagLds];
    q_ragged<BF16, BITS, RH, TWO>(dp, blockIdx.x, lds, grads, codes, scales, Phat, ws, Qout);
}

// go(bf16, bits, rank / 4, two vectors)
template <typename F>
void by_type(const DevicePlan &dp, F &&go)
{
    auto two = [&](auto bf, auto bits, auto rh) {
        if (dp.i_codes) go(bf, bits, rh, std::true_type{});
        else go(bf, bits, rh, std::false_type{});
    };
    auto rank = [&](auto bf, auto bits) {
        if (dp.rpad == 4) two(bf, bits, std::integral_constant<int, 1>{});
        else if (dp.rpad == 8) two(bf, bits, std::integral_constant<int, 2>{});
        else if (dp.rpad == 16) two(bf, bits, std::integral_constant<int, 4>{});
        else two(bf, bits, std::integral_constant<int, 8>{});
    };
    auto bits = [&](auto bf) {
        if (dp.bits == 2) rank(bf, std::integral_constant<int, 2>{});
        else if (dp.bits == 4) rank(bf, std::integral_constant<int, 4>{});
        else rank(bf, std::integral_constant<int, 8>{});
    };
    if (dp.dtype == 1) bits(std::true_type{});
    else bits(std::false_type{});
}

}  // namespace

void ragged_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Q, float *P,
                   double *ws, hipStream_t st)
{
    if (dp.n_p_r <= 0) return;
    by_type(dp, [&](auto bf, auto bits, auto rh, auto two) {
        hipLaunchKernelGGL((k_p_ragged<decltype(bf)::value, decltype(bits)::value, decltype(rh)::value, decltype(two)::value>), dim3(dp.n_p_r),
                           dim3(256), 0, st, octet_items(dp), grads, codes, scales, Q, P, ws);
    });
}

void ragged_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat, double *ws,
                   float *Qout, hipStream_t st)
{
    if (dp.n_q_r <= 0) return;
    by_type(dp, [&](auto bf, auto bits, auto rh, auto two) {
        hipLaunchKernelGGL((k_q_ragged<decltype(bf)::value, decltype(bits)::value, decltype(rh)::value, decltype(two)::value>), dim3(dp.n_q_r),
                           dim3(256), 0, st, octet_items(dp), grads, codes, scales, Phat, ws, Qout);
    });
}

}  // namespace conef
