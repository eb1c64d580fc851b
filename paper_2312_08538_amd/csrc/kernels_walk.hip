// The strip family's err pass where a matrix's Q+ fits into LDS (walk_device.h).  Bound by its vector instructions (about 250 per
// octet, 60 of them for the random numbers) and the loads in flight: no barriers after the first, seven or eight waves per
// SIMD.  On strips p goes through LDS twice, with two barriers per run and scalar work for every row.  us a step, on strips / so (the
// difference is this pass): 28.4 M fp32 elements in matrices of 650 columns at rank 4 112 / 96, at rank 8 125 / 113, with two vectors
// 153 / 148; 53 M of 1300 columns at rank 4 213 / 152; 100000 x 33 58 / 50, 300000 x 15 in bf16 87 / 82; 600 x 300 25.0 / 24.4.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "walk_device.h"

namespace conef {

namespace {

template <bool BF16, int BITS, int R, bool TWO>
__global__ __launch_bounds__(256) void k_err_walk(KernelPlan dp, const void *__restrict__ grads, uint32_t *codes, float *scales,
                                                  uint32_t *codes2, float *scales2, const float *__restrict__ Phat,
                                                  const float *__restrict__ Qn, uint32_t step_lo, uint32_t step_hi)
{
    extern __shared__ __attribute__((aligned(16))) float walk_lds[];
    err_walk<BF16, BITS, R, TWO>(dp, blockIdx.x, walk_lds, grads, codes, scales, codes2, scales2, Phat, Qn, step_lo, step_hi);
}

}  // namespace

// codes2 / scales2: the second error vector of Algorithm 3 (codes / scales then hold the first), or null
void walk_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2, float *scales2,
                   const float *Phat, const float *Qn, uint64_t step, hipStream_t st)
{
    if (dp.n_err_w <= 0) return;
    const uint32_t lo = (uint32_t)step, hi = (uint32_t)(step >> 32);
    auto go = [&](auto bf, auto bits, auto rank, auto two) {
        hipLaunchKernelGGL((k_err_walk<decltype(bf)::value, decltype(bits)::value, decltype(rank)::value, decltype(two)::value>),
                           dim3(dp.n_err_w), dim3(256), (size_t)dp.ew_lds * 4, st, dp, grads, codes, scales, codes2, scales2, Phat, Qn, lo, hi);
    };
    auto vectors = [&](auto bf, auto bits, auto rank) {
        if (codes2) go(bf, bits, rank, std::true_type{});
        else go(bf, bits, rank, std::false_type{});
    };
    auto rank = [&](auto bf, auto bits) {
        switch (walk_rank(dp.rank)) {
        case 1: vectors(bf, bits, std::integral_constant<int, 1>{}); break;
        case 2: vectors(bf, bits, std::integral_constant<int, 2>{}); break;
        case 4: vectors(bf, bits, std::integral_constant<int, 4>{}); break;
        default: vectors(bf, bits, std::integral_constant<int, 8>{}); break;
        }
    };
    auto width = [&](auto bf) {
        if (dp.bits == 2) rank(bf, std::integral_constant<int, 2>{});
        else if (dp.bits == 4) rank(bf, std::integral_constant<int, 4>{});
        else rank(bf, std::integral_constant<int, 8>{});
    };
    if (dp.dtype == 1) width(std::true_type{});
    else width(std::false_type{});
}

}  // namespace conef
