// Launches that carry the octet family's and the strip family's workgroups together, for models most of whose matrices are
// on the octet kernels and a few small ones on the strip kernels (a convolutional network's odd layers).  A launch of a few
// dozen strip workgroups takes 5 - 15 us, the time of one workgroup's chain of loads, on a chip that is otherwise empty;
// beside the octet workgroups it costs next to nothing.
//
// The strip workgroups come first (they are the longer chains), their number rounded up to a multiple of eight, so that
// the octet workgroups keep their XCDs (workgroup b runs on XCD b % 8).
//
// Measured on the 18-layer residual network (64 x 147 and five more shapes of 576 columns on the strip kernels, 11.4 M of
// 11.7 M elements on the octet kernels, rank 4, fp32 gradients):
// the three passes 20 + 19 + 35 us in launches of their own, 15 + 14 + 20 us together, the step 89 -> 65 us.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "octet_device.h"
#include "ragged_device.h"
#include "strip_device.h"
#include "walk_device.h"

namespace conef {

namespace {

constexpr int larger(int a, int b) { return a > b ? a : b; }

template <bool BF16, int BITS, int RH>
__global__ __launch_bounds__(256) CONEF_P_OCTET_WAVES(false)
void k_p_mixed(KernelPlan dp, int lead, const void *__restrict__ grads, const uint32_t *__restrict__ codes,
               const float *__restrict__ scales, const float *__restrict__ Q, float *P, double *ws)
{
    __shared__ __attribute__((aligned(16))) float lds[larger(kPOctetLds, kRagLds)];
    const int b = blockIdx.x;
    if (b >= lead) {
        const POctetLds o = {lds, reinterpret_cast<uint32_t *>(lds + kPOctetTiles), lds + kPOctetTiles + kPOctetCodes, nullptr, nullptr};
        p_octet<BF16, BITS, RH, false>(dp, b - lead, o, grads, codes, scales, Q, P, ws);
    } else if (b < dp.n_p) {
        p_ragged<BF16, BITS, RH, false>(dp, b, lds, grads, codes, scales, Q, P, ws);
    }
}

template <bool BF16, int BITS, int R, int JOINED>
__global__ __launch_bounds__(256) CONEF_Q_OCTET_WAVES(BF16, false)
void k_q_mixed(KernelPlan dp, int lead, const void *__restrict__ grads, const uint32_t *__restrict__ codes,
               const float *__restrict__ scales, const float *__restrict__ Phat, double *ws, float *Qout)
{
    __shared__ __attribute__((aligned(16))) float lds[larger(kQOctetLds, kRagLds)];
    const int b = blockIdx.x;
    if (b >= lead) {
        q_octet<BF16, BITS, (R > 4 ? 2 : 1), false, JOINED>(dp, b - lead, lds, grads, codes, scales, Phat, ws, Qout);
    } else if (b < dp.n_q) {
        q_ragged<BF16, BITS, (R > 4 ? 2 : 1), false>(dp, b, lds, grads, codes, scales, Phat, ws, Qout);
    }
}

// WALK: the strip family's workgroups are those with Q+ in LDS
template <bool BF16, int BITS, int R, bool WIDE, bool WALK>
__global__ __launch_bounds__(256, 2) void k_err_mixed(KernelPlan dp, int lead, const void *__restrict__ grads, uint32_t *codes,
                                                      float *scales, const float *__restrict__ Phat, const float *__restrict__ Qn,
                                                      uint32_t step_lo, uint32_t step_hi)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int b = blockIdx.x;
    if (b >= lead)
        err_tile<BF16, BITS, R, WIDE, false>(dp, b - lead, lds, grads, codes, scales, Phat, Qn, step_lo, step_hi, nullptr, nullptr);
    else if (WALK && b < dp.n_err_w)
        err_walk<BF16, BITS, R, false>(dp, b, lds, grads, codes, scales, nullptr, nullptr, Phat, Qn, step_lo, step_hi);
    else if (!WALK && b < dp.n_err_s)
        err_strip<R, true, false, false>(dp, b, lds, grads, codes, scales, nullptr, nullptr, Phat, Qn, step_lo, step_hi);
}

// At most two strip workgroups per CU: with more, the strip kernels fill the chip by themselves, and their own launch
// does not hold them to the octet kernels' registers and LDS.
constexpr int kMixedStrips = 512;
constexpr int kMixedLds = 10240;        // floats per workgroup of the err pass (four workgroups per CU)

int lead_of(int n_strip) { return (n_strip + 7) & ~7; }

template <typename F>
void by_type(const DevicePlan &dp, F &&go)
{
    auto bits = [&](auto bf) {
        if (dp.bits == 2) go(bf, std::integral_constant<int, 2>{});
        else if (dp.bits == 4) go(bf, std::integral_constant<int, 4>{});
        else go(bf, std::integral_constant<int, 8>{});
    };
    if (dp.dtype == 1) bits(std::true_type{});
    else bits(std::false_type{});
}

}  // namespace

bool mixed_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Q, float *P,
                  double *ws, hipStream_t st)
{
    if (dp.n_p_r <= 0 || dp.n_p_f <= 0 || dp.i_codes || dp.n_p_r > kMixedStrips) return false;
    const int lead = lead_of(dp.n_p_r);
    by_type(dp, [&](auto bf, auto bits) {
        constexpr bool BF = decltype(bf)::value;
        constexpr int B = decltype(bits)::value;
        const dim3 grid(lead + dp.n_p_f), block(256);
        if (dp.rank > 4) hipLaunchKernelGGL((k_p_mixed<BF, B, 2>), grid, block, 0, st, octet_items(dp), lead, grads, codes, scales, Q, P, ws);
        else hipLaunchKernelGGL((k_p_mixed<BF, B, 1>), grid, block, 0, st, octet_items(dp), lead, grads, codes, scales, Q, P, ws);
    });
    return true;
}

bool mixed_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat, double *ws,
                  float *Qout, hipStream_t st)
{
    if (dp.n_q_r <= 0 || dp.n_q_f <= 0 || dp.i_codes || dp.n_q_r > kMixedStrips) return false;
    const int lead = lead_of(dp.n_q_r);
    by_type(dp, [&](auto bf, auto bits) {
        constexpr bool BF = decltype(bf)::value;
        constexpr int B = decltype(bits)::value;
        const dim3 grid(lead + q_octet_groups(dp)), block(256);
        auto go = [&](auto rank, auto joined) {
            hipLaunchKernelGGL((k_q_mixed<BF, B, decltype(rank)::value, decltype(joined)::value>), grid, block, 0, st, octet_items(dp), lead, grads,
                               codes, scales, Phat, ws, Qout);
        };
        if (dp.rank == 8 && dp.q_joined) go(std::integral_constant<int, 8>{}, std::integral_constant<int, kQJoinedYes>{});
        else if (dp.rank == 8) go(std::integral_constant<int, 8>{}, std::integral_constant<int, kQJoinedNo>{});
        else if (dp.rank == 4) go(std::integral_constant<int, 4>{}, std::integral_constant<int, kQJoinedAtRunTime>{});
        else go(std::integral_constant<int, 2>{}, std::integral_constant<int, kQJoinedAtRunTime>{});
    });
    return true;
}

bool mixed_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat, const float *Qn,
                    uint64_t step, hipStream_t st)
{
    const bool walk = dp.n_err_w > 0;
    const int n_strip = walk ? dp.n_err_w : dp.n_err_s, strip_lds = walk ? dp.ew_lds : dp.es_lds;
    if (n_strip <= 0 || dp.n_err_t <= 0 || dp.i_codes || n_strip > kMixedStrips || strip_lds > kMixedLds) return false;
    const int lead = lead_of(n_strip);
    const uint32_t lo = (uint32_t)step, hi = (uint32_t)(step >> 32);
    by_type(dp, [&](auto bf, auto bits) {
        constexpr bool BF = decltype(bf)::value;
        constexpr int B = decltype(bits)::value;
        const dim3 grid(lead + (dp.n_err_t + 3) / 4), block(256);
        auto go = [&](auto rank, auto wide) {
            constexpr int R = decltype(rank)::value;
            constexpr bool W = decltype(wide)::value;
            const size_t lds = 4 * (size_t)larger(strip_lds, err_tile_lds<R, W>());
            if (walk) hipLaunchKernelGGL((k_err_mixed<BF, B, R, W, true>), grid, block, lds, st, dp, lead, grads, codes, scales, Phat, Qn, lo, hi);
            else hipLaunchKernelGGL((k_err_mixed<BF, B, R, W, false>), grid, block, lds, st, dp, lead, grads, codes, scales, Phat, Qn, lo, hi);
        };
        auto width = [&](auto rank) {
            if (dp.block == 256) go(rank, std::true_type{});
            else go(rank, std::false_type{});
        };
        if (dp.rank == 8) width(std::integral_constant<int, 8>{});
        else width(std::integral_constant<int, 4>{});
    });
    return true;
}

}  // namespace conef
