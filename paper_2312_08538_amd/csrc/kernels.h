// Launch interface between the C ABI (api.cpp) and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "plan.h"

namespace conef {

// Device-resident copy of a plan: descriptor array and work tables.  What kernels read of it, and so what every launch carries: a
// line of 64 bytes more costs 0.1 - 0.4 us a launch, in the copy and, if the kernel reads it, in the fetch.  The scalars that most
// kernels read are one line, a table and the counts read beside it neighbours.  us a step of six launches, 664 bytes / so: 4482 x 147 at
// rank 4 30.1 / 28.4, 600 x 200 at rank 32 56.2 / 55.6, scaled sign of 4 M elements 16.0 / 15.5, 28.4 M elements in matrices of 650 columns
// 109.4 / 108.1.
struct KernelPlan {
    const MatDesc *mats = nullptr;
    int rank = 0, bits = 0, block = 0, dtype = 0;
    int wshift = 0, lb_shift = 0;   // log2(code fields per word), log2(block / 8)
    int block_shift = -1;           // log2(block), -1 if it is not a power of two
    float inv_s = 0.0f;             // fl32(1 / s)
    uint64_t bmagic = 0;            // j / block = mulhi64(j, bmagic) for j < 2^35
    uint32_t seed_lo = 0, seed_hi = 0;
    float beta = 0.0f, omb = 1.0f;  // beta and fl32(1 - beta)
    const WorkItem *p_items = nullptr, *q_items = nullptr, *err_s_items = nullptr;        // strip kernels (any shape)
    const WorkItem *err_w_items = nullptr;      // strip err pass with Q+ in LDS
    int n_p = 0, n_q = 0, n_err_s = 0, n_err_w = 0;
    // count-sketch mode
    const int32_t *row_hash = nullptr;
    int table_dtype = 0;            // 0 fp32, 1 fp16
    int cs_cols_mode = 0;       // count sketch in the column form: row_hash / bucket lists are over columns, tables rows x w
    const WorkItem *upd_items = nullptr;                                                   // decompress / update
    const int32_t *bucket_ptr = nullptr, *bucket_rows = nullptr;
    const int2 *row_order = nullptr;        // row sketch: a matrix's rows bucket by bucket: (row, bit 31: sign -1; bucket)
    const WorkItem *cs_err_items = nullptr, *cs_err_f_items = nullptr;
    const WorkItem *csc_p_items = nullptr;      // column form, P pass by rows
    const WorkItem *q_flat_items = nullptr, *err_g_items = nullptr;     // few rows (Q+ pass), few columns (err pass)
    const WorkItem *p_f_items = nullptr, *q_f_items = nullptr, *err_f_items = nullptr;    // octet family
    const WorkItem *err_t_items = nullptr;      // octet family, err pass with the residual on the fp32 matrix cores
    int n_p_f = 0, n_q_f = 0, n_err_f = 0, n_err_t = 0;
    int q_joined = 0;               // octet Q+ pass: a workgroup per strip, its waves the row tiles, Q+ straight from there
    int n_mats = 0;
    const WorkItem *p_m_items = nullptr, *q_m_items = nullptr, *err_m_items = nullptr;    // MFMA family
    const WorkItem *split_p_items = nullptr, *split_qn_items = nullptr;
    int n_p_m = 0, n_q_m = 0, n_err_m = 0;
    int n_p_k = 0;
    const WorkItem *p_k_items = nullptr;        // packed-split passes
    // element-wise gradient compressors
    const WorkItem *rb_items = nullptr, *rb_g_items = nullptr;
    int n_rb = 0;
    int norm_back = 0;              // the scaled sign's norm pass goes backwards (set by its launcher)
    // Algorithm 3, version 2, around an element-wise gradient compressor: the first error vector (a random block of
    // every matrix, MatDesc::i2_k values at i2_off) as it comes in and where the new one goes (another buffer)
    const float *i2_in = nullptr;
    float *i2_out = nullptr;
    // Improved contractive error feedback around the rank-r compressor: the FIRST error vector, laid out like the
    // codes / scales arguments of the pass kernels (which then hold the second one): p = g + first + second.  Null in
    // every other call; set in a copy of the plan by the launchers of the two-vector passes.
    const uint32_t *i_codes = nullptr;
    const float *i_scales = nullptr;
    int n_apply = 0, n_cs_lin = 0;
    const WorkItem *q_k_items = nullptr;
    int n_q_k = 0;
    const WorkItem *cs_t_items = nullptr, *cs_qt_items = nullptr, *cs_u_items = nullptr, *cs_lin_items = nullptr;   // count sketch, linear form
    const WorkItem *err_items = nullptr;        // err pass of blocks the strip kernel does not take
    const WorkItem *pred_items = nullptr, *gram_items = nullptr, *apply_items = nullptr, *qred_items = nullptr,
                   *elem_items = nullptr;
    const OrthItem *gram_s_items = nullptr, *apply_s_items = nullptr;      // orthonormalisation, ranks up to 8
    const int32_t *orth_first = nullptr;        // both in one launch: each matrix's first gram_s_items entry; null: two launches
    uint64_t pad = 0;               // a kernel's other arguments start a line
};
static_assert(sizeof(KernelPlan) == 8 * 64, "whole lines, and a line more for every launch");

// ... and what only their launchers read
struct DevicePlan : KernelPlan {
    int n_rb_g = 0;
    int n_cs_t = 0, n_cs_qt = 0, n_cs_u = 0, n_cs_err = 0, n_cs_err_f = 0;
    int n_cs_err_f_old = 0;     // matrices of the octet path that are NOT in the linear form (0: skip their update launch)
    int n_csc_p = 0, csc_p_lds = 0, csc_p_threads = 0;      // column form, P pass by rows
    int csc_lds = 0, csc_threads = 0;   // column form: LDS floats and threads per workgroup of the update pass
    int n_gram_s = 0, n_apply_s = 0, n_err = 0, n_split_p = 0, n_split_qn = 0;
    int n_upd = 0, upd_many = 0;    // upd_many: its items may be of several row tiles
    int n_pred = 0, n_gram = 0, n_qred = 0, n_elem = 0;
    int rpad = 0, n_q_flat = 0, n_err_g = 0;
    int most_p_chunks = 1;          // column chunks of P of the matrix that has the most
    int ew_lds = 0, es_lds = 0;     // floats of LDS per workgroup of the strip err passes
    int norm_back_one = 0, norm_back_two = 0;
    long long q_elems = 0;
    // Strip kernels, P and Q+ passes on octets.  The launchers of those kernels put them in the place of p_items and the others
    // (octet_items).
    const WorkItem *p_r_items = nullptr, *q_r_items = nullptr;
    int n_p_r = 0, n_q_r = 0;
    size_t small_lds = 0;           // bytes of LDS of the step in one launch (0: the model does not take it)
};

// What the step in one launch reads of it
struct SmallPlan {
    const MatDesc *mats;
    int rank;
    float omb;
    uint32_t seed_lo, seed_hi;
};

// workgroups of the octet Q+ pass
inline int q_octet_groups(const DevicePlan &dp) { return dp.q_joined ? dp.n_q_f : (dp.n_q_f + 3) / 4; }

inline DevicePlan octet_items(DevicePlan dp)
{
    dp.p_items = dp.p_r_items; dp.q_items = dp.q_r_items;
    dp.n_p = dp.n_p_r; dp.n_q = dp.n_q_r;
    return dp;
}

// Optional pair of events recorded immediately before and after a stage's main kernel.
struct Span {
    hipEvent_t begin = nullptr, end = nullptr;
};

// Each launcher enqueues on `st` and returns hipGetLastError().  `ws` is the caller's workspace.
// add_chunks: the partial sums of column chunks are added up into P; a full step leaves that to launch_orthonormalise's first
// launch (p_chunks there) where orth_adds_chunks says so
hipError_t launch_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales,
                         const float *Q, float *P, double *ws, bool add_chunks, hipStream_t st, Span span = Span());
// Ranks up to 4: up to 16 chunks, 5 to 8: up to 8.  A workgroup of that launch adds the chunks of its 64 rows one group of loads
// after another, 0.13 us a chunk (0.25), where the launch for the sums has a thread per entry of P and costs 2 us.  A step of 64
// rows in 2 / 8 / 16 / 24 / 64 chunks: rank 4 1.2 / 0.8 / 0.4 us faster, 0.3 / 4.4 slower than with that launch; rank 8 1.4 /
// 0.5 faster, 0.6 / 2.5 / 10 slower (512 rows: 1.7 / 1.8 / 0.9, 0.1 / 5.3; 1.7 / 1.3, 1.8 / 1.4 / 9.8).
inline bool orth_adds_chunks(const DevicePlan &dp) { return dp.rpad <= 8 && dp.most_p_chunks <= (dp.rpad == 4 ? 16 : 8); }
// tr_a / tr_b (the full step only): block scales of the error vector(s) whose column-block-major copies are made for
// the rank-32 family alongside the factorisations (into the first / the second workspace region); launch_pass_q is then
// called with scales_ready
hipError_t launch_orthonormalise(const DevicePlan &dp, float *P, double *ws, bool p_chunks, hipStream_t st,
                                 Span span = Span(), const float *tr_a = nullptr, const float *tr_b = nullptr);
hipError_t launch_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales,
                         const float *Phat, float *Qout, double *ws, bool scales_ready, hipStream_t st,
                         Span span = Span());
hipError_t launch_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales,
                           const float *Phat, const float *Qn, uint64_t step, double *ws, bool splits_ready,
                           hipStream_t st, Span span = Span());
// The whole step of a model of small matrices (dp.small_lds > 0; kernels_small.hip).  Q_out may be Q_in.
hipError_t launch_step_small(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Q_in, float *P_out,
                             float *Q_out, uint64_t step, hipStream_t st);
hipError_t launch_update(const DevicePlan &dp, const float *Phat, const float *Qn, float *x, bool subtract,
                         hipStream_t st);
// Random-block gradient compressor: one streaming pass (decode + add, keep the block, compress the rest).
// Improved contractive error feedback around the rank-r compressor: the P and Q+ passes are launch_pass_p /
// launch_pass_q on a plan that carries the first vector (i_codes, i_scales) with the second vector as their codes /
// scales; the err pass decodes both vectors and writes both (splits_ready as in launch_pass_err).
hipError_t launch_pass_err_two(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2,
                               float *scales2, const float *Phat, const float *Qn, uint64_t step, double *ws, bool splits_ready,
                               hipStream_t st, Span span);
void octet_pass_err_two(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2,
                        float *scales2, const float *Phat, const float *Qn, uint64_t step, hipStream_t st);
// The element-wise gradient compressors of the streaming kernels: random block, the two passes of the scaled sign (l1
// norm, then sign bits), random-k with one coordinate per stratum, random-k as a uniformly drawn subset.
constexpr int kModeBlock = 0, kModeNorm = 1, kModeSign = 2, kModeStrata = 3, kModeUniform = 4;
// codes2 / scales2 (here, in octet_stream_step and in launch_ss_step): the second error vector of Algorithm 3, or null;
// mode: kModeBlock, kModeStrata or kModeUniform
hipError_t launch_rb_step(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, float *delta,
                          uint64_t step, uint32_t *codes2, float *scales2, int mode, hipStream_t st);
hipError_t launch_cs_rb_step(const DevicePlan &dp, const void *grads, void *table, float *delta, uint64_t step,
                             int mode, hipStream_t st);
void octet_stream_step(const DevicePlan &dp, int mode, const void *grads, uint32_t *codes, float *scales, float *delta,
                       uint64_t step, uint32_t *sign_words, const float *c_scale, double *ws, uint32_t *codes2,
                       float *scales2, hipStream_t st);
// Scaled-sign gradient compressor: l1 norm pass, scale, sign bits + compression.
hipError_t launch_ss_step(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *sign_words,
                          float *c_scale, double *ws, uint64_t step, uint32_t *codes2, float *scales2, hipStream_t st);
hipError_t launch_cs_ss_step(const DevicePlan &dp, const void *grads, void *table, uint32_t *sign_words, float *c_scale,
                             double *ws, hipStream_t st);
void launch_ss_scale(const DevicePlan &dp, const double *ws, float *c_scale, hipStream_t st);
void launch_ss_clear(const DevicePlan &dp, uint32_t *sign_words, hipStream_t st);

// Count-sketch mode: the same three passes with a table as the error state.
hipError_t launch_cs_pass_p(const DevicePlan &dp, const void *grads, const void *table, const float *Q, float *P,
                            double *ws, bool add_chunks, hipStream_t st, Span span = Span());
hipError_t launch_cs_pass_q(const DevicePlan &dp, const void *grads, const void *table, const float *Phat, float *Qout,
                            double *ws, hipStream_t st, Span span = Span());
hipError_t launch_cs_pass_err(const DevicePlan &dp, const void *grads, void *table, const float *Phat, const float *Qn,
                              double *ws, hipStream_t st, Span span = Span());
// the count sketch in its linear form on the bf16 matrix cores (rank 32): see kernels_sketch.hip
void mfma_cs_pass_p(const DevicePlan &dp, const void *grads, const void *table, const float *Q, float *P, double *ws, hipStream_t st);
void mfma_cs_pass_q(const DevicePlan &dp, const void *grads, const void *table, const float *Phat, double *ws, hipStream_t st);
hipError_t launch_cs_decode(const DevicePlan &dp, const void *table, float *e_out, hipStream_t st);
hipError_t launch_decode(const DevicePlan &dp, const uint32_t *codes, const float *scales, float *e_out,
                         hipStream_t st);
hipError_t launch_reset(const DevicePlan &dp, uint32_t *codes, float *scales, size_t n_words, size_t n_scales,
                        hipStream_t st);

// Kernel families (each enqueues its own grouped launches; no-ops when their tables are empty).
// packed-split P and Q+ passes on the bf16 matrix cores (ranks 2, 4, 8; kernels_pack.hip); dp.i_codes as in mfma_pass_p
void pack_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Q, float *P,
                 hipStream_t st);
void pack_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat,
                 double *ws, float *Qout, hipStream_t st);
// any shape, a lane per column (kernels_strip.hip); dp.i_codes as in mfma_pass_p
void strip_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Q, float *P,
                  double *ws, hipStream_t st);
void strip_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat,
                  double *ws, float *Qout, hipStream_t st);
void strip_pass_q_flat(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat,
                       float *Qout, hipStream_t st);
void strip_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat, const float *Qn,
                    uint64_t step, hipStream_t st);
void strip_pass_err_two(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2, float *scales2,
                        const float *Phat, const float *Qn, uint64_t step, hipStream_t st);
// err pass with Q+ in LDS (kernels_walk.hip); codes2 / scales2: the second error vector (codes / scales the first), or null
void walk_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2, float *scales2,
                   const float *Phat, const float *Qn, uint64_t step, hipStream_t st);
// the same for the matrices that the plan takes on octets (kernels_ragged.hip)
void ragged_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Q, float *P,
                   double *ws, hipStream_t st);
void ragged_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat, double *ws,
                   float *Qout, hipStream_t st);
void strip_cs_pass_p(const DevicePlan &dp, const void *grads, const void *table, const float *Q, float *P, double *ws, hipStream_t st);
void strip_cs_pass_q(const DevicePlan &dp, const void *grads, const void *table, const float *Phat, double *ws, float *Qout,
                     hipStream_t st);
void generic_p_reduce(const DevicePlan &dp, double *ws, float *P, hipStream_t st);       // adds the column-chunk partials of P
void generic_q_reduce(const DevicePlan &dp, double *ws, float *Qout, hipStream_t st);   // adds the row-tile partials of Q+
void generic_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat,
                      const float *Qn, uint64_t step, hipStream_t st);
// The octet family's and the strip family's workgroups in one launch (kernels_mixed.hip), where that is the faster way:
// false if it is not, and then nothing has been enqueued.  The err pass takes the plan's err_t_items and err_w_items, or
// err_s_items where it has none of those.
bool mixed_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Q, float *P,
                  double *ws, hipStream_t st);
bool mixed_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales, const float *Phat, double *ws,
                  float *Qout, hipStream_t st);
bool mixed_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat, const float *Qn,
                    uint64_t step, hipStream_t st);
void octet_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales,
                  const float *Q, float *P, double *ws, hipStream_t st);
void octet_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales,
                  const float *Phat, double *ws, float *Qout, hipStream_t st);
void octet_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat,
                    const float *Qn, uint64_t step, hipStream_t st);

// MFMA family.
void mfma_pass_p(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales,
                 const float *Q, float *P, hipStream_t st);

void mfma_transpose_scales(const DevicePlan &dp, const float *scales, double *ws, bool second, hipStream_t st);
void mfma_pass_q(const DevicePlan &dp, const void *grads, const uint32_t *codes, const float *scales,
                 const float *Phat, double *ws, float *Qout, hipStream_t st);
void mfma_pass_err_two(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, uint32_t *codes2, float *scales2,
                       const float *Phat, const double *ws, uint64_t step, hipStream_t st);
void mfma_pass_err(const DevicePlan &dp, const void *grads, uint32_t *codes, float *scales, const float *Phat,
                   const double *ws, uint64_t step, hipStream_t st);
void mfma_split_q_new(const DevicePlan &dp, const float *Qn, double *ws, hipStream_t st);

}  // namespace conef
