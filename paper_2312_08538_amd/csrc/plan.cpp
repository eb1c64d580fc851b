#include "plan.h"

#include "../../include/conef.h"

#include <array>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <utility>

#include <algorithm>
#include <new>

namespace conef {

namespace {
constexpr int kOk = 0, kEinval = -1, kEnomem = -2;
constexpr int kMfmaPasses = 7;      // bit 0: P pass, bit 1: Q+ pass, bit 2: err pass
constexpr int kPackQRows = 512;     // rows per partial of Q+ of the packed-split Q+ pass

inline int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }
inline int64_t ceil_div(int64_t v, int64_t a) { return (v + a - 1) / a; }
inline bool is_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }
inline int log2i(int64_t v) { int s = 0; while ((int64_t(1) << s) < v) ++s; return s; }
}  // namespace

namespace {
int make_plan_impl(Plan &plan, const int64_t *rows, const int64_t *cols, int n_mats, int rank, int bits, int block,
                   int dtype, uint64_t seed, bool sketch, bool cs_lin_ok, bool all_generic = false);
}

int make_plan(Plan &plan, const int64_t *rows, const int64_t *cols, int n_mats, int rank, int bits,
              int block, int dtype, uint64_t seed)
{
    return make_plan_impl(plan, rows, cols, n_mats, rank, bits, block, dtype, seed, false, false);
}

namespace {
// Philox4x32-10 (Salmon et al., SC'11) on the host, for the set-up values the library derives from the seed
void host_philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint64_t seed, uint32_t out[4])
{
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)p1; c3 = (uint32_t)p0; c0 = n0; c2 = n2;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}
}  // namespace

void sketch_hash(uint64_t seed, uint32_t mat, uint32_t row, int64_t w, int32_t *bucket, bool *negative)
{
    // counter (row, matrix, ~0, ~0): the counter of a step no run reaches
    uint32_t out[4];
    host_philox4x32_10(row, mat, 0xFFFFFFFFu, 0xFFFFFFFFu, seed, out);
    *bucket = (int32_t)(((uint64_t)out[0] * (uint64_t)w) >> 32);
    *negative = (out[1] & 1u) != 0;
}

int64_t random_block_start(uint64_t seed, uint32_t mat, uint64_t step, int64_t N, int64_t k)
{
    // counter (matrix, ~0, step): no element draw uses it (their second word is a matrix index)
    uint32_t out[4];
    host_philox4x32_10(mat, 0xFFFFFFFFu, (uint32_t)step, (uint32_t)(step >> 32), seed, out);
    const uint64_t r = (uint64_t)out[0] | ((uint64_t)out[1] << 32);
    return (int64_t)(((unsigned __int128)r * (unsigned __int128)(uint64_t)(N - k + 1)) >> 64);
}

int configure_random_block(Plan &plan, const int64_t *keep)
{
    if (!keep) return kEinval;
    const int n_mats = (int)plan.mats.size();
    for (int l = 0; l < n_mats; ++l)
        if (keep[l] < 1 || keep[l] > plan.mats[l].N) return kEinval;
    try {
        int64_t off = 0;
        for (int l = 0; l < n_mats; ++l) {
            MatDesc &d = plan.mats[l];
            d.rb_k = keep[l];
            d.rb_delta_off = off;
            off += round_up(keep[l], kAlign);
        }
        plan.rb_delta_elems = (size_t)off;
    } catch (const std::bad_alloc &) {
        return kEnomem;
    }
    return kOk;
}

int64_t i2_block_start(uint64_t seed, uint32_t mat, uint64_t step, int64_t N, int64_t ke)
{
    // counter (matrix, ~0 - 1, step): neither the gradient compressor's block nor an element draw uses it
    uint32_t out[4];
    host_philox4x32_10(mat, 0xFFFFFFFEu, (uint32_t)step, (uint32_t)(step >> 32), seed, out);
    const uint64_t r = (uint64_t)out[0] | ((uint64_t)out[1] << 32);
    return (int64_t)(((unsigned __int128)r * (unsigned __int128)(uint64_t)(N - ke + 1)) >> 64);
}

int configure_i2(Plan &plan, const int64_t *keep_e)
{
    if (!keep_e) return kEinval;
    const int n_mats = (int)plan.mats.size();
    for (int l = 0; l < n_mats; ++l)
        if (keep_e[l] < 0 || keep_e[l] > plan.mats[l].N) return kEinval;
    int64_t off = 0;
    for (int l = 0; l < n_mats; ++l) {
        MatDesc &d = plan.mats[l];
        d.i2_k = keep_e[l];
        d.i2_off = off;
        off += round_up(keep_e[l], kAlign);
    }
    plan.i2_elems = (size_t)(off > 0 ? off : kAlign);
    plan.i2_configured = true;
    return kOk;
}

int64_t random_k_index(uint64_t seed, uint32_t mat, uint64_t step, int64_t N, int64_t G, int64_t i)
{
    // counter (stratum / 4, matrix + 2^30, step): four strata per call, word i % 4
    uint32_t out[4];
    host_philox4x32_10((uint32_t)(i >> 2), mat + 0x40000000u, (uint32_t)step, (uint32_t)(step >> 32), seed, out);
    const int64_t len = (N - i * G < G) ? N - i * G : G;
    return i * G + (int64_t)(((uint64_t)out[i & 3] * (uint64_t)len) >> 32);
}

int configure_random_k(Plan &plan, const int64_t *group)
{
    if (!group) return kEinval;
    const int n_mats = (int)plan.mats.size();
    if (n_mats >= (1 << 30)) return kEinval;
    for (int l = 0; l < n_mats; ++l)
        if (group[l] < 1 || group[l] > plan.mats[l].N || plan.mats[l].N >= ((int64_t)1 << 32)) return kEinval;
    int64_t off = 0;
    for (int l = 0; l < n_mats; ++l) {
        MatDesc &d = plan.mats[l];
        d.rk_g = (uint32_t)group[l];
        d.rk_pad = 0;
        // j / g = mulhi64(j, magic) for every j < 2^32: magic = 2^64 / g for a power of two (a shift), else
        // floor(2^64 / g) + 1, whose excess j (g - 2^64 mod g) / (g 2^64) < 2^-32 < 1 / g never reaches the next integer
        if (d.rk_g == 1) d.rk_magic = 0;
        else if ((d.rk_g & (d.rk_g - 1)) == 0) d.rk_magic = ((uint64_t)1 << 63) / (d.rk_g >> 1);
        else d.rk_magic = ~(uint64_t)0 / d.rk_g + 1;
        d.rk_delta_off = off;
        off += round_up((d.N + group[l] - 1) / group[l], kAlign);
    }
    plan.rk_delta_elems = (size_t)off;
    plan.rk_uniform = false;
    return kOk;
}

namespace {
uint32_t rku_mix(uint32_t u)
{
    u *= 0x9E3779B1u; u ^= u >> 15; u *= 0x85EBCA77u; u ^= u >> 13;
    return u;
}
}  // namespace

int configure_random_k_uniform(Plan &plan, const int64_t *keep)
{
    if (!keep) return kEinval;
    const int n_mats = (int)plan.mats.size();
    for (int l = 0; l < n_mats; ++l)
        if (keep[l] < 1 || keep[l] > plan.mats[l].N || plan.mats[l].N >= ((int64_t)1 << 32)) return kEinval;
    int64_t off = 0;
    for (int l = 0; l < n_mats; ++l) {
        MatDesc &d = plan.mats[l];
        d.rk_g = 0;
        d.rk_uk = (uint32_t)keep[l];
        uint64_t a = (uint64_t)std::sqrt((double)d.N);              // a = ceil(sqrt(N)), exactly
        while (a * a < (uint64_t)d.N) ++a;
        while (a > 1 && (a - 1) * (a - 1) >= (uint64_t)d.N) --a;
        d.rk_ua = (uint32_t)a;
        d.rk_ub = (uint32_t)(((uint64_t)d.N + a - 1) / a);
        d.rk_umagic = d.rk_ub == 1 ? 0 : ~(uint64_t)0 / d.rk_ub + 1;     // (a power of two: 2^64 / b, also exact)
        if (d.rk_ub > 1 && (d.rk_ub & (d.rk_ub - 1)) == 0) d.rk_umagic = ((uint64_t)1 << 63) / (d.rk_ub >> 1);
        d.rk_delta_off = off;
        off += round_up(keep[l], kAlign);
    }
    plan.rk_delta_elems = (size_t)off;
    plan.rk_uniform = true;
    return kOk;
}

int64_t random_k_uniform_index(uint64_t seed, uint32_t mat, uint64_t step, const MatDesc &d, int64_t i)
{
    uint32_t o0[4], o1[4];
    host_philox4x32_10(mat, 0xFFFFFFFDu, (uint32_t)step, (uint32_t)(step >> 32), seed, o0);
    host_philox4x32_10(mat, 0xFFFFFFFCu, (uint32_t)step, (uint32_t)(step >> 32), seed, o1);
    const uint32_t key[6] = {o0[0], o0[1], o0[2], o0[3], o1[0], o1[1]};
    const uint32_t a = d.rk_ua, b = d.rk_ub;
    uint32_t x = (uint32_t)i;
    do {                                                    // the rounds backwards, walked again while outside [0, N)
        uint32_t L = x / b, R = x % b;
        for (int r = 5; r >= 0; --r) {
            if ((r & 1) == 0) {
                const uint32_t f = (uint32_t)(((uint64_t)rku_mix(R ^ key[r]) * a) >> 32);
                L = L >= f ? L - f : L + a - f;
            } else {
                const uint32_t f = (uint32_t)(((uint64_t)rku_mix(L ^ key[r]) * b) >> 32);
                R = R >= f ? R - f : R + b - f;
            }
        }
        x = L * b + R;
    } while ((int64_t)x >= d.N);
    return (int64_t)x;
}

namespace {
// The column form: every matrix on the kernels for any shape; table rows x w; one hash per column; the update walks one row
// of the matrix per workgroup, over the bucket lists of columns.
int make_sketch_plan_columns(Plan &plan, const int64_t *rows, const int64_t *cols, const int64_t *buckets, int n_mats, int rank,
                             float beta, int table_dtype, int dtype, uint64_t seed)
{
    for (int l = 0; l < n_mats; ++l)
        if (buckets[l] < 1 || buckets[l] > cols[l] || cols[l] > kCscMaxCols) return kEinval;
    int rc = make_plan_impl(plan, rows, cols, n_mats, rank, 8, 4, dtype, seed, true, false, true);
    if (rc != kOk) return rc;
    try {
        plan.sketch = true; plan.sketch_cols = true; plan.beta = beta; plan.table_dtype = table_dtype;
        plan.code_words = 0; plan.n_scales = 0;
        int64_t t = 0, h = 0, bp = 0;
        for (int l = 0; l < n_mats; ++l) {
            MatDesc &d = plan.mats[l];
            d.w = buckets[l];
            d.table_off = t; t += round_up(d.n * d.w, kAlign);
            d.hash_off = h;  h += d.m;
            d.bptr_off = bp; bp += d.w + 1;
        }
        plan.table_elems = (size_t)t;
        plan.row_hash.assign((size_t)h, 0);
        plan.bucket_rows.assign((size_t)h, 0);
        plan.bucket_ptr.assign((size_t)bp, 0);
        // Update: eight rows per workgroup, fewer where that would leave less than 256 workgroups (960 rows of convolutions, rank
        // 4: 7.5 us in groups of two, 11.1 of eight, 9.4 one by one), and no more threads than the widest matrix has columns
        // (100000 x 33, rank 32: 142 us with 64 threads, 504 with 512).
        int64_t all_rows = 0, widest = 0;
        for (const MatDesc &d : plan.mats) { all_rows += d.n; widest = std::max(widest, d.m); }
        int32_t most_rows = 8;
        while (most_rows > 1 && all_rows / most_rows < 256) most_rows /= 2;
        plan.csc_threads = (int)std::min<int64_t>(kCscThreads, round_up(widest, 64));
        if (plan.csc_rows_p) {
            // (threads in equal trips over the widest matrix's columns)
            plan.csc_p_threads = (int)round_up(ceil_div(widest, ceil_div(widest, kCscThreads)), 64);
        }
        for (int l = 0; l < n_mats; ++l) {
            MatDesc &d = plan.mats[l];
            int32_t *ptr = plan.bucket_ptr.data() + d.bptr_off;
            for (int64_t k = 0; k < d.m; ++k) {
                int32_t b; bool neg;
                sketch_hash(seed, (uint32_t)l, (uint32_t)k, d.w, &b, &neg);
                plan.row_hash[(size_t)(d.hash_off + k)] = b | (neg ? INT32_MIN : 0);
                ptr[b + 1] += 1;
            }
            for (int64_t b = 0; b < d.w; ++b) ptr[b + 1] += ptr[b];
            std::vector<int32_t> fill(ptr, ptr + d.w);            // columns in ascending order within each bucket
            for (int64_t k = 0; k < d.m; ++k) {
                const int32_t hv = plan.row_hash[(size_t)(d.hash_off + k)];
                plan.bucket_rows[(size_t)(d.hash_off + fill[hv & INT32_MAX]++)] = (int32_t)k | (hv & INT32_MIN);
            }
            d.cs_cols = most_rows;
            while (d.cs_cols > 1 && d.cs_cols * (d.m + d.w) > kCscLds) d.cs_cols /= 2;
            // P pass by rows: the same rows with the table alone in LDS
            if (plan.csc_rows_p) {
                int32_t rows_p = most_rows;
                while (rows_p > 1 && rows_p * d.w > kCscLds) rows_p /= 2;
                for (int64_t i = 0; i < d.n; i += rows_p)
                    plan.csc_p_items.push_back({l, (int32_t)i, (int32_t)std::min<int64_t>(rows_p, d.n - i), rows_p});
                plan.csc_p_lds = std::max(plan.csc_p_lds, (int)(rows_p * d.w));
            }
            d.st_first = (int32_t)plan.cs_err_items.size();
            for (int64_t i = 0; i < d.n; i += d.cs_cols)
                plan.cs_err_items.push_back({l, (int32_t)i, (int32_t)std::min<int64_t>(d.cs_cols, d.n - i), 0});
            d.st_slots = 0;
        }
    } catch (const std::bad_alloc &) {
        return kEnomem;
    }
    return kOk;
}
}  // namespace

int make_sketch_plan(Plan &plan, const int64_t *rows, const int64_t *cols, const int64_t *sketch_rows, int n_mats,
                     int rank, float beta, int table_dtype, int dtype, uint64_t seed, bool columns)
{
    if (columns) {
        if (!sketch_rows || !(beta >= 0.0f && beta < 1.0f) || (table_dtype != 0 && table_dtype != 1)) return kEinval;
        if (!rows || !cols || n_mats < 1) return kEinval;
        return make_sketch_plan_columns(plan, rows, cols, sketch_rows, n_mats, rank, beta, table_dtype, dtype, seed);
    }
    if (!sketch_rows || !(beta >= 0.0f && beta < 1.0f) || (table_dtype != 0 && table_dtype != 1)) return kEinval;
    if (!rows || n_mats < 1) return kEinval;
    for (int l = 0; l < n_mats; ++l)
        if (sketch_rows[l] < 1 || sketch_rows[l] > rows[l]) return kEinval;
    // the quantiser's parameters are not used in this mode; any valid pair will do
    // the linear form (see MatDesc::cs_lin) needs an fp16 table: its entries split into two bf16 operands exactly
    int rc = make_plan_impl(plan, rows, cols, n_mats, rank, 8, 4, dtype, seed, true, table_dtype == 1);
    if (rc != kOk) return rc;
    try {
        plan.sketch = true; plan.beta = beta; plan.table_dtype = table_dtype;
        plan.code_words = 0; plan.n_scales = 0;
        int64_t t = 0, h = 0, bp = 0;
        for (int l = 0; l < n_mats; ++l) {
            MatDesc &d = plan.mats[l];
            d.w = sketch_rows[l];
            d.table_off = t; t += round_up(d.w * d.m, kAlign);
            d.hash_off = h;  h += d.n;
            d.bptr_off = bp; bp += d.w + 1;
        }
        plan.table_elems = (size_t)t;
        // rows per item of the octet path's update pass: as many as leave about 2048 items, 32 to 256 (an item
        // first loads its 512 rows of Q+; measured on 124 M to 1.3 G elements: 4096 and 1024 items are both slower)
        int64_t total_elems = 0;
        for (int l = 0; l < n_mats; ++l) total_elems += rows[l] * cols[l];
        const int64_t min_items = 2048;
        int64_t cs_rows = 32;
        while (cs_rows < 256 && total_elems / (cs_rows * 2 * 512) >= min_items) cs_rows *= 2;
        plan.row_hash.assign((size_t)h, 0);
        plan.bucket_rows.assign((size_t)h, 0);
        // (entries of the matrices whose P and Q+ passes read them, up to the last one of those)
        size_t ordered = 0;
        for (const MatDesc &d : plan.mats)
            if (reads_row_order(d)) ordered = (size_t)(d.hash_off + d.n);
        plan.row_order.resize(ordered);
        plan.bucket_ptr.assign((size_t)bp, 0);
        for (int l = 0; l < n_mats; ++l) {
            const MatDesc &d = plan.mats[l];
            int32_t *ptr = plan.bucket_ptr.data() + d.bptr_off;
            for (int64_t i = 0; i < d.n; ++i) {
                int32_t b; bool neg;
                sketch_hash(seed, (uint32_t)l, (uint32_t)i, d.w, &b, &neg);
                plan.row_hash[(size_t)(d.hash_off + i)] = b | (neg ? INT32_MIN : 0);
                ptr[b + 1] += 1;
            }
            for (int64_t b = 0; b < d.w; ++b) ptr[b + 1] += ptr[b];
            // rows in ascending order within each bucket (a counting sort keeps the order of arrival)
            std::vector<int32_t> fill(ptr, ptr + d.w);
            for (int64_t i = 0; i < d.n; ++i) {
                const int32_t hv = plan.row_hash[(size_t)(d.hash_off + i)];
                const int32_t b = hv & INT32_MAX;
                const size_t at = (size_t)(d.hash_off + fill[b]++);
                plan.bucket_rows[at] = (int32_t)i | (hv & INT32_MIN);
                if (reads_row_order(d)) plan.row_order[at] = {plan.bucket_rows[at], b};
            }
            // buckets per item: about 16 rows of the matrix each (at most 64 buckets); on the octet path, where
            // a workgroup first loads 512 rows of Q+, `cs_rows` rows (at most 256 buckets)
            const bool fast = d.path == kPathOctet;
            const int64_t nb = fast ? std::max<int64_t>(1, std::min<int64_t>(256, cs_rows * d.w / d.n))
                                    : std::max<int64_t>(1, std::min<int64_t>(64, 16 * d.w / d.n));
            plan.mats[l].cs_cols = fast ? 512 : kCsCols;
            const int32_t nct = (int32_t)ceil_div(d.m, plan.mats[l].cs_cols);
            std::vector<WorkItem> &items = fast ? plan.cs_err_f_items : plan.cs_err_items;
            plan.mats[l].st_first = (int32_t)items.size();
            for (int64_t b0 = 0; b0 < d.w; b0 += nb)
                for (int32_t ct = 0; ct < nct; ++ct)
                    items.push_back({l, (int32_t)b0, (int32_t)std::min<int64_t>(nb, d.w - b0), ct});
            // element-wise gradient compressors walk the same items: one partial l1 sum per wave (octet path: one
            // wave per item, else four)
            plan.mats[l].st_slots = (int32_t)(items.size() - plan.mats[l].st_first) * (fast ? 1 : kCsCols / 64);
            plan.mats[l].st_atomic = fast ? 0 : 1;
        }
        int64_t wd = (int64_t)plan.ws_doubles;
        for (int l = 0; l < n_mats; ++l) {
            plan.mats[l].st_part_off = wd;
            wd += plan.mats[l].st_slots;
        }
        // the linear form: T and U, partial sums of the Q+ pass for the table's row tiles behind the gradient's, work tables
        for (int l = 0; l < n_mats; ++l) {
            MatDesc &d = plan.mats[l];
            if (!d.cs_lin) continue;
            d.cs_t_off = wd; wd += round_up(d.w * 32, 32);
            d.cs_u_off = wd; wd += round_up(d.w * 32 / 2, 32);
            d.cs_q_tiles_g = d.n_q_tiles;
            const int32_t tiles_t = (int32_t)ceil_div(d.w, d.q_tile_rows);
            d.n_q_tiles = d.cs_q_tiles_g + tiles_t;
            d.qpart_off = wd; wd += round_up((int64_t)d.n_q_tiles * d.m * 32, 32);
            for (int64_t r0 = 0; r0 < d.w; r0 += kMfmaRows) plan.cs_t_items.push_back({l, (int32_t)r0, 0, 0});
            for (int32_t rt = 0; rt < tiles_t; ++rt)
                for (int32_t cp = 0; cp < (int32_t)((d.m / 128 + 1) / 2); ++cp) plan.cs_qt_items.push_back({l, cp, rt, 0});
            for (int64_t b0 = 0; b0 < d.w; b0 += 8) plan.cs_u_items.push_back({l, (int32_t)b0, (int32_t)std::min<int64_t>(8, d.w - b0), 0});
            for (int64_t b0 = 0; b0 < d.w; b0 += 128)
                for (int32_t st = 0; st < (int32_t)(d.m / 128); ++st)
                    plan.cs_lin_items.push_back({l, st, (int32_t)b0, (int32_t)std::min<int64_t>(128, d.w - b0)});
        }
        plan.ws_doubles = (size_t)round_up(wd, 32);
        plan.workspace_bytes = (size_t)round_up((int64_t)plan.ws_doubles * 8, 256);
    } catch (const std::bad_alloc &) {
        return kEnomem;
    }
    return kOk;
}

namespace {
int make_plan_impl(Plan &plan, const int64_t *rows, const int64_t *cols, int n_mats, int rank, int bits, int block,
                   int dtype, uint64_t seed, bool sketch, bool cs_lin_ok, bool all_generic)
{
    if (!rows || !cols || n_mats < 1) return kEinval;
    if (rank < 1 || rank > kMaxRank) return kEinval;
    if (bits != 2 && bits != 4 && bits != 8) return kEinval;
    const int W = 32 / bits;
    if (block < W || block % W != 0 || block > (1 << 20)) return kEinval;
    if (dtype != 0 && dtype != 1) return kEinval;
    for (int l = 0; l < n_mats; ++l) {
        if (rows[l] < 1 || cols[l] < 1) return kEinval;
        if (rows[l] > (int64_t(1) << 31) - 1 || cols[l] > (int64_t(1) << 31) - 1) return kEinval;
        if (rows[l] * cols[l] >= (int64_t(1) << 35)) return kEinval;
        if (rank > rows[l] || rank > cols[l]) return kEinval;
    }
    try {
        plan = Plan();
        plan.rank = rank; plan.bits = bits; plan.block = block; plan.dtype = dtype; plan.seed = seed;
        plan.rpad = rank <= 4 ? 4 : rank <= 8 ? 8 : rank <= 16 ? 16 : 32;
        plan.wshift = log2i(W);
        plan.inv_s = 1.0f / (float)((1 << (bits - 1)) - 1);
        plan.bmagic = is_pow2(block) ? ((uint64_t)1 << 63) / (uint64_t)(block >> 1) : ~(uint64_t)0 / (uint64_t)block + 1;
        // blocks that a power-of-two number of lanes, at most a wave, holds in octets: the strip err pass takes them
        const bool octet_blocks = block % 8 == 0 && is_pow2(block / 8) && block / 8 <= 64;
        plan.lb_shift = octet_blocks ? log2i(block / 8) : 0;
        plan.block_shift = is_pow2(block) ? log2i(block) : -1;
        plan.mats.resize(n_mats);

        // The octet family needs whole scale blocks per row, a power-of-two number of lanes (8 elements
        // each) per block, at most one wave wide, and rank 2, 4 or 8.  Its P pass stages codes and scales
        // in 128-byte lines: blocks of at least 64 elements and rows of a multiple of 64 columns.
        const bool block_ok = block % 8 == 0 && is_pow2(block / 8) && block / 8 <= 64 && block >= 64;
        // CONEF_PACK=0 in the environment keeps the octet family's own P and Q+ passes (fp64 matrix cores, results that agree
        // with a plain fp64 loop to the last bits) for the matrices that would otherwise take the packed-split passes
        const char *pack_env = std::getenv("CONEF_PACK");
        const bool pack_enabled = !(pack_env && pack_env[0] == '0');
        int64_t total_elems = 0;
        for (int l = 0; l < n_mats; ++l) total_elems += rows[l] * cols[l];
        // rows per wave item of the err pass: aim at >= ~8192 wave items over the model (measured on 124 M and
        // 210 M elements: half and twice as many rows per item are both slower)
        int err_rows = 128;
        while (err_rows > 8 && total_elems / ((int64_t)err_rows * 512) < 8192) err_rows >>= 1;
        // rows per wave item of the Q+ pass (64 columns wide): at least 4000 wave items, a matrix's rows in equal tiles (124 M fp32
        // elements at rank 4, most of them in matrices of 768 rows: 128 / 256 / 384 / 512 rows 363.6 / 361.0 / 358.6 / 366.8 us a step,
        // 365.5 with 256 and short last tiles)
        int q_rows = 512;
        for (int rows : {384, 256, 192, 128, 96, 64})
            if (total_elems / ((int64_t)q_rows * 64) < 4000) q_rows = rows;
        // columns per workgroup item of the P pass (64 rows high): a multiple of every code group
        // (1024 / bits columns) and of every block size of the family
        const int p_cols = 512;

        int64_t g = 0, w = 0, s = 0, p = 0, q = 0, wd = 0, strip_elems = 0;
        for (int l = 0; l < n_mats; ++l) {
            MatDesc &d = plan.mats[l];
            d = MatDesc();
            d.n = rows[l]; d.m = cols[l]; d.N = d.n * d.m;
            d.nblk = ceil_div(d.N, block);
            d.grad_off = g;  g += round_up(d.N, kAlign);
            d.word_off = w;  w += round_up(ceil_div(d.N, W), kAlign);
            d.scale_off = s; s += round_up(d.nblk, kAlign);
            d.p_off = p;     p += round_up(d.n * rank, kAlign);
            d.q_off = q;     q += round_up(d.m * rank, kAlign);
            d.path = (!sketch && block_ok && (rank == 2 || rank == 4 || rank == 8) && d.m % 64 == 0 && d.m % block == 0 && d.m <= kOctetMaxCols) ? kPathOctet
                                                                                             : kPathGeneric;
            // count-sketch mode: the octet path needs whole octets per row only (16-byte aligned rows of
            // the gradient and of the table), at any rank
            const bool sketch_octet = sketch && !all_generic && d.m % 8 == 0 && d.m <= kOctetMaxCols;
            d.m8 = (int32_t)(d.m / 8);
            d.lb_shift = block_ok ? log2i(block / 8) : 0;
            d.cs_lin = (sketch && cs_lin_ok && rank == 32 && dtype == 1 && d.m % 128 == 0 && d.m <= (1 << 24)) ? 1 : 0;
            if (sketch_octet) d.path = kPathOctet;
            else if (d.path == kPathOctet) {
                // lanes per row segment: the largest power of two <= 64 that divides m/8 and holds a block
                int lr = 64;
                while (lr > 8 && (d.m8 % lr) != 0) lr >>= 1;
                if ((d.m8 % lr) != 0 || lr < (block / 8)) d.path = kPathGeneric;
                d.lr_shift = log2i(lr);
            }
            // MFMA family: dense rank-32 contractions on the matrix cores
            if (!sketch && rank == 32 && dtype == 1 && bits == 4 && block == 128 && d.m % 128 == 0 && d.m <= (1 << 24)) d.path = kPathMfma;
            // octet family: the err pass with the residual on the fp32 matrix cores, in strips of 128 columns (256 for blocks of 256)
            d.err_tile = (d.path == kPathOctet && !sketch && (rank == 4 || rank == 8) && block <= 256 &&
                          d.m % (block == 256 ? 256 : 128) == 0) ? 1 : 0;
            // octet family: the P and Q+ passes on the bf16 matrix cores with packed factor splits
            d.pack = (pack_enabled && d.path == kPathOctet && !sketch && dtype == 1 && (bits == 2 || bits == 4) && block >= 128 &&
                      d.m % 128 == 0 && d.m <= (1 << 24)) ? 1 : 0;
            if (d.path == kPathOctet) plan.any_octet = true;
            else if (d.path == kPathMfma) plan.any_mfma = true;
            else {
                plan.any_generic = true;
                strip_elems += d.N;
            }
        }
        // The strip kernels: about 1536 workgroups per launch (six per CU) where the model is large enough, with limits that
        // keep a workgroup's fixed part (operand set-up, the sum over its waves, partial sums to be added later) small
        // against its share of the elements.  The P pass on octets: 512, since fewer of them fit on a CU (three at rank 4, two at rank
        // 32) and a wave with several strips has the next one's loads in flight (us for the pass, chunks for 1536 / 512 workgroups:
        // 600 x 20001 fp32 at rank 1 23.5 / 17.8, at 16 29.8 / 23.1, six of 2600 x 650 at rank 4 18.6 / 11.5, at 32 32.4 / 22.7, 4000 x
        // 5001 at 8 27.8 / 25.7, smaller models the same).
        // Where no matrix has more than 512 columns they stay in one chunk: a wave has two strips then, and the launch that adds
        // the chunks, which nothing else needs, costs more (600 x 300 at rank 4: 9.3 us for the pass in two chunks, 7.8 in one;
        // not so with the sketch, whose gathered rows are the longer chain: 10.3 and 11.6).
        int64_t widest = 0;
        for (const MatDesc &d : plan.mats) widest = std::max(widest, d.m);
        const int64_t strip_chunk = !sketch && widest <= 512 ? 512
            : std::min<int64_t>(2048, std::max<int64_t>(256, round_up(strip_elems / (kStripRows * (!sketch && octet_blocks ? 512 : 1536)), 256)));
        auto on_octets = [&](const MatDesc &d) { return !sketch && octet_blocks && d.path == kPathGeneric && d.m <= kRaggedMaxCols; };
        // the Q+ pass of most of these matrices decides for all of them (two launches cost more than either form does), and where
        // the octet family's kernels run too, the launch for both takes them on octets
        int64_t pays = 0, of = 0;
        bool joint = false;
        for (const MatDesc &d : plan.mats) {
            joint = joint || (d.path == kPathOctet && !d.pack);
            if (!on_octets(d) || d.n <= kFlatRows) continue;
            of += d.N;
            if (ragged_q_pays(rank, d.n, strip_elems)) pays += d.N;
        }
        const bool q_octets = joint || 2 * pays >= of;
        auto q_on_octets = [&](const MatDesc &d) { return q_octets && on_octets(d); };
        // On octets a wave works in steps of 32 rows, and a workgroup's four waves have one each.  Above rank 16 a CU holds one
        // workgroup or two: 256 of them with more steps each (rank 32, fp32, in tiles for 1024 / 256 workgroups: 10000 x 650 59 / 30
        // us, 100000 x 65 95 / 50, 256 x 20001 47 / 35; element by element 52, 77 and 40).
        const int64_t ragged_q_rows = std::min<int64_t>(512, std::max<int64_t>(128, round_up(strip_elems / (64 * (rank > 16 ? 256 : 1024)), 128)));
        const int64_t strip_q_rows = std::min<int64_t>(512, std::max<int64_t>(32, round_up(strip_elems / (64 * 1536), 32)));
        const int64_t strip_err = strip_elems / 8192 >= 1024 ? 8192 : strip_elems / 4096 >= 768 ? 4096 : strip_elems / 2048 >= 64 ? 2048 : 1024;
        bool coarse_gram = false;
        // times: how much coarser the row tiles of the strip Q+ pass are than by the rules above
        // Octet Q+ pass: where no matrix has more than 256 rows a workgroup takes a strip whole, a quarter of the rows per wave, and
        // writes Q+; nothing is left for the launch that adds partial sums.  us a step without / so: fp32 at rank 4 64 x 2048 25.6 / 21.9,
        // 256 x 8192 29.6 / 27.5, 600 x 2048 28.4 / 29.2, 1000 x 512 28.2 / 32.3; bf16, 8-bit codes, at rank 8 64 x 512 32.6 / 27.3, 256 x 2048
        // 38.0 / 35.4, 600 x 512 39.4 / 49.2, 80 of 256 x 1024 93 / 90.
        // Models of more than 112 MB of gradients and codes in rows of up to 1024 columns (512 at rank 8) have enough workgroups, and few
        // enough partial sums, without: 400 of 256 x 512 at rank 4 152.7 / 159.6, at rank 2 143 / 152, with two vectors 256 of them 131 / 141; 500 of
        // 64 x 1024 at rank 4 119.3 / 121.4, at rank 8 154 / 152; 128 of 256 x 2048 at rank 4 222 / 207; below, 128 of 256 x 512 at rank 4 59.3 / 59.4,
        // 64 of them 37.9 / 37.6.
        int64_t all_rows = 0;
        for (const MatDesc &d : plan.mats) all_rows += d.n;
        const int64_t model_bits = total_elems * ((dtype == 0 ? 32 : 16) + bits);
        bool q_joined = !sketch && !(model_bits > (int64_t)7 << 27 && total_elems <= all_rows * (rank <= 4 ? 1024 : 512));
        for (const MatDesc &d : plan.mats) q_joined = q_joined && (d.path != kPathOctet || d.pack || d.n <= 256);
        plan.q_joined = q_joined;
        // Column sketch, P pass: by whole rows (k_csc_p) for ranks up to 4, where most elements are in matrices of 1024 columns or more and
        //   - the rows are one workgroup of four per CU (1024), or up to some four of eight for three CUs (2048 to 3200), which the strip
        //     kernels' launches do not get below: 1024 x 2500 strips / rows 42.3 / 40.4 us a step, 2200 x 1024 40.1 / 39.2, 3000 x 2500 59.4 / 53.9;
        //   - or, beyond, the rows are long enough to pay for a workgroup's table and sums: 1700 columns in the mean, or most elements in
        //     matrices of 2500 or more, whose strips are in several chunks.  6000 x 2000 72.8 / 67.9, 8000 x 4998 287.6 / 235.9, 18-layer residual
        //     network of 64 channels 92.6 / 87.6, of 96 211 / 180, GPT layers of 1024 491 / 478; 16000 x 1024 83.1 / 88.8, 16000 x 1500 123.0 / 123.6, GPT
        //     layers of 512 140 / 160, of 768 312 / 335, 43.7 M elements in matrices of 650 columns 168 / 206.
        // Between, in workgroups of four rows and a second, short turn of them, from 12 M elements on: 1500 x 1024 34.0 / 41.6, 1135 x 9000
        // 130.1 / 136.6, 1500 x 9000 153.9 / 153.0, 2000 x 9000 160.0 / 137.6.  Fewer rows: 64 x 16000 57 / 62.  Rank 8: the network of 64 channels 154 / 192.
        int64_t wide_elems = 0, very_wide_elems = 0;
        for (const MatDesc &d : plan.mats) {
            wide_elems += d.m >= 1024 ? d.N : 0;
            very_wide_elems += d.m >= 2500 ? d.N : 0;
        }
        const bool rows_pay = all_rows <= 1024 ? all_rows == 1024
                            : all_rows < 2048  ? total_elems >= 12000000
                                               : all_rows <= 3200 || total_elems >= 1700 * all_rows || 2 * very_wide_elems >= total_elems;
        const bool rows_p = all_generic && rank <= 4 && 2 * wide_elems >= total_elems && rows_pay;
        plan.csc_rows_p = rows_p;
        auto lay_out = [&](int64_t chunk_cols, int64_t times) {
            wd = 0;
            plan.any_p_chunks = false;
            for (int l = 0; l < n_mats; ++l) {
                MatDesc &d = plan.mats[l];
                if (d.path == kPathMfma) {
                    d.scT_off = wd; wd += round_up((d.m / 128) * d.n * 4 / 8 + 1, 32);
                    d.scT2_off = wd; wd += round_up((d.m / 128) * d.n * 4 / 8 + 1, 32);
                    d.qs_off = wd;  wd += round_up(3 * 32 * d.m * 2 / 8, 32);
                }

                d.gram_tile_rows = d.n > 8192 ? 2 * kGramRows : kGramRows;
                if (rank <= 8) d.gram_tile_rows = (int32_t)std::max<int64_t>(gram_rows_small(d.n), coarse_gram ? d.gram_tile_rows : 0);
                d.n_gram_tiles = (int32_t)ceil_div(d.n, d.gram_tile_rows);
                d.gram_off = wd; wd += (int64_t)d.n_gram_tiles * rank * rank;
                if (rank > 8) {                     // up to 8 the sum and the factor stay in the second launch's workgroups
                    d.gsum_off = wd; wd += rank * rank;
                    d.rinv_off = wd; wd += rank * rank;
                }
                d.q_tile_rows = d.cs_lin ? 2048 : d.pack ? kPackQRows : d.path == kPathOctet ? (int32_t)round_up(ceil_div(d.n, ceil_div(d.n, q_rows)), 32) : (d.path == kPathMfma && (kMfmaPasses & 2)) ? 2048
                                : (int32_t)std::min<int64_t>(std::min<int64_t>(512, times * (q_on_octets(d) ? ragged_q_rows : strip_q_rows)),
                                                             4 * std::max<int64_t>(1, kStripSpan / d.m));
                if (q_joined && d.path == kPathOctet && !d.pack) d.q_tile_rows = (int32_t)round_up(ceil_div(d.n, 4), 32);
                d.n_q_tiles = q_joined && d.path == kPathOctet && !d.pack ? 1 : (int32_t)ceil_div(d.n, d.q_tile_rows);
                d.qpart_off = wd; wd += round_up((int64_t)d.n_q_tiles * d.m * rank, 32);
                d.n_p_chunks = 1;
                d.p_chunk_cols = (int32_t)d.m;
                const bool strip = d.path == kPathGeneric;
                if (((d.path == kPathOctet && !d.cs_lin && !d.pack) || strip) && !rows_p) {
                    // strip kernels: chunks of one size, a multiple of a strip
                    d.p_chunk_cols = strip ? (int32_t)std::min<int64_t>(round_up(ceil_div(d.m, ceil_div(d.m, chunk_cols)), 64), INT32_MAX / 64 * 64) : p_cols;
                    d.n_p_chunks = (int32_t)ceil_div(d.m, d.p_chunk_cols);
                    if (d.n_p_chunks > 1) {
                        d.ppart_off = wd; wd += round_up((int64_t)d.n_p_chunks * d.n * rank, 32);
                        plan.any_p_chunks = true;
                    }
                }
            }
        };
        // Stream kernels of the element-wise gradient compressors for the quantiser: the wave-per-run kernel needs blocks of
        // 8 * 2^j elements (j <= 6).  A wave takes eight runs of 512 elements, fewer where that would leave the chip with fewer
        // than eight waves per SIMD (a wave's items are one serial chain of loads), and leaves one partial sum; elsewhere a
        // wave takes 16 blocks, or one of a small matrix.
        const bool stream_ok = block % 8 == 0 && is_pow2(block / 8) && block / 8 <= 64;
        const int64_t stream_runs_rule = std::min<int64_t>(8, std::max<int64_t>(1, total_elems / (512 * 8192)));
        int64_t stream_runs = stream_runs_rule;
        auto blocks_per_wave = [](const MatDesc &d) { return d.nblk <= 16384 ? 1 : 16; };
        auto stream_slots = [&](const MatDesc &d) {
            return stream_ok ? ceil_div(ceil_div(d.N, 512), stream_runs) : 4 * ceil_div(d.nblk, 4 * blocks_per_wave(d));
        };
        lay_out(strip_chunk, 1);
        // Partial sums of small and middle-sized models at high ranks can take the workspace beyond the static one of
        // conef_step_static (98304 wave-rows x 32 entries: 25 MB), and so can the partial Gram matrices of 64 rows of models of
        // hundreds of matrices at ranks up to 8 (350 of 8192 x 64 at rank 8: 44 MB, 28 with 256 rows).  They are split more
        // coarsely until it fits: first the Gram matrices (256 rows, 512 of more than 8192), then whole rows of P and 512 rows
        // per partial of Q+ are the least, then longer items of the stream kernels.  Where that does not fit either, nothing
        // is gained by a coarser split.
        auto fits = [&]() {
            int64_t all = wd;
            for (const MatDesc &d : plan.mats) all += stream_slots(d);
            return all <= (int64_t)CONEF_STATIC_WORKSPACE_BYTES / 8;
        };
        if (!sketch && !fits()) {
            coarse_gram = true;
            lay_out(strip_chunk, 1);
            for (int64_t k = 2; k <= 16 && strip_elems > 0 && !fits(); k *= 2)
                lay_out(strip_chunk * k, k);
            if (strip_elems > 0 && !fits()) lay_out(INT32_MAX, 16);
            while (stream_ok && stream_runs < 64 && !fits()) stream_runs *= 2;
            if (!fits()) {
                stream_runs = stream_runs_rule;
                coarse_gram = false;
                lay_out(strip_chunk, 1);
            }
        }
        // The strip err pass: runs of the flat index of strip_err elements where that is at least eight rows (a wave's row of
        // Q+ per lane serves all rows of a run), else eight rows of a column segment.
        // With Q+ in LDS: all of them or none, since two launches cost more than the others gain (400 x 650 beside 100 x 5000 29.7 us
        // a step on strips, 34.1 in two launches, 16000 x 650 beside 2000 x 5000 94.5 and 97); matrices of less than eight columns,
        // which have a launch of their own, aside.  About 2048 workgroups, eight per CU (512 - 4096 of them are within 6 %).
        auto walks = [&](const MatDesc &d) { return rank <= 8 && d.path == kPathGeneric && d.m >= 8 && walk_lds(d.m, rank) <= kWalkLds; };
        int64_t walk_elems = 0, thin_elems = 0;
        for (const MatDesc &d : plan.mats) {
            walk_elems += walks(d) ? d.N : 0;
            thin_elems += rank <= 8 && d.path == kPathGeneric && d.m < 8 ? d.N : 0;
        }
        const bool walk = walk_elems + thin_elems == strip_elems;
        const int64_t walk_runs = std::min<int64_t>(64, 4 * std::max<int64_t>(1, ceil_div(walk_elems / 512, 4 * 2048)));
        // Matrices of up to 32 columns that are not among those (less than eight columns, ranks above 8) are walked in groups of rows,
        // by a launch of their own.  With 16 columns or more they do not pay for one beside other matrices (64 x 27 in a small
        // convolutional network: 10 - 17 us for the pass without groups, 15 - 21 with; the launches of 600 x 27 alone 9.0 and 7.7).
        bool all_narrow = true;
        for (const MatDesc &d : plan.mats) all_narrow = all_narrow && d.m <= 32;
        for (int l = 0; l < n_mats && !sketch && octet_blocks; ++l) {
            MatDesc &d = plan.mats[l];
            if (d.path != kPathGeneric) continue;
            d.es_rows = 1;
            if (walk && walks(d)) {
                d.es_walk = 1;
                plan.ew_lds = std::max(plan.ew_lds, (int)walk_lds(d.m, rank));
                continue;
            }
            if (d.m <= 1024) {
                if (d.m < 16 || (all_narrow && d.m <= 32)) d.es_rows = (int32_t)(64 / d.m);
                int64_t tile = strip_err;
                while (tile < 8192 && tile < 8 * d.m && strip_elems / tile >= 512) tile *= 2;      // (shorter runs rather than an empty chip)
                d.es_tile = (int32_t)round_up(tile, block);
                plan.es_lds = std::max(plan.es_lds, d.es_tile + 8);
            } else {
                const bool whole = d.m % block == 0;
                const int64_t cols_want = std::max<int64_t>(strip_err / 8, whole ? block : 2 * block);
                d.es_seg = (int32_t)(whole ? round_up(cols_want, block) : ceil_div(d.m, ceil_div(d.m, cols_want)));
                d.es_over = whole ? 0 : block;
                d.es_pitch = (int32_t)round_up(d.es_seg + d.es_over, 8);
                plan.es_lds = std::max(plan.es_lds, 8 * d.es_pitch + 8);
            }
        }
        // The step in one launch
        if (!sketch && octet_blocks && rank <= 8 && !coarse_gram && small_pays(n_mats, total_elems)) {
            for (const MatDesc &d : plan.mats) {
                const int64_t lds = small_lds_bytes(d.n, d.m, plan.rpad);
                if (d.pack || d.m % 8 != 0 || d.n > kSmallMaxRows || d.N > kSmallMaxElems || lds > kSmallLds) {
                    plan.small_lds = 0;
                    break;
                }
                plan.small_lds = std::max(plan.small_lds, lds);
            }
        }
        // Stream tables of the element-wise gradient compressors.
        // The scaled sign's norm pass goes backwards in models of more than 256 MB: the pass behind it begins with what the last-level
        // cache still holds of it.  In smaller ones it only takes an item to another XCD than the one that has it in its L2.  us for the
        // step, forwards / backwards: fp32 with 8-bit codes 5 M elements 17.7 / 19.0, 24 M 57.0 / 57.6, 50 M (251 MB) 109.5 / 109.3, 67 M 159.0 / 145.3,
        // 134 M 309.6 / 287.7; bf16 with 2-bit codes 8 M 18.2 / 19.2, 100 M (226 MB) 111.0 / 111.8, 134 M (302 MB) 148.7 / 142.4; two vectors, fp32
        // with 4-bit codes, 33 M (167 MB) 83.9 / 84.0, 67 M (335 MB) 163.2 / 149.4.
        plan.norm_back = model_bits > (int64_t)8 << 28;
        plan.norm_back_two = model_bits + total_elems * bits > (int64_t)8 << 28;
        int64_t sw = 0;
        for (int l = 0; l < n_mats; ++l) {
            MatDesc &d = plan.mats[l];
            d.sign_off = sw; sw += round_up(ceil_div(d.N, 32), kAlign);
            if (sketch) continue;                   // the count-sketch mode walks its bucket lists
            if (stream_ok) {
                d.lb_shift = log2i(block / 8);
                const int64_t runs = ceil_div(d.N, 512);
                d.st_first = (int32_t)plan.rb_items.size();
                for (int64_t r0 = 0; r0 < runs; r0 += stream_runs)
                    plan.rb_items.push_back({l, (int32_t)r0, (int32_t)std::min<int64_t>(stream_runs, runs - r0), 0});
            } else {
                const int32_t per_wave = blocks_per_wave(d);
                d.st_first = (int32_t)plan.rb_g_items.size();
                for (int64_t b0 = 0; b0 < d.nblk; b0 += 4 * per_wave) plan.rb_g_items.push_back({l, (int32_t)b0, per_wave, 0});
                d.st_atomic = 1;
            }
            d.st_slots = (int32_t)stream_slots(d);       // one per wave (four waves per item of the second kind)
            d.st_part_off = wd; wd += d.st_slots;
        }
        plan.sign_words = (size_t)sw;
        plan.grad_elems = (size_t)g; plan.code_words = (size_t)w; plan.n_scales = (size_t)s;
        plan.p_elems = (size_t)p; plan.q_elems = (size_t)q;
        plan.ws_doubles = (size_t)round_up(wd, 32);
        plan.workspace_bytes = (size_t)round_up((int64_t)plan.ws_doubles * 8, 256);

        // The orthonormalisation in one launch (kOrthRows)
        bool orth_rows = rank <= 8 && !coarse_gram && n_mats <= (rank <= 4 ? 512 : 128);
        for (const MatDesc &d : plan.mats) orth_rows = orth_rows && d.n <= orth_most_rows(rank) && d.n * d.n_p_chunks <= 5000;
        // Rows per item (wave) of the octet family's err pass on the matrix cores: 64, 128 at rank 8, whose rows of Q+ an item loads
        // first are twice as many, and fewer where that would leave less than 800 items; at least a trip's 16.  us a step with 16 / 32 /
        // 64 / 128 rows: 124 M fp32 elements at rank 4 387 / 367 / 362 / 366, at rank 8 491 / 453 / 434 / 427; 210 M bf16 at rank 8 480 / 425
        // / 400 / 382; 2000 x 4096 at rank 4 44.5 / 43.5 / 42.6 / 48.8, 8000 x 2048 in blocks of 256 at rank 8 88 / 84 / 82 / 94; 256 x 2048
        // 26.5 / 28.4 / 31.8 / 38.5.
        const int64_t tile_cols = block == 256 ? 256 : 128;
        int64_t err_t_elems = 0, err_t_rows = rank == 8 ? 128 : 64;
        for (const MatDesc &d : plan.mats) err_t_elems += d.err_tile ? d.N : 0;
        while (err_t_rows > 16 && err_t_elems / (err_t_rows * tile_cols) < 800) err_t_rows /= 2;
        // the longest table, an entry per 1024 elements
        int64_t n_elem = 0;
        for (const MatDesc &d : plan.mats) n_elem += ceil_div(d.N, 1024);
        plan.elem_items.reserve((size_t)n_elem);
        for (int l = 0; l < n_mats; ++l) {
            const MatDesc &d = plan.mats[l];
            // passes of the MFMA family that exist; the others fall back to the generic kernels
            const bool mf = d.path == kPathMfma;
            const bool mf_p = (mf && (kMfmaPasses & 1)) || d.cs_lin, mf_q = (mf && (kMfmaPasses & 2)) || d.cs_lin,
                       mf_e = mf && (kMfmaPasses & 4);
            if (mf_p) {
                for (int64_t r0 = 0; r0 < d.n; r0 += kMfmaRows) plan.p_m_items.push_back({l, (int32_t)r0, 0, 0});
            }
            if (mf_q) {
                // one item per pair of neighbouring column blocks (the last pair of an odd count has one)
                for (int32_t rt = 0; rt < d.n_q_tiles; ++rt)
                    for (int32_t cp = 0; cp < (int32_t)((d.m / 128 + 1) / 2); ++cp) plan.q_m_items.push_back({l, cp, rt, 0});
            }
            if ((mf_q || mf_e) && mf)
                for (int64_t r0 = 0; r0 < d.n; r0 += 64) plan.split_p_items.push_back({l, (int32_t)(r0 / 64), 0, 0});
            if (mf_e) {
                for (int64_t k0 = 0; k0 < d.m; k0 += 64) plan.split_qn_items.push_back({l, (int32_t)(k0 / 64), 0, 0});
                const int32_t ncb = (int32_t)(d.m / 128);
                for (int64_t r0 = 0; r0 < d.n; r0 += kErrRows)
                    for (int32_t cb0 = 0; cb0 < ncb; cb0 += kErrRun)
                        plan.err_m_items.push_back({l, (int32_t)r0, cb0, std::min<int32_t>(kErrRun, ncb - cb0)});
            }
            if (d.path == kPathGeneric || mf) {
                const int64_t prow = std::min<int64_t>(kStripRows, std::max<int64_t>(1, kStripSpan / d.m));
                if (!mf_p && !rows_p)
                    for (int64_t r0 = 0; r0 < d.n; r0 += prow)
                        for (int32_t cc = 0; cc < d.n_p_chunks; ++cc)
                            (on_octets(d) ? plan.p_r_items : plan.p_items).push_back({l, (int32_t)r0, cc, (int32_t)std::min<int64_t>(prow, d.n - r0)});
                const int32_t nct = (int32_t)ceil_div(d.m, 64);
                if (!mf_q && d.n <= kFlatRows && d.n_q_tiles == 1 && d.N <= kStripSpan)
                    for (int32_t ct = 0; ct < nct; ct += 4) plan.q_flat_items.push_back({l, ct / 4, 0, 0});
                else if (!mf_q)
                    for (int32_t rt = 0; rt < d.n_q_tiles; ++rt)
                        for (int32_t ct = 0; ct < nct; ++ct) (q_on_octets(d) ? plan.q_r_items : plan.q_items).push_back({l, ct, rt, 0});
                if (!mf_p && d.n_p_chunks > 1)
                    for (int64_t e0 = 0; e0 < d.n * rank; e0 += 256) plan.pred_items.push_back({l, (int32_t)e0, 0, 0});
                if (!mf_e && !sketch && d.es_walk) {
                    const int64_t runs = ceil_div(d.N, 512);
                    for (int64_t r0 = 0; r0 < runs; r0 += walk_runs)
                        plan.err_w_items.push_back({l, (int32_t)r0, (int32_t)std::min<int64_t>(walk_runs, runs - r0), (int32_t)(r0 * 512 / d.m)});
                }
                if (!mf_e && !sketch && d.es_tile > 0)
                    for (int64_t t = 0; t * d.es_tile < d.N; ++t) {
                        const int64_t row = d.m * d.es_rows;
                        const int64_t i0 = t * d.es_tile / row, i1 = (std::min<int64_t>((t + 1) * d.es_tile, d.N) - 1) / row;
                        (d.es_rows > 1 ? plan.err_g_items : plan.err_s_items).push_back({l, (int32_t)t, (int32_t)i0, (int32_t)(i1 - i0 + 1)});
                    }
                const int64_t erow = std::min<int64_t>(8, std::max<int64_t>(1, kStripSpan / d.m));
                if (!mf_e && !sketch && d.es_seg > 0)
                    for (int64_t r0 = 0; r0 < d.n; r0 += erow)
                        for (int32_t sg = 0; sg < (int32_t)ceil_div(d.m, d.es_seg); ++sg)
                            plan.err_s_items.push_back({l, (int32_t)r0, sg, (int32_t)std::min<int64_t>(erow, d.n - r0)});
                // 4 waves per workgroup, each wave takes blocks b0+wave, b0+wave+4, ...: 16 per wave, or
                // one per wave for small matrices (a: first block, b: blocks per wave)
                if (!mf_e && !sketch && d.es_tile == 0 && d.es_seg == 0 && !d.es_walk) {
                    const int32_t per_wave = d.nblk <= 16384 ? 1 : 16;
                    for (int64_t b0 = 0; b0 < d.nblk; b0 += 4 * per_wave)
                        plan.err_items.push_back({l, (int32_t)b0, per_wave, 0});
                }
            } else if (!d.cs_lin) {
                const int lr = 1 << d.lr_shift, rw = 64 / lr;
                const int32_t strips = d.m8 / lr;
                // consecutive items are the column chunks of one row tile: they run side by side on one
                // XCD and share the lines of block scales that span several chunks
                for (int64_t r0 = 0; r0 < d.n && !d.pack; r0 += kPTileRows)
                    for (int32_t cc = 0; cc < d.n_p_chunks; ++cc) plan.p_f_items.push_back({l, (int32_t)r0, cc, 0});
                const int32_t qstrips = (int32_t)ceil_div(d.m, 64);
                for (int32_t rt = 0; rt < d.n_q_tiles && !d.pack; ++rt)
                    for (int32_t st = 0; st < qstrips; ++st) plan.q_f_items.push_back({l, st, rt, 0});
                if (d.pack) {
                    // one item per 128 rows (dealt to the XCDs further down); one per pair of neighbouring column blocks and row tile
                    for (int64_t r0 = 0; r0 < d.n; r0 += kMfmaRows) plan.p_k_items.push_back({l, (int32_t)r0, 0, 0});
                    for (int32_t rt = 0; rt < d.n_q_tiles; ++rt)
                        for (int32_t cp = 0; cp < (int32_t)((d.m / 128 + 1) / 2); ++cp) plan.q_k_items.push_back({l, cp, rt, 0});
                }
                const int64_t rows_item = (int64_t)std::max(err_rows, rw);
                // the err pass with the residual on the fp32 matrix cores: strips of 128 columns (256 for blocks of 256)
                if (d.err_tile) {
                    for (int64_t r0 = 0; r0 < d.n; r0 += err_t_rows)
                        for (int32_t st = 0; st < (int32_t)(d.m / tile_cols); ++st)
                            plan.err_t_items.push_back({l, st, (int32_t)r0, (int32_t)std::min<int64_t>(err_t_rows, d.n - r0)});
                }
                for (int64_t r0 = 0; r0 < d.n && !sketch && !d.err_tile; r0 += rows_item)
                    for (int32_t st = 0; st < strips; ++st)
                        plan.err_f_items.push_back({l, st, (int32_t)r0, (int32_t)std::min<int64_t>(rows_item, d.n - r0)});
                if (d.n_p_chunks > 1)
                    for (int64_t e0 = 0; e0 < d.n * rank; e0 += 256) plan.pred_items.push_back({l, (int32_t)e0, 0, 0});
            }
            if (rank <= 8) {
                if (orth_rows) plan.orth_first.push_back((int32_t)plan.gram_s_items.size());
                for (int64_t t = 0; t < d.n_gram_tiles; ++t)
                    plan.gram_s_items.push_back({d.p_off, t * d.gram_tile_rows, std::min<int64_t>((t + 1) * d.gram_tile_rows, d.n), d.n,
                                                 d.gram_off + t * rank * rank, d.ppart_off, d.n_gram_tiles, d.n_p_chunks, 0});
                const int64_t per = apply_rows(rank, d.n);
                for (int64_t r0 = 0; r0 < d.n; r0 += per)
                    plan.apply_s_items.push_back({d.p_off, r0, std::min<int64_t>(r0 + per, d.n), d.n, d.gram_off, 0, d.n_gram_tiles, 0, 0});
            } else {
                for (int32_t t = 0; t < d.n_gram_tiles; ++t) plan.gram_items.push_back({l, t, 0, 0});
                for (int64_t r0 = 0; r0 < d.n; r0 += 64) plan.apply_items.push_back({l, (int32_t)r0, 0, 0});
            }
            // a matrix-core matrix with a single row tile gets its Q+ straight from the Q+ pass
            if (!((mf_q || d.pack || d.path == kPathGeneric || q_joined) && d.n_q_tiles == 1) || d.cs_lin)
            {
                // 256 entries per workgroup, a thread per entry; with kQredManyTiles partial sums or more per entry, 16
                // entries per workgroup and 16 threads per entry (item.c = 1)
                const int per = (!d.cs_lin && d.n_q_tiles >= kQredManyTiles) ? 16 : 256;      // (the sketch's linear form adds tiles later)
                for (int64_t e0 = 0; e0 < d.m * rank; e0 += per)
                    plan.qred_items.push_back({l, (int32_t)e0, 0, per == 16 ? 1 : 0});
            }
            for (int64_t e0 = 0; e0 < d.N; e0 += 1024) plan.elem_items.push_back({l, (int32_t)(e0 >> 10), 0, 0});
        }
        // The Q+ pass of a model of more than 256 MB goes backwards: it begins with what the P pass has just read, and the err pass,
        // forwards again, with what it ends on, of which the 256 MB last-level cache still holds a part.  us a step, forwards / so: 124 M
        // fp32 elements at rank 4 369.0 / 359.7, two vectors 462.8 / 457.7; 210 M bf16 at rank 8 391.3 / 389.7, the row sketch 460.3 /
        // 457.8; models many times as large the same; 28 M fp32, which fit into the cache whole, 106.5 / 107.3.  (The
        // matrix-core tables dealt to the XCDs in the P pass's order, shape by shape: 388.8, not worth its code.)
        if (model_bits > ((int64_t)8 << 28))
            for (auto *items : {&plan.q_items, &plan.q_r_items, &plan.q_f_items, &plan.q_m_items, &plan.q_k_items})
                std::reverse(items->begin(), items->end());
        // Decompress / update: row tiles per workgroup.  On the matrix cores a workgroup keeps its strip of Q+ for several of
        // them (a matrix's tiles in equal shares), where that leaves enough workgroups.  Measured, rank 32, a tile / 4 / 8 tiles
        // per workgroup: 4096 x 8192 (4096 tiles) 64 / 54 / 52 us, 4096 x 4096 35 / 32 / 28, 15.7 M elements in ten matrices
        // (1920 tiles) 34 / 32 / 51, 2048 x 2048 (512 tiles) 11.6 / 14.7 / 21.  Rows that do not start on 16-byte boundaries
        // cannot be fetched ahead: a tile per workgroup (33278 x 650, rank 16: 103 us, four tiles 129), and models with more
        // than an eighth of such tiles stay with the kernel for one tile, whose waves are twice as many.
        int64_t upd_total = 0, upd_odd = 0;
        for (const MatDesc &d : plan.mats) {
            const int64_t tiles = ceil_div(d.n, kUpdRows) * ceil_div(d.m, kUpdCols);
            upd_total += tiles;
            if (d.m % 4 != 0) upd_odd += tiles;
        }
        plan.upd_many = update_on_cores(rank) && upd_total >= 1024 && 8 * upd_odd <= upd_total ? 1 : 0;
        // (up to rank 16 the strip of Q+ is paid for by four tiles, and shorter items end more evenly: 124 M elements 216 us, eight
        // tiles 232; rank 32: 257 and 249)
        const int64_t upd_most = plan.upd_many ? std::min<int64_t>(rank <= 16 ? 4 : 8, std::max<int64_t>(4, upd_total / 512)) : 1;
        for (int l = 0; l < n_mats; ++l) {
            const MatDesc &d = plan.mats[l];
            const int64_t tiles = ceil_div(d.n, kUpdRows), per = d.m % 4 == 0 ? ceil_div(tiles, ceil_div(tiles, upd_most)) : 1;
            for (int64_t t = 0; t < tiles; t += per)
                for (int64_t c0 = 0; c0 < d.m; c0 += kUpdCols)
                    plan.upd_items.push_back({l, (int32_t)t, (int32_t)(c0 / kUpdCols), (int32_t)std::min<int64_t>(per, tiles - t)});
        }
        // The P pass of the matrix-core family: workgroups are dealt to the eight XCDs in turn (workgroup b runs on
        // XCD b % 8), and a pass streams faster when every XCD stays inside an address range of its own (measured
        // with a read-only kernel of this tile shape: 5.7 TB/s against 4.4 TB/s for tiles dealt round-robin).  So
        // the table is cut into eight lists, one per XCD, entry j of list x at index x * L + j:
        //   - matrices of one shape in groups of eight go whole, one to each XCD; what is left of a shape is cut
        //     into eight contiguous row ranges;
        //   - every list holds its items longest rows first (a workgroup walks a whole row range, so its duration
        //     grows with the number of columns, and the last workgroups to start should be the short ones); the
        //     lists have the same shapes at the same positions, so the XCDs stay in step;
        //   - lists are padded to one length L with empty items (mat = -1).
        auto xcd_lists = [&](std::vector<WorkItem> &table, auto member) {
            if (table.empty()) return;
            std::vector<int> order;                         // the family's matrices, longest rows first, then by shape
            for (int l = 0; l < n_mats; ++l)
                if (member(plan.mats[l])) order.push_back(l);
            std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
                const MatDesc &a = plan.mats[x], &b = plan.mats[y];
                return a.m != b.m ? a.m > b.m : a.n > b.n;
            });
            std::vector<WorkItem> lists[8];
            size_t i = 0;
            int rot = 0;
            while (i < order.size()) {
                size_t j = i;
                while (j < order.size() && plan.mats[order[j]].m == plan.mats[order[i]].m && plan.mats[order[j]].n == plan.mats[order[i]].n) ++j;
                const size_t whole = (j - i) / 8 * 8;
                for (size_t k = i; k < i + whole; ++k) {           // whole matrices, eight at a time
                    const int l = order[k], x = (int)((k - i) / ((j - i) / 8));
                    for (int64_t r0 = 0; r0 < plan.mats[l].n; r0 += kMfmaRows) lists[x].push_back({l, (int32_t)r0, 0, 0});
                }
                for (size_t k = i + whole; k < j; ++k) {           // the rest: eight row ranges each
                    const int l = order[k];
                    const int64_t T = ceil_div(plan.mats[l].n, kMfmaRows);
                    for (int x = 0; x < 8; ++x) {
                        const int dst = (x + rot) & 7;            // remainders of successive matrices fall on different XCDs
                        for (int64_t t = x * T / 8; t < (x + 1) * T / 8; ++t) lists[dst].push_back({l, (int32_t)(t * kMfmaRows), 0, 0});
                    }
                    ++rot;
                }
                i = j;
            }
            size_t L = 0;
            for (const auto &v : lists) L = std::max(L, v.size());
            table.clear();
            for (auto &v : lists) {
                v.resize(L, WorkItem{-1, 0, 0, 0});
                table.insert(table.end(), v.begin(), v.end());
            }
        };
        xcd_lists(plan.p_m_items, [](const MatDesc &d) { return (d.path == kPathMfma && (kMfmaPasses & 1)) || d.cs_lin; });
        xcd_lists(plan.p_k_items, [](const MatDesc &d) { return d.pack != 0; });
        // The err pass in strips: items are dispatched in table order, and a kernel ends when its last wave does.  With a
        // few thousand equal items on a chip that holds two or three thousand waves, the last items to start run on a
        // nearly empty chip for a whole item's duration.  So the items at the end of the table are cut into shorter ones
        // (rows stay multiples of the 16 of a trip): halves from 75 % of the work on, quarters from 90 % (measured on 124 M
        // and 210 M elements: 6 - 7 % on the pass; cutting earlier or finer costs more in short items than it gains).  Up to
        // 2048 items, two workgroups per CU, start side by side, and there is no end to fill (16384 x 1024 at rank 4, 2048 items, cut / whole:
        // fp32 65.9 / 63.5, bf16 54.0 / 52.9; 130 of 256 x 512, 2080: 63.0 / 65.9; 5000 x 4096, 2528: 78.1 / 79.5, bf16 66.8 / 68.4).
        if (plan.err_t_items.size() > 2048) {
            int64_t total = 0, done = 0;
            for (const WorkItem &it : plan.err_t_items) total += it.c;
            std::vector<WorkItem> cut;
            cut.reserve(plan.err_t_items.size() * 2);
            for (const WorkItem &it : plan.err_t_items) {
                const int parts = done * 10 >= total * 9 ? 4 : done * 4 >= total * 3 ? 2 : 1;
                const int32_t piece = std::max<int32_t>(16, (int32_t)round_up(ceil_div(it.c, parts), 16));
                for (int32_t r0 = 0; r0 < it.c; r0 += piece)
                    cut.push_back({it.mat, it.a, it.b + r0, std::min<int32_t>(piece, it.c - r0)});
                done += it.c;
            }
            plan.err_t_items.swap(cut);
        }
    } catch (const std::bad_alloc &) {
        return kEnomem;
    }
    return kOk;
}
}  // namespace

namespace {

struct Cover {
    std::vector<int64_t> area;                                   // per matrix
    std::vector<std::array<int32_t, 4>> seen;                    // items, for the duplicate check
    bool ok = true;
    explicit Cover(size_t n) : area(n, 0) {}
    // a rectangle [r0, r0 + rows) x [c0, c0 + cols), clipped to the matrix; must start inside it
    void add(const Plan &plan, const WorkItem &it, int64_t r0, int64_t rows, int64_t c0, int64_t cols)
    {
        if (it.mat < 0 || it.mat >= (int)plan.mats.size()) { ok = false; return; }
        const MatDesc &d = plan.mats[it.mat];
        if (r0 < 0 || c0 < 0 || r0 >= d.n || c0 >= d.m || rows <= 0 || cols <= 0) { ok = false; return; }
        area[it.mat] += std::min<int64_t>(rows, d.n - r0) * std::min<int64_t>(cols, d.m - c0);
        seen.push_back({it.mat, it.a, it.b, it.c});
    }
    void add_elems(const Plan &plan, const WorkItem &it, int64_t e0, int64_t count)      // a run of the flat index
    {
        if (it.mat < 0 || it.mat >= (int)plan.mats.size()) { ok = false; return; }
        const MatDesc &d = plan.mats[it.mat];
        if (e0 < 0 || e0 >= d.N || count <= 0) { ok = false; return; }
        area[it.mat] += std::min<int64_t>(count, d.N - e0);
        seen.push_back({it.mat, it.a, it.b, it.c});
    }
    bool complete(const Plan &plan)
    {
        if (!ok) return false;
        std::sort(seen.begin(), seen.end());
        if (std::adjacent_find(seen.begin(), seen.end()) != seen.end()) return false;
        for (size_t l = 0; l < plan.mats.size(); ++l)
            if (area[l] != plan.mats[l].N) return false;
        return true;
    }
};

}  // namespace

bool check_plan(const Plan &plan)
{
    const size_t nm = plan.mats.size();
    // random-k: the multiply-high division by the stratum length, on the coordinates around every kind of boundary
    if (plan.rk_delta_elems != 0 && plan.rk_uniform)
        for (const MatDesc &d : plan.mats) {
            // the keyed permutation's shape and its division by b, on the coordinates around every kind of boundary
            if (d.rk_g != 0 || d.rk_uk < 1 || d.rk_uk > d.N || d.N >= ((int64_t)1 << 32)) return false;
            const uint64_t a = d.rk_ua, b = d.rk_ub;
            if (a * a < (uint64_t)d.N || (a > 1 && (a - 1) * (a - 1) >= (uint64_t)d.N) || b != ((uint64_t)d.N + a - 1) / a) return false;
            if (b == 1) continue;
            const uint64_t last = a * b - 1;
            const uint64_t probes[] = {0, 1, b - 1, b, b + 1, 2 * b - 1, last / 2, last / b * b - 1, last / b * b, last - 1, last,
                                       0xFFFFFFFFull / b * b - 1, 0xFFFFFFFFull / b * b, 0xFFFFFFFFull};
            for (uint64_t j : probes) {
                j &= 0xFFFFFFFFull;
                if ((uint64_t)(((unsigned __int128)j * d.rk_umagic) >> 64) != j / b) return false;
            }
        }
    else if (plan.rk_delta_elems != 0)
        for (const MatDesc &d : plan.mats) {
            if (d.rk_g < 1 || d.rk_g > d.N || d.N >= ((int64_t)1 << 32)) return false;
            if (d.rk_g == 1) continue;
            const uint64_t g = d.rk_g, last = (uint64_t)d.N - 1;
            const uint64_t probes[] = {0, 1, g - 1, g, g + 1, 2 * g - 1, 2 * g, last / 2, last / g * g - 1, last / g * g, last - 1, last,
                                       0xFFFFFFFFull / g * g - 1, 0xFFFFFFFFull / g * g, 0xFFFFFFFEull, 0xFFFFFFFFull};
            for (uint64_t j : probes) {
                j &= 0xFFFFFFFFull;
                if ((uint64_t)(((unsigned __int128)j * d.rk_magic) >> 64) != j / g) return false;
            }
        }
    // pass 1: P = p Q
    {
        Cover c(nm);
        // the kernels' own end of a chunk, on the last chunk of every row
        for (const MatDesc &d : plan.mats) {
            const int64_t c_begin = (int64_t)(d.n_p_chunks - 1) * d.p_chunk_cols;
            if (d.n_p_chunks < 1 || c_begin < 0 || c_begin >= d.m || chunk_end(d.m, d.p_chunk_cols, (int)c_begin) != d.m) return false;
        }
        for (const WorkItem &it : plan.p_items)
            c.add(plan, it, it.a, it.c <= kStripRows && it.c * plan.mats[it.mat].m < 2 * kStripSpan * 2 ? it.c : 0,
                  (int64_t)it.b * plan.mats[it.mat].p_chunk_cols, plan.mats[it.mat].p_chunk_cols);
        for (const WorkItem &it : plan.csc_p_items) {
            if (!plan.sketch_cols || plan.rank > 4 || it.b > it.c || it.c > 8 || it.c * plan.mats[it.mat].w > plan.csc_p_lds) return false;
            c.add(plan, it, it.a, it.b, 0, plan.mats[it.mat].m);
        }
        for (const WorkItem &it : plan.p_r_items) {
            const MatDesc &d = plan.mats[it.mat];
            if (plan.sketch || d.m > kRaggedMaxCols || it.c > kStripRows) return false;
            c.add(plan, it, it.a, it.c, (int64_t)it.b * d.p_chunk_cols, d.p_chunk_cols);
        }
        for (const std::vector<WorkItem> *items : {&plan.p_f_items, &plan.q_f_items})
            for (const WorkItem &it : *items)
                if (plan.sketch && !reads_row_order(plan.mats[it.mat])) return false;
        for (const WorkItem &it : plan.p_f_items)
            c.add(plan, it, it.a, kPTileRows, (int64_t)it.b * plan.mats[it.mat].p_chunk_cols, plan.mats[it.mat].p_chunk_cols);
        if (plan.p_m_items.size() % 8 != 0) return false;                  // eight lists of one length
        for (const WorkItem &it : plan.p_m_items)
            if (it.mat >= 0) c.add(plan, it, it.a, kMfmaRows, 0, INT64_MAX);           // (mat = -1: padding)
        if (plan.p_k_items.size() % 8 != 0) return false;
        for (const WorkItem &it : plan.p_k_items)
            if (it.mat >= 0) {
                if (!plan.mats[it.mat].pack) return false;
                c.add(plan, it, it.a, kMfmaRows, 0, INT64_MAX);
            }
        if (!c.complete(plan)) return false;
    }
    // pass 2: Q+ = p^T P^
    {
        Cover c(nm);
        for (const WorkItem &it : plan.q_items)
            c.add(plan, it, (int64_t)it.b * plan.mats[it.mat].q_tile_rows, plan.mats[it.mat].q_tile_rows, (int64_t)it.a * 64, 64);
        for (const WorkItem &it : plan.q_r_items) {
            const MatDesc &d = plan.mats[it.mat];
            if (plan.sketch || d.m > kRaggedMaxCols || d.q_tile_rows % 128 != 0) return false;
            c.add(plan, it, (int64_t)it.b * d.q_tile_rows, d.q_tile_rows, (int64_t)it.a * 64, 64);
        }
        for (const WorkItem &it : plan.q_flat_items) {
            const MatDesc &d = plan.mats[it.mat];
            if (d.n > kFlatRows || plan.rank > kFlatRows || d.n_q_tiles != 1 || d.N > kStripSpan) return false;
            c.add(plan, it, 0, d.n, (int64_t)it.a * 256, 256);
        }
        for (const WorkItem &it : plan.q_f_items) {
            const MatDesc &d = plan.mats[it.mat];
            if (plan.q_joined && (plan.sketch || it.b != 0 || d.n_q_tiles != 1 || 4 * (int64_t)d.q_tile_rows < d.n)) return false;
            c.add(plan, it, (int64_t)it.b * d.q_tile_rows, plan.q_joined ? d.n : d.q_tile_rows, (int64_t)it.a * 64, 64);
        }
        for (const WorkItem &it : plan.q_m_items)
            c.add(plan, it, (int64_t)it.b * plan.mats[it.mat].q_tile_rows, plan.mats[it.mat].q_tile_rows, (int64_t)it.a * 256, 256);
        for (const WorkItem &it : plan.q_k_items)
            c.add(plan, it, (int64_t)it.b * plan.mats[it.mat].q_tile_rows, plan.mats[it.mat].q_tile_rows, (int64_t)it.a * 256, 256);
        if (!c.complete(plan)) return false;
    }
    // pass 3 of the count-sketch mode, column form: every row of every matrix once; bucket lists hold every column once, ascending
    if (plan.sketch && plan.sketch_cols) {
        std::vector<int64_t> rows_seen(nm, 0);
        for (const WorkItem &it : plan.cs_err_items) {
            if (it.mat < 0 || it.mat >= (int)nm || it.a != rows_seen[it.mat] || it.b < 1 || it.b > plan.mats[it.mat].cs_cols) return false;
            rows_seen[it.mat] += it.b;
        }
        for (size_t l = 0; l < nm; ++l) {
            const MatDesc &d = plan.mats[l];
            if (rows_seen[l] != d.n || d.m > kCscMaxCols || d.path != kPathGeneric) return false;
            const int32_t *ptr = plan.bucket_ptr.data() + d.bptr_off;
            if (ptr[0] != 0 || ptr[d.w] != d.m) return false;
            std::vector<char> seen(d.m, 0);
            for (int64_t b = 0; b < d.w; ++b) {
                if (ptr[b + 1] < ptr[b]) return false;
                for (int32_t k = ptr[b]; k < ptr[b + 1]; ++k) {
                    const int32_t hv = plan.bucket_rows[(size_t)(d.hash_off + k)], c = hv & INT32_MAX;
                    if (c >= d.m || seen[c]) return false;
                    if (k > ptr[b] && c <= (plan.bucket_rows[(size_t)(d.hash_off + k - 1)] & INT32_MAX)) return false;
                    if (plan.row_hash[(size_t)(d.hash_off + c)] != ((int32_t)b | (hv & INT32_MIN))) return false;
                    seen[c] = 1;
                }
            }
        }
    } else
    // pass 3 of the count-sketch mode: every table entry once; bucket lists hold every row once, ascending
    if (plan.sketch) {
        std::vector<int64_t> area(nm, 0);
        for (const std::vector<WorkItem> *tab : {&plan.cs_err_items, &plan.cs_err_f_items})
            for (const WorkItem &it : *tab) {
                if (it.mat < 0 || it.mat >= (int)nm) return false;
                const MatDesc &d = plan.mats[it.mat];
                if ((d.path == kPathOctet) != (tab == &plan.cs_err_f_items)) return false;
                if (it.a < 0 || it.b < 1 || it.a + it.b > d.w || it.c < 0 || (int64_t)it.c * d.cs_cols >= d.m) return false;
                area[it.mat] += (int64_t)it.b * std::min<int64_t>(d.cs_cols, d.m - (int64_t)it.c * d.cs_cols);
            }
        for (size_t l = 0; l < nm; ++l) {
            const MatDesc &d = plan.mats[l];
            if (area[l] != d.w * d.m) return false;
            const int32_t *ptr = plan.bucket_ptr.data() + d.bptr_off;
            if (ptr[0] != 0 || ptr[d.w] != d.n) return false;
            std::vector<char> seen(d.n, 0);
            for (int64_t b = 0; b < d.w; ++b) {
                if (ptr[b + 1] < ptr[b]) return false;
                for (int32_t k = ptr[b]; k < ptr[b + 1]; ++k) {
                    const int32_t hv = plan.bucket_rows[(size_t)(d.hash_off + k)], i = hv & INT32_MAX;
                    if (i >= d.n || seen[i]) return false;
                    if (k > ptr[b] && i <= (plan.bucket_rows[(size_t)(d.hash_off + k - 1)] & INT32_MAX)) return false;
                    if (plan.row_hash[(size_t)(d.hash_off + i)] != ((int32_t)b | (hv & INT32_MIN))) return false;
                    // the octet kernels take their rows of gradient, table and factor from here
                    if (reads_row_order(d) && ((size_t)(d.hash_off + k) >= plan.row_order.size() ||
                                               plan.row_order[(size_t)(d.hash_off + k)] != std::array<int32_t, 2>{hv, (int32_t)b}))
                        return false;
                    seen[i] = 1;
                }
            }
        }
    } else
    // pass 3: residual, quantiser, pack
    {
        Cover c(nm);
        for (const WorkItem &it : plan.err_items) c.add_elems(plan, it, (int64_t)it.a * plan.block, (int64_t)4 * it.b * plan.block);
        for (const WorkItem &it : plan.err_s_items) {
            const MatDesc &d = plan.mats[it.mat];
            if (d.es_rows != 1) return false;
            if (d.es_seg > 0) {
                // the blocks that start in this rectangle: up to es_over columns more per row, inside the pitch
                if (d.es_pitch < d.es_seg + d.es_over || (d.m % plan.block != 0 && d.es_over < plan.block) ||
                    (d.m % plan.block == 0 && d.es_seg % plan.block != 0) || 8 * d.es_pitch > plan.es_lds || it.c > 8)
                    return false;
                // every lane of the last segment's strips takes its row of Q+ from this matrix, the owners of an element from its column
                const int64_t c0 = (int64_t)it.b * d.es_seg;
                if (it.a == 0 && c0 + d.es_seg >= d.m) {
                    const int64_t own = d.m - c0 + d.es_over;
                    for (int64_t v = 0; v < round_up(own, 64); ++v) {
                        const int64_t k = virtual_column((uint32_t)d.m, (uint32_t)c0, (uint32_t)v);
                        if (k < 0 || k >= d.m || (v < own && k != std::min<int64_t>((c0 + v) % d.m, d.m - 1))) return false;
                    }
                }
                c.add(plan, it, it.a, it.c, (int64_t)it.b * d.es_seg, d.es_seg);
            } else {
                const int64_t j0 = (int64_t)it.a * d.es_tile, j1 = std::min<int64_t>(j0 + d.es_tile, d.N);
                if (d.es_tile % plan.block != 0 || d.es_tile > plan.es_lds || it.b != j0 / d.m || it.b + it.c - 1 != (j1 - 1) / d.m)
                    return false;
                c.add_elems(plan, it, j0, d.es_tile);
            }
        }
        for (const WorkItem &it : plan.err_w_items) {
            const MatDesc &d = plan.mats[it.mat];
            if (!d.es_walk || it.b < 1 || it.b > 64 || it.c != (int64_t)it.a * 512 / d.m || walk_lds(d.m, plan.rank) > plan.ew_lds) return false;
            c.add_elems(plan, it, (int64_t)it.a * 512, (int64_t)it.b * 512);
        }
        for (const WorkItem &it : plan.err_g_items) {
            const MatDesc &d = plan.mats[it.mat];
            const int64_t j0 = (int64_t)it.a * d.es_tile, j1 = std::min<int64_t>(j0 + d.es_tile, d.N), group = d.m * d.es_rows;
            if (d.es_rows < 2 || group > 64 || d.es_seg != 0 || d.es_tile % plan.block != 0 || d.es_tile > plan.es_lds ||
                it.b != j0 / group || it.b + it.c - 1 != (j1 - 1) / group)
                return false;
            c.add_elems(plan, it, j0, d.es_tile);
        }
        for (const WorkItem &it : plan.err_f_items) {
            const int64_t strip = (int64_t)8 << plan.mats[it.mat].lr_shift;
            c.add(plan, it, it.b, it.c, (int64_t)it.a * strip, strip);
        }
        for (const WorkItem &it : plan.err_t_items) {
            const int64_t strip = plan.block == 256 ? 256 : 128;
            if (!plan.mats[it.mat].err_tile) return false;
            c.add(plan, it, it.b, it.c, (int64_t)it.a * strip, strip);
        }
        for (const WorkItem &it : plan.err_m_items) c.add(plan, it, it.a, kErrRows, (int64_t)it.b * 128, (int64_t)it.c * 128);
        if (!c.complete(plan)) return false;
    }
    // decompression / update
    {
        Cover c(nm);
        for (const WorkItem &it : plan.upd_items) {
            if (it.c < 1 || it.c > (plan.upd_many ? 8 : 1)) return false;
            c.add(plan, it, (int64_t)it.a * kUpdRows, (int64_t)it.c * kUpdRows, (int64_t)it.b * kUpdCols, kUpdCols);
        }
        if (!c.complete(plan)) return false;
    }
    // per-matrix helpers, and the workspace map
    std::vector<std::pair<int64_t, int64_t>> regions;            // [begin, end) in doubles
    std::vector<int64_t> gram(nm, 0), apply(nm, 0), qred(nm, 0), pred(nm, 0);
    for (const WorkItem &it : plan.gram_items) gram[it.mat] += 1;
    for (const WorkItem &it : plan.apply_items) apply[it.mat] += 1;
    if (plan.rank <= 8) {                                        // in the order of the matrices, each row once
        auto rows_once = [&](const std::vector<OrthItem> &items, std::vector<int64_t> &count, bool partial) {
            size_t l = 0;
            int64_t next = 0;
            for (const OrthItem &it : items) {
                while (l < nm && next == plan.mats[l].n) { ++l; next = 0; }
                if (l == nm) return false;
                const MatDesc &d = plan.mats[l];
                if (it.p_off != d.p_off || it.n != d.n || it.row0 != next || it.row1 <= it.row0 || it.row1 > d.n || it.tiles != d.n_gram_tiles)
                    return false;
                if (it.gram_off != d.gram_off + (partial ? count[l] * plan.rank * plan.rank : 0)) return false;
                if (partial && (it.chunks != d.n_p_chunks || it.ppart_off != d.ppart_off)) return false;
                next = it.row1;
                count[l] += 1;
            }
            return l + 1 == nm && next == plan.mats[l].n;
        };
        if (!rows_once(plan.gram_s_items, gram, true) || !rows_once(plan.apply_s_items, apply, false)) return false;
        // the orthonormalisation in one launch: an item per matrix, its first one, and no more rows or tiles than a workgroup holds
        if (!plan.orth_first.empty()) {
            if (plan.orth_first.size() != nm) return false;
            int64_t first = 0;
            for (size_t l = 0; l < nm; ++l) {
                const MatDesc &d = plan.mats[l];
                if (plan.orth_first[l] != first || d.n > orth_most_rows(plan.rank) || d.gram_tile_rows != 64 || d.n_gram_tiles > 16) return false;
                first += d.n_gram_tiles;
            }
        }
    } else if (!plan.orth_first.empty()) {
        return false;
    }
    // the step in one launch: every matrix inside the kernel's limits and the launch's LDS
    if (plan.small_lds > 0) {
        if (plan.sketch || plan.rank > 8 || plan.rank > plan.rpad || plan.small_lds > kSmallLds || plan.block % 8 != 0 ||
            plan.block / 8 > 64 || plan.block != 8 << plan.lb_shift)
            return false;
        for (const MatDesc &d : plan.mats)
            if (d.n > kSmallMaxRows || d.N > kSmallMaxElems || d.m % 8 != 0 || d.m8 * 8 != d.m || d.pack || d.lb_shift != plan.lb_shift ||
                small_lds_bytes(d.n, d.m, plan.rpad) > plan.small_lds)
                return false;
    }
    for (const WorkItem &it : plan.qred_items) qred[it.mat] += 1;
    for (const WorkItem &it : plan.pred_items) pred[it.mat] += 1;
    for (size_t l = 0; l < nm; ++l) {
        const MatDesc &d = plan.mats[l];
        if (gram[l] != d.n_gram_tiles || apply[l] != ceil_div(d.n, plan.rank <= 8 ? apply_rows(plan.rank, d.n) : 64)) return false;
        const bool direct_q = (d.path == kPathMfma || d.path == kPathGeneric || d.pack || plan.q_joined) && d.n_q_tiles == 1;
        if (d.pack && (d.path != kPathOctet || d.n_p_chunks != 1 || (d.m & 127) != 0 || plan.block < 128 || plan.dtype != 1 ||
                       (plan.bits != 2 && plan.bits != 4)))
            return false;
        const int64_t qper = (!d.cs_lin && d.n_q_tiles >= kQredManyTiles) ? 16 : 256;
        if (qred[l] != (direct_q ? 0 : (d.m * plan.rank + qper - 1) / qper)) return false;
        if (pred[l] != (d.n_p_chunks > 1 ? (d.n * plan.rank + 255) / 256 : 0)) return false;
        regions.push_back({d.gram_off, d.gram_off + (int64_t)d.n_gram_tiles * plan.rank * plan.rank});
        if (plan.rank > 8) {
            regions.push_back({d.gsum_off, d.gsum_off + (int64_t)plan.rank * plan.rank});
            regions.push_back({d.rinv_off, d.rinv_off + (int64_t)plan.rank * plan.rank});
        }
        regions.push_back({d.qpart_off, d.qpart_off + (int64_t)d.n_q_tiles * d.m * plan.rank});
        if (d.st_slots > 0) regions.push_back({d.st_part_off, d.st_part_off + d.st_slots});
        if (d.n_p_chunks > 1) regions.push_back({d.ppart_off, d.ppart_off + (int64_t)d.n_p_chunks * d.n * plan.rank});
        if (d.path == kPathMfma) {
            regions.push_back({d.scT_off, d.scT_off + ((d.m / 128) * d.n * 4 + 7) / 8});
            regions.push_back({d.scT2_off, d.scT2_off + ((d.m / 128) * d.n * 4 + 7) / 8});
            regions.push_back({d.qs_off, d.qs_off + 3 * 32 * d.m * 2 / 8});
        }
    }
    std::sort(regions.begin(), regions.end());
    for (size_t i = 0; i < regions.size(); ++i) {
        if (regions[i].first < 0 || regions[i].second > (int64_t)plan.ws_doubles) return false;
        if (i > 0 && regions[i].first < regions[i - 1].second) return false;
    }
    return true;
}

}  // namespace conef
