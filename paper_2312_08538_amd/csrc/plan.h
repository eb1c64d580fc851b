// Host-side plan of a model: per-matrix descriptors, buffer offsets and the work tables
// the grouped kernels index with blockIdx.  Plain C++, no device code.
#pragma once
#include <array>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace conef {

constexpr int kAlign = 64;          // every per-matrix offset is a multiple of 64 elements
constexpr int kMaxRank = 32;
constexpr int kGramRows = 256;      // rows per LDS piece of the Gram kernel
// Ranks up to 8: threads and rows per workgroup of the second orthonormalisation launch, and rows per partial Gram matrix (64
// are one trip of a workgroup).  Every workgroup of the second launch adds the partial ones up for itself, one or two
// rounds of eight loads per thread: at most 128 of them; a very tall matrix has up to four times as many, and 512 workgroups
// (1000000 x 16, rank 8: 76 us for the stage with a workgroup per 256 rows, 53 so).
constexpr int64_t kTallRows = 131072;
constexpr int orth_threads(int rank) { return rank <= 4 ? 256 : 512; }
constexpr int64_t gram_rows_small(int64_t n)
{
    const int64_t most = n > kTallRows ? 512 : 128;
    return ((n + most - 1) / most + 63) / 64 * 64;
}
constexpr int64_t apply_rows(int rank, int64_t n)
{
    const int64_t t = orth_threads(rank);
    return n > kTallRows ? ((n + 511) / 512 + t - 1) / t * t : t;
}
// Ranks up to 8: models of matrices of few rows are orthonormalised in one launch, a workgroup per matrix (k_orth_rows), which saves
// the time of a launch where a workgroup has little to add up.  us a step, two launches / one: rank 4 64 x 500 20.6 / 19.6, 600 x
// 2048 (4 chunks of P) 34.2 / 33.5, 1000 x 500 24.7 / 24.5, 600 x 8192 (16 chunks) 41.0 / 42.8, 500 of 1000 x 260 345 / 341; rank 8 256 x 2048
// 41.1 / 40.0, 600 x 500 30.2 / 30.6, 1000 x 500 30.4 / 34.6, 100 and 300 of 64 x 260 27.8 / 26.2 and 43.4 / 45.3.
constexpr int kOrthRows = 1024;
constexpr int64_t orth_most_rows(int rank) { return rank <= 4 ? kOrthRows : 256; }
constexpr int kQredManyTiles = 32;  // partial sums of Q+ per entry from which 16 threads share an entry's sum
constexpr int kStripRows = 32;      // rows per workgroup item of the strip P pass
constexpr int64_t kStripSpan = (int64_t)1 << 29;    // elements a strip workgroup's rows may span (32-bit byte offsets)
// Strip family, quantiser, blocks of whole octets.  P pass: on octets unless 32 rows span more than kStripSpan elements (the
// matrix then takes the kernels that load element by element, and only that matrix).
constexpr int64_t kRaggedMaxCols = kStripSpan / kStripRows;
// Q+ pass: also only where a matrix gives the kernel enough to do.  A wave takes 32 rows at a time, so that a matrix of few rows
// leaves waves idle, which costs where the workgroups fill the chip, and a workgroup sets up more; element by element, a row tile
// is 32 rows and not 128, and a matrix of more rows needs the launch that adds partial sums.  `total`: elements of the model's strip
// matrices.  us for a step of one matrix with fp32 gradients, element by element / on octets:
//   ranks to 4    32 x 5000 at rank 1 23.9 / 24.8, 16 x 100001 40 / 45, 256 x 1300 25.6 / 27.2, 600 x 650 24.0 / 25.3; 64 x 5000 needs no
//                 launch for partial sums on octets (the pass 6.5 / 4.8), 10000 x 33 and 600 x 5000 have fewer of them (8.5 / 7.8, 10.6 / 9.3)
//   8             the same for up to 32 rows (16 x 100001 49 / 55), from there on octets are as good or better
//   16            600 x 300 44.1 / 44.9, 64 x 300 38.7 / 37.0, 38 of 64 x 2500 84 / 92, eight 82 / 82, 10000 x 65 51.2 / 48.8
//   32            64 x 300 57.2 / 57.6, 42 of 40 x 300 66.9 / 63.7, 38 of 64 x 2500 125 / 165, 128 x 300 57.5 / 58.9, 19 of 128 x 2500
//                 134 / 129, 128 x 100001 195 / 222, 600 x 300 61.6 / 64.5, 600 x 1300 70 / 73
//   between       element by element the padding of the rank is multiplied too: the pass at rank 24 600 x 300 18.4 / 15.9, 32 x 20001
//                 18.5 / 24.2, at 12 16.5 / 11.4
constexpr bool ragged_q_pays(int rank, int64_t n, int64_t total)
{
    constexpr int64_t M = 1000000;
    if (n <= 32) return rank > 8 && rank != 16 && rank != 32 && (rank < 16 || total < M / 2);
    if (rank <= 4) return n <= 128 || n > 2048 || total >= M;
    if (rank == 16) return n <= 64 ? total < 2 * M : n <= 128 || n > 4096 || total >= M;
    if (rank == 32) return n <= 128 ? total > M / 4 && total < (n <= 64 ? 1 : 8) * M : n > 4096 || total >= M;
    return true;
}
// Strip err pass of matrices whose Q+ fits into LDS (kernels_walk.hip): ranks up to 8, eight columns or more, 48 KB, three
// workgroups per CU.  us a step, bf16 and fp32, the err pass on strips / with Q+ in LDS: rank 4 250 x 3300 (60 KB) 28.8 / 28.2, 250 x 4500
// (81 KB) 31.4 / 34.9, 1000 x 6001 50.9 / 73; rank 8 1000 x 1300 (48 KB) 35.7 / 32.6, 1000 x 1700 37.2 / 37.9; rank 2 250 x 5001 (50 KB)
// 30.7 / 30.4, 250 x 8001 32.4 / 38.3.
constexpr int kWalkLds = 12288;     // floats
constexpr int walk_rank(int rank) { return rank <= 2 ? rank : rank <= 4 ? 4 : 8; }
constexpr int64_t walk_lds(int64_t m, int rank) { return (m + 8) * walk_rank(rank) + (m + 15) / 8 * 4; }
constexpr int kFlatRows = 8;        // matrices of at most so many rows: a wave of the strip Q+ pass takes all of them
// The step in one launch, a workgroup per matrix (kernels_small.hip): matrices whose p = g + e and factors fit into the LDS of a
// CU, rows of whole octets, blocks of 8 * 2^j elements, ranks up to 8, no matrix of the packed-split family (whose stages add up in
// fp32; fp64 sums in another order are the stages' but for a last bit of an fp32 entry now and then).  Up to 256 matrices, a CU each; more, which take turns, only if they are worth
// a CU.  us a step, in one launch / in the stages' six: 8 x 8 at rank 4, bf16 7.9 / 19.6, at rank 8 10.3 / 19.6, 300 of them 15.3 /
// 19.6 and 20.1 / 19.6, 1000 29 / 19 and 39 / 25; 64 x 64 at rank 8 11.1 / 21.1, 300 of them 22.0 / 25.8, 1000 42.6 / 47, 4000 167 / 134;
// 16 x 1024 at rank 8 17.0 / 30.1, 300 of them 38.6 / 66.6, 4000 346 / 648; 256 x 128 at rank 2 14.6 / 23.1, at rank 4, bf16 16.6 / 22.5, 256
// of them 18.6 / 45.8, 4000 272 / 401.
constexpr int64_t kSmallMaxElems = 32768, kSmallMaxRows = 1024;
constexpr bool small_pays(int64_t n_mats, int64_t total) { return n_mats <= 256 || total >= 8192 * n_mats; }
constexpr int kSmallPad = 4;        // floats between the rows of p in LDS: 16 rows of a matrix-core operand fall on distinct banks
constexpr int64_t kSmallLds = 160 * 1024 - 2048;      // (2 KB: the factorisation's own)
constexpr int64_t small_lds_bytes(int64_t n, int64_t m, int rpad)
{
    const int64_t n16 = (n + 15) / 16 * 16, m16 = (m + 15) / 16 * 16;
    return 8 * (16 * 16 + m16 + n16) * rpad + 4 * n16 * (rpad + m16 + kSmallPad);
}
constexpr int kFastMaxRank = 8;     // the octet family holds rank <= 8 in registers
constexpr int kPTileRows = 64;      // rows per workgroup item of the octet P pass

enum Path { kPathGeneric = 0, kPathOctet = 1, kPathMfma = 2 };
constexpr int kMfmaRows = 128;      // rows per workgroup item of the MFMA P pass
constexpr int kUpdRows = 64;        // tile of the decompress / update kernel
constexpr int kUpdCols = 128;
// ranks for which that kernel is the one on the fp32 matrix cores (elsewhere the vector ALU keeps up with the memory)
constexpr bool update_on_cores(int rank) { return rank > 8 && (rank & 3) == 0; }
// End of the chunk of columns that starts at c_begin (the last chunk may be short, and c_begin + chunk beyond 2^31).
constexpr int chunk_end(int64_t m, int chunk, int c_begin) { return m - c_begin > chunk ? c_begin + chunk : (int)m; }
// Strip err pass: the column whose row of Q+ belongs to virtual column c0 + v of a segment (those past the end belong to the next
// row; a segment's last strip may reach further still: the last column).  Unsigned: m + v may pass 2^31.
constexpr uint32_t virtual_column(uint32_t m, uint32_t c0, uint32_t v)
{
    const uint32_t k = c0 + v < m ? c0 + v : c0 + v - m;
    return k < m ? k : m - 1;
}
// Widest matrix of the octet kernels, whose column indices run ahead of a row's end in 32 bits; the strip kernels take wider ones.
constexpr int64_t kOctetMaxCols = ((int64_t)1 << 31) - 4096;
constexpr int kErrRows = 128;       // rows per workgroup item of the MFMA err pass (8 waves x 16)
constexpr int kErrRun = 16;         // column blocks of 128 per item of the MFMA err pass (at most 16)
constexpr int kCsCols = 256;        // columns per workgroup item of the count-sketch update pass

// One matrix of the model as the kernels see it (device copy is an array of these).
// Workspace offsets are in doubles from the start of the workspace.
struct MatDesc {
    int64_t n, m, N;                // rows, cols, n*m
    int64_t grad_off, word_off, scale_off, p_off, q_off;   // element offsets in the flat buffers
    int64_t nblk;                   // number of scale blocks
    int64_t gram_off;               // partial Gram matrices, [n_gram_tiles][r*r]
    int64_t gsum_off;               // r*r Gram matrix (the partial ones added up in a fixed order), ranks above 8
    int64_t rinv_off;               // r*r inverse triangular factor, ranks above 8
    int64_t qpart_off;              // partial sums of Q+, [n_q_tiles][m*r]
    int64_t ppart_off;              // partial sums of P, [n_p_chunks][n*r] (only if n_p_chunks > 1)
    int32_t n_gram_tiles, n_q_tiles, n_p_chunks;
    int32_t gram_tile_rows;         // rows per partial Gram matrix (a multiple of kGramRows, or of 64 up to rank 8)
    int32_t q_tile_rows;            // rows per partial of Q+
    int32_t p_chunk_cols;           // columns per partial of P
    int32_t path;                   // kernel family chosen for this matrix
    // strip err pass: a run of es_tile elements of the flat index per item, or (es_seg > 0) rows of a column segment of es_seg
    // columns, es_over columns past it that the segment's last blocks may reach, es_pitch floats of LDS per row;
    // es_rows: rows of a narrow matrix that a wave takes as one (64 / columns), else 1
    int32_t es_tile, es_seg, es_over, es_pitch, es_rows;
    int32_t es_walk;                // 1: the err pass walks octets with Q+ in LDS (err_w_items), the others are not set
    // octet family: a lane owns 8 consecutive elements of a row; lr lanes share a row
    int32_t lr_shift;               // log2(lanes per row segment), 3..6
    int32_t lb_shift;               // log2(lanes per scale block) = log2(block/8)
    int32_t m8;                     // m / 8
    // MFMA family: workspace offsets in doubles; bf16 triple split of Q+ (x = hi + mid + lo)
    int64_t scT_off;                // block scales, column-block-major: [m / 128][n] fp32
    int64_t scT2_off;               // the same for the other error vector of Algorithm 3
    int64_t qs_off;                 // Q+, tile order:      [m/128][3][8][16][32]
    // count-sketch error compressor (row sketch, one table row per bucket)
    int64_t w;                      // table rows (buckets) of this matrix
    int64_t table_off;              // element offset of the w x m table in the flat table buffer
    int64_t hash_off;               // offset of the matrix's n entries in row_hash and bucket_rows
    int64_t bptr_off;               // offset of its w + 1 entries in bucket_ptr
    int32_t cs_cols;                // columns per item of the sketch update pass; column form: rows per item (1, 2, 4 or 8)
    // count sketch in its linear form (rank 32, bf16 gradients, fp16 table, columns a multiple of 128): the sketch is
    // never decoded per element; T = S Q and U = (signed bucket sums of P^) carry its share of the factors
    int32_t cs_lin;                 // 1: this matrix takes the linear form
    int32_t cs_q_tiles_g;           // row tiles of the Q+ pass over the gradient; the table's tiles follow them
    int64_t cs_t_off;               // workspace offset (doubles) of T, w x 32 fp64
    int64_t cs_u_off;               // workspace offset (doubles) of U, w x 32 fp32
    // random-block gradient compressor
    int32_t err_tile;               // octet family: the err pass runs in strips with the residual on the fp32 matrix cores
    int32_t pack;                   // octet family: the P and Q+ passes run on the bf16 matrix cores with packed factor splits
    int64_t rb_k;                   // coordinates kept per step (0: not configured)
    int64_t rb_delta_off;           // offset of the matrix's kept values in the flat Delta buffer
    // random-k gradient compressor (stratified: one coordinate kept per stratum of rk_g consecutive ones)
    uint32_t rk_g;                  // stratum length (0: not configured)
    uint32_t rk_pad;
    uint64_t rk_magic;              // floor(2^64 / rk_g) + 1: j / rk_g = mulhi64(j, rk_magic) for j < 2^32 (unused for rk_g = 1)
    int64_t rk_delta_off;           // offset of the matrix's kept values (one per stratum) in the flat Delta buffer
    // ... or a uniformly drawn subset (rk_g = 0): rk_uk coordinates kept, the keyed permutation's shape a x b
    uint32_t rk_uk, rk_ua, rk_ub, rk_upad;
    uint64_t rk_umagic;             // floor(2^64 / rk_ub) + 1
    // Algorithm 3, version 2: the first error vector is a random block of the matrix, kept as it is
    int64_t i2_k;                   // coordinates it keeps (0: none)
    int64_t i2_off;                 // offset of the matrix's kept values in the flat buffer of first error vectors
    // element-wise gradient compressors (random block, scaled sign): the matrix's items in its stream table
    int32_t st_first, st_slots;     // index of its first item; partial-sum slots (one per wave that works on it)
    int32_t st_atomic;              // its sign bits are set with atomic ORs (kernels for any shape): cleared first
    int64_t st_part_off;            // workspace offset (doubles) of its partial l1 sums
    int64_t sign_off;               // offset (words) of its sign bits in the flat sign buffer
};

// One unit of work of a grouped launch: matrix index and kernel-specific coordinates.
struct WorkItem {
    int32_t mat, a, b, c;
};

// A unit of the two orthonormalisation launches for ranks up to 8, with all that a workgroup needs of its matrix: the
// descriptor's own line is one more round trip to memory, of the five or six that such a launch consists of.
struct OrthItem {
    int64_t p_off;                  // element offset of the matrix in P
    int64_t row0, row1;             // rows of this item
    int64_t n;                      // rows of the matrix
    int64_t gram_off;               // workspace offset: first launch, of this item's partial Gram matrix; second, of the matrix's first one
    int64_t ppart_off;              // column chunks of P (first launch)
    int32_t tiles, chunks;          // partial Gram matrices of the matrix, column chunks of P
    int64_t pad;
};

struct Plan {
    int rank = 0, bits = 0, block = 0, dtype = 0, rpad = 0;
    uint64_t seed = 0;
    // count-sketch mode (the error state is a table instead of codes and scales)
    bool sketch = false;
    float beta = 0.0f;              // share of the error kept back (partial update)
    int table_dtype = 0;            // 0 fp32, 1 fp16
    size_t table_elems = 0;
    std::vector<int32_t> row_hash;      // per row: bucket, bit 31 set for sign -1
    std::vector<int32_t> bucket_ptr;    // per matrix w + 1 entries: rows of bucket b are bucket_rows[ptr[b] .. ptr[b+1])
    std::vector<std::array<int32_t, 2>> row_order;  // row sketch, n entries per matrix of reads_row_order: bucket_rows' entry, its bucket
    std::vector<int32_t> bucket_rows;   // per matrix n entries: row index (bit 31: sign -1), ascending within a bucket
    std::vector<WorkItem> cs_err_items; // sketch update: (mat, first bucket, buckets, column tile of cs_cols); column form: (mat, first row, rows, 0)
    std::vector<WorkItem> cs_err_f_items;  // the same for matrices of the octet path (wider tiles)
    // linear form: (mat, first table row, 0, 0) tiles of 128 table rows for T = S Q; (mat, pair of column blocks, table row
    // tile, 0) for S^T U; (mat, first bucket, buckets, 0) for U; (mat, strip of 128 columns, first bucket, buckets) for the update
    std::vector<WorkItem> cs_t_items, cs_qt_items, cs_u_items, cs_lin_items;
    std::vector<MatDesc> mats;
    size_t grad_elems = 0, code_words = 0, n_scales = 0, p_elems = 0, q_elems = 0;
    bool any_octet = false, any_generic = false, any_p_chunks = false, any_mfma = false;
    size_t ws_doubles = 0;
    size_t workspace_bytes = 0;
    // strip kernels (any shape)
    std::vector<WorkItem> p_items;      // pass 1: (mat, first row, column chunk, rows: kStripRows or fewer)
    std::vector<WorkItem> q_items;      // pass 2: (mat, strip of 64 columns, row tile)
    std::vector<WorkItem> p_r_items, q_r_items;     // the same of the quantiser on octets (kernels_ragged.hip)
    std::vector<WorkItem> q_flat_items; // pass 2, few rows: (mat, four strips)
    std::vector<WorkItem> err_s_items;  // pass 3: (mat, tile, its first row, rows it spans), or with segments (mat, first row, segment, rows)
    std::vector<WorkItem> err_g_items;  // pass 3, es_rows > 1: (mat, tile, its first group of rows, groups it spans)
    std::vector<WorkItem> err_w_items;  // pass 3, Q+ in LDS: (mat, first run of 512 elements, runs, its first row)
    bool q_joined = false;              // q_f_items: (mat, strip, 0), a workgroup each, whose four waves are the row tiles
    int ew_lds = 0;                     // floats of LDS of that pass
    std::vector<WorkItem> err_items;    // pass 3, blocks that are not 8 * 2^j elements (j <= 6): (mat, first block, blocks per wave)
    int es_lds = 0;                     // floats of LDS of the strip err pass
    int wshift = 0, lb_shift = 0;       // log2(code fields per word); log2(block / 8) for power-of-two blocks of 8 elements or more
    int block_shift = -1;               // log2(block), -1 if it is not a power of two
    float inv_s = 0.0f;                 // fl32(1 / s)
    uint64_t bmagic = 0;                // floor(2^64 / block) + 1 (exactly 2^64 / block for a power of two)
    // octet family (one item per wave for p and err, per workgroup for q)
    std::vector<WorkItem> p_f_items;    // (mat, first row, column chunk), one workgroup each
    std::vector<WorkItem> q_f_items;    // (mat, 64-column strip, row tile)
    std::vector<WorkItem> err_f_items;  // (mat, strip, first row, rows)
    std::vector<WorkItem> err_t_items;  // (mat, strip of 128 or 256 columns, first row, rows): matrices of the octet family whose
                                        // err pass forms the residual on the fp32 matrix cores (rank 4 or 8, block <= 256)
    // packed-split passes (matrices of the octet family with bf16 gradients, 2- or 4-bit codes, blocks and rows of 128 or more)
    std::vector<WorkItem> p_k_items;    // (mat, first row), 128 rows per workgroup; eight lists of one length, one per XCD (mat = -1: padding)
    std::vector<WorkItem> q_k_items;    // (mat, pair of column blocks of 128, row tile)
    // MFMA family (rank 32, bf16 gradients, 4-bit codes, block 128)
    std::vector<WorkItem> p_m_items;    // (mat, first row), 128 rows per workgroup; eight lists of one length, one per XCD (mat = -1: padding)
    std::vector<WorkItem> q_m_items;    // (mat, pair of column blocks of 128, row tile)
    std::vector<WorkItem> err_m_items;  // (mat, first row, first column block of 128, blocks)   128 rows per workgroup
    std::vector<WorkItem> split_p_items;   // transpose the scales: (mat, first row / 64)
    std::vector<WorkItem> split_qn_items;  // split Q+ (row-major):         (mat, first k / 64)
    // shared
    std::vector<WorkItem> pred_items;   // reduce partial P: (mat, first entry of n*r)
    std::vector<WorkItem> gram_items;   // (mat, gram tile)
    std::vector<WorkItem> apply_items;  // (mat, first row)                    64 rows per workgroup
    std::vector<OrthItem> gram_s_items, apply_s_items;      // the same for ranks up to 8
    std::vector<int32_t> orth_first;    // one launch for both: each matrix's first gram_s_items entry; empty: two launches
    std::vector<WorkItem> qred_items;   // reduce partial Q+: (mat, first entry of m*r)
    std::vector<WorkItem> elem_items;   // element-wise helpers: (mat, first element / 1024)
    std::vector<WorkItem> upd_items;    // decompress / update: (mat, row tile of 64, column tile of 128, row tiles)
    bool csc_rows_p = false;            // column form: the P pass takes whole rows (csc_p_items), not the strip kernels'
    std::vector<WorkItem> csc_p_items;  // (mat, first row, rows, rows per workgroup)
    int csc_p_lds = 0, csc_p_threads = 0;
    int csc_threads = 0;                // column form of the sketch: threads per workgroup of the update
    int64_t small_lds = 0;              // bytes of LDS of the step in one launch; 0: not for this model
    int upd_many = 0;                   // 1: the kernel that walks several row tiles takes them (else all are of one tile)
    // element-wise gradient compressors with the quantiser: stream tables (made with the plan)
    bool norm_back = false, norm_back_two = false;      // the scaled sign's norm pass goes backwards, one and two error vectors
    size_t sign_words = 0;
    size_t rb_delta_elems = 0;      // set by configure_random_block
    size_t rk_delta_elems = 0;      // set by configure_random_k / configure_random_k_uniform
    bool rk_uniform = false;        // the latter
    bool sketch_cols = false;       // count sketch in the column form: tables are rows x w, hashes and bucket lists are over columns
    size_t i2_elems = 0;            // set by configure_i2 (never 0 once configured)
    bool i2_configured = false;
    std::vector<WorkItem> rb_items;     // matrices of whole power-of-two blocks: (mat, first run of 512 elements, runs), one item per wave
    std::vector<WorkItem> rb_g_items;   // any other matrix: (mat, first block, blocks per wave), 4 waves per item
};

// Checks that the work tables of each of the three passes cover every element of every matrix exactly
// once (items inside their matrix, no item twice, covered areas adding up to rows x cols), that every
// matrix has its reduction, Gram and apply items, and that the workspace regions do not overlap.
// Returns true if so.
bool check_plan(const Plan &plan);
// row sketch: the matrix's P and Q+ passes walk its rows bucket by bucket (the octet kernels; the linear form does not)
inline bool reads_row_order(const MatDesc &d) { return d.path == kPathOctet && !d.cs_lin; }

// Returns 0 or a negative CONEF_E* code.  `rows`/`cols` have n_mats entries.
int make_plan(Plan &plan, const int64_t *rows, const int64_t *cols, int n_mats, int rank, int bits,
              int block, int dtype, uint64_t seed);

// The same for the count-sketch error compressor: sketch_rows[l] buckets (1 .. rows[l]) for matrix l,
// beta in [0, 1), table_dtype 0 (fp32) or 1 (fp16).  Also computes the hash of every row and the
// bucket lists.
// columns: the column form (sketch_rows then holds the number of buckets per matrix, at most its columns)
int make_sketch_plan(Plan &plan, const int64_t *rows, const int64_t *cols, const int64_t *sketch_rows, int n_mats,
                     int rank, float beta, int table_dtype, int dtype, uint64_t seed, bool columns = false);
constexpr int kCscMaxCols = 16384;  // column form: a row of the residual and one of the table are staged in LDS
constexpr int kCscThreads = 512;   // most threads per workgroup
constexpr int kCscLds = 20 * 1024;  // LDS floats that several rows of a workgroup may take: two workgroups per CU

// Random-block gradient compressor: keep[l] coordinates of matrix l per step (1 .. rows * cols).  Sets the
// per-matrix fields, the Delta layout and (for a quantiser plan) the work tables.  Returns 0 or a negative code.
int configure_random_block(Plan &plan, const int64_t *keep);
// Random-k, stratified: group[l] = stratum length of matrix l, 1 <= group[l] <= rows*cols < 2^32.
int configure_random_k(Plan &plan, const int64_t *group);
// Kept coordinate of stratum i of a matrix of N coordinates with strata of G (host; the kernels compute the same).
int64_t random_k_index(uint64_t seed, uint32_t mat, uint64_t step, int64_t N, int64_t G, int64_t i);

// First coordinate of the kept block of a matrix of N elements at `step` (Philox4x32-10 of (matrix, ~0, step)).
int64_t random_block_start(uint64_t seed, uint32_t mat, uint64_t step, int64_t N, int64_t k);
// random-k as a uniformly drawn subset of keep[l] coordinates; the coordinate that goes to slot i (pi^-1(i))
int configure_random_k_uniform(Plan &plan, const int64_t *keep);
int64_t random_k_uniform_index(uint64_t seed, uint32_t mat, uint64_t step, const MatDesc &d, int64_t i);
// Algorithm 3, version 2: sizes of the first error vectors (keep_e[l] in 0 .. N_l) and where each one's block starts
int configure_i2(Plan &plan, const int64_t *keep_e);
int64_t i2_block_start(uint64_t seed, uint32_t mat, uint64_t step, int64_t N, int64_t ke);

// Bucket and sign of a row (Philox4x32-10 of (row, matrix) keyed by the seed).
void sketch_hash(uint64_t seed, uint32_t mat, uint32_t row, int64_t w, int32_t *bucket, bool *negative);

}  // namespace conef
