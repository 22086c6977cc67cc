// Launch interface between the C ABI (host) and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime_api.h>

#include <cstdint>

#include "analysis.h"

namespace spmv {

struct MatrixView {
    int32_t m, n, nnz;
    const int32_t* rowptr;  // device [m+1]
    const int32_t* colidx;  // device [nnz]
    const void* vals;       // device [nnz] float or bf16 bits
    bool bf16;
    bool vec_ok;            // colidx and vals are 16-byte aligned: 128-bit loads allowed
};

constexpr int kMaxColBlocks = 16;  // most column blocks of the column-blocked plan
constexpr int kCbTile = 2048;      // entries a wavefront regroups at a time
constexpr int kMaxXVectors = 1024;     // most 16-byte x vectors a row block may keep in LDS
constexpr int kMaxTileEntries = 8192;  // most entries of a row block
constexpr int kMaxRowsPerBlock = 1024; // most rows of a row block
constexpr int kMaxPatternRuns = 4;     // most runs of rows in a patterned block
constexpr int kMaxPatternLen = 64;     // longest row of a patterned block

// x windows of the row blocks (device arrays owned by the handle).
struct XWindows {
    const int32_t* xv_ptr;    // [nb+1]
    const int32_t* xv_start;  // [xv_ptr[nb]]
    const int32_t* xv_pad;    // [nb * max_vectors] xv_start at a fixed stride per block, -1 padded: what the kernel reads
    const uint16_t* lidx8;    // [nnz / 8] lidx[8g] where the positions are grouped (see launch_lidx_groups), else null
    const uint16_t* lidx;     // [nnz rounded up to a multiple of 8]
    int32_t max_vectors;      // largest xv_ptr[b+1] - xv_ptr[b]
    const int32_t* run_desc;  // [8 * nb] packed runs of the row patterns (see launch_pattern_build), or null: no patterns
    const uint16_t* pat_pad;  // [nb * pt_cap] the blocks' pattern lists
    int32_t pt_cap;           // a multiple of 8, at most kMaxPatternRuns * kMaxPatternLen
    const unsigned char* sheets;  // [nb * sheet_stride] (see SheetRun), or null: some block has none
    int32_t sheet_stride;
    int32_t cus;              // compute units of the device (with sheets)
    int32_t common_len;       // common_row_length() (with sheets)
};

// What the stream kernel needs to know of a row block besides its values and its x vectors, in one piece (a "sheet"): a byte per
// row with the number of its run (sheet_map_bytes of them), the runs, and their lists: 16-bit byte offsets from the x value of a row's
// first entry, every list from a multiple of four bytes on, runs with equal lists sharing one.  Runs as in run_desc, up to
// kMaxSheetRuns of them.  For row i of the block:
constexpr int kMaxSheetRuns = 16;  // a line of a grid is three runs: all blocks of 128 rows in grids of lines of 32 points and more
struct SheetRun {
    int32_t value;        // value + i * len: its first entry's place among the block's values, counted from a 16-byte boundary of vals
    int32_t pos;          // pos + i * (stride_list >> 16): byte position of its first entry's x value in the window
    int32_t len;          // its entries
    int32_t stride_list;  // the step in bytes (high half, signed), and where its list starts in the sheet (low half)
};
inline int32_t sheet_map_bytes(int32_t rows_max) { return (rows_max + 15) & ~15; }

struct Scalars {
    float alpha, beta;
};

// Records a failing HIP call for spmv_last_hip_error() and clears the runtime's sticky error; true when e is an error.
bool note_hip_error(hipError_t e);

// rows == nullptr: rows 0..count-1; otherwise the `count` row ids listed in rows[].
hipError_t launch_scalar(const MatrixView& A, const int32_t* rows, int32_t count, const void* x, float* y, Scalars s,
                         hipStream_t st);
// lanes: power of two in [2, 64].
hipError_t launch_vector(const MatrixView& A, int lanes, const int32_t* rows, int32_t count, const void* x, float* y,
                         Scalars s, hipStream_t st);
// block_desc: device [2*(nb+1)], pairs (row_blocks[b], rowptr[row_blocks[b]]).
// block_nnz, rows_max: the limits the partition was built with.
hipError_t launch_adaptive(const MatrixView& A, const int32_t* block_desc, int32_t nb,
                           int32_t block_nnz, int32_t rows_max, const void* x, float* y, Scalars s, hipStream_t st);
// The adaptive plan with x served from per-block windows in LDS.  staged_max: the most entries
// of any block that is staged (i.e. not a single over-long row); <= block_nnz.
hipError_t launch_windowed(const MatrixView& A, const int32_t* block_desc, int32_t nb,
                           int32_t block_nnz, int32_t staged_max, int32_t rows_max, const XWindows& w, const void* x,
                           float* y, Scalars s, hipStream_t st);
// The kernel that launch_windowed launches for these arguments.
WindowKernel windowed_kernel(const MatrixView& A, int32_t staged_max, int32_t rows_max, const XWindows& w, const void* x, float beta);
// Analysis-time construction of the x windows.  fill == false: nv[b] = distinct x vectors of
// block b.  fill == true: writes xv_start, xv_pad (stride x_cap >= every nv[b]) and lidx given
// xv_ptr = exclusive prefix sums of nv.
hipError_t launch_window_build(const MatrixView& A, const int32_t* block_nz, int32_t nb, int32_t block_nnz, bool fill,
                               int32_t* nv, const int32_t* xv_ptr, int32_t* xv_start, int32_t* xv_pad, int32_t x_cap,
                               uint16_t* lidx, hipStream_t st);
// Merge-path cuts that fall inside a row of at most this many entries are moved back to the row's first entry, so that only
// longer rows leave parts to be put together (finish_cut): no chunk then grows by more than these entries, and none becomes
// empty, since a row that starts with a chunk and is shorter than it ends inside it.
constexpr int32_t kMergeSnap = 256;  // chunks of 512 steps, 4.8 M entries in rows of 16, 32: without it 71 and 145 us, with it 27 and 51
inline __host__ __device__ int32_t merge_snap(int32_t items_per_chunk) { return items_per_chunk > kMergeSnap ? kMergeSnap : items_per_chunk - 1; }
// Scratch for the rows that chunks cut, device [chunks] each: carry_val, and either arrivals (zero before the first run, see
// finish_cut) or carry_row (the pieces are added by a kernel of its own), the other null.
struct CutScratch {
    unsigned* arrivals;
    int32_t* carry_row;
    float* carry_val;
};
// Whether the pieces of `cuts` chunks that begin inside a row are left to a kernel of their own.  That kernel costs 1 to 3 us whatever
// it finds, finish_cut some 12 us in every chunk that takes part, during which its place stays taken: nothing while all
// chunks run at once, more the more rounds there are.  Both, us (FP32, rows of 300 or 16 entries, left without and right with the
// kernel): 1.5 M entries, 290 cuts 14.1 / 14.8, 730 cuts 15.5 / 14.4; 6 M entries, 590 cuts 36.0 / 37.4, 1170 cuts 39.6 / 37.6, 2930
// cuts 55.2 / 37.2; 24 M entries, 1170 cuts 116.2 / 118.3, 2340 cuts 117.8 / 116.4, 11700 cuts 185 / 118; two passes, rows of 700: 24 M
// entries, 260 cuts 78.8 / 79.0, 1140 cuts 82.6 / 78.0, 2930 cuts 92 / 78.6.
inline bool use_cut_rows_kernel(int64_t cuts, int64_t chunks) { return 12 * (cuts - 600) > chunks; }
// chunk_desc: device [2*(P+1)], pairs (mp_row[p], mp_nz[p]) moved back as said above.  done: null, or an event that is recorded
// at the end of the last dispatch.
hipError_t launch_merge(const MatrixView& A, const int32_t* chunk_desc, int32_t P, int32_t items_per_chunk, const CutScratch& cut,
                        const void* x, float* y, Scalars s, hipStream_t st, hipEvent_t done);
hipError_t launch_cut_rows(const CutScratch& cut, int32_t P, float* y, float alpha, hipStream_t st, hipEvent_t done);
// C <- alpha*A*B + beta*C; A CSR, B device [n x ldb] in A's storage type, C device float[m x ldc], row-major, K columns used.
// rows: device int32[m], the order in which the rows are handed to the wavefronts (a permutation
// of 0..m-1), or NULL for the natural order.
hipError_t launch_spmm(const MatrixView& A, const int32_t* rows, const void* B, int64_t ldb, float* C, int64_t ldc,
                       int32_t K, Scalars s, hipStream_t st);
// The packed copy of A the sparse-times-dense product can run from (device pointers).
constexpr int kSpmmCol16MaxN = 32768;  // up to this many columns the packed column numbers take 16 bits
struct PackedRows {
    const int32_t* rows;  // [m] row order
    const int32_t* desc;  // [2 * (num_groups + 1)] pairs (first block, steps of 4 entries)
    const void* pcol;     // [(blocks + 1) * 256] uint16 (col16) or int32
    const float* pval;    // [(blocks + 1) * 256]
    int32_t num_groups;
    bool col16;
};
// Fills pcol / pval of all blocks of all groups from the CSR arrays (the extra closing block is not written), and psrc, if not
// null, with every slot's place in colidx / vals, -1 in padding.
hipError_t launch_spmm_pack(const MatrixView& A, const int32_t* rows, const int32_t* desc, int32_t num_groups, bool col16,
                            void* pcol, float* pval, int32_t* psrc, hipStream_t st);
hipError_t launch_spmm_packed_values(const MatrixView& A, const int32_t* psrc, float* pval, int64_t slots, hipStream_t st);  // pval from the CSR values
hipError_t launch_spmm_packed(const MatrixView& A, const PackedRows& P, const void* B, int64_t ldb, float* C, int64_t ldc,
                              int32_t K, Scalars s, hipStream_t st);
const char* spmm_packed_kernel_name();
const char* spmm_pair_kernel_name();
// Whether 128-bit (float) or 64-bit (bf16) accesses to B and 128-bit ones to C are possible.
bool spmm_vec_ok(bool bf16, const void* B, int64_t ldb, const float* C, int64_t ldc);
// The pairs form of A, kept next to the packed copy while B's slice fits one LDS block (n <= kSpmmPairMaxN; device pointers):
// groups of 32 rows of the order rows[], blocks of 32 rows x 4 entries, two lanes per row.  Position t of the group's row i
// belongs to lane q = ((first + t / 4) * 64 + 2 i + t mod 2), element (t mod 4) / 2: ent[4 q + element] is the LDS offset of
// the entry's row of B, ent[4 q + 2 + element] its value, src[2 q + element] its place in colidx / vals, -1 in padding.
constexpr int kSpmmPairMaxN = 2048;
struct PairRows {
    const int32_t* rows;  // [m] row order: decreasing length inside windows of SPMV_SPMM_WINDOW rows
    const int32_t* desc;  // [2 * (num_groups + 1)] pairs (first block, steps of two entries: at least 1)
    uint32_t* ent;        // [(num_blocks + 1) * 256]
    int32_t* src;         // [num_blocks * 128]
    int32_t num_groups;
    int32_t longest_steps;  // most steps of any group
    int64_t num_blocks;
};
hipError_t launch_spmm_pair_pack(const MatrixView& A, const PairRows& P, hipStream_t st);    // off, src and val from the CSR arrays
hipError_t launch_spmm_pair_values(const MatrixView& A, const PairRows& P, hipStream_t st);  // val from the CSR values
hipError_t launch_spmm_pair(const MatrixView& A, const PairRows& P, const void* B, int64_t ldb, float* C, int64_t ldc, int32_t K,
                            Scalars s, hipStream_t st);
// Whole aligned groups of eight entries (groups = nnz / 8): lidx8[g] = lidx[8g]; *flag (device int32, 0 on entry) is set to 1
// if some group's eight positions are not consecutive numbers.
hipError_t launch_lidx_groups(const uint16_t* lidx, int32_t groups, uint16_t* lidx8, int32_t* flag, hipStream_t st);
// Row patterns of the window positions (analysis).  block_desc as for launch_adaptive.  fill == false: run_desc[8b..8b+7] =
// the runs of block b, packed: words 0-1 rows per run, 3-4 base of the run's first row, 5-6 stride (two's complement), 16 bits
// each in run order; word 2 entries per row, 8 bits each; word 7 the number of runs (0: the block has no pattern, all words 0);
// *max_table (device int32, 0 on entry) = longest pattern list of any block; *covered (device uint64, 0 on entry) = entries
// of the patterned blocks.  fill == true: pat_pad[b * pt_cap ..] = block b's list (rel of the first row of every run), then zeros.
hipError_t launch_pattern_build(const int32_t* block_desc, int32_t nb, const int32_t* rowptr, const uint16_t* lidx, int32_t block_nnz,
                                bool fill, int32_t* run_desc, int32_t* max_table, unsigned long long* covered, uint16_t* pat_pad,
                                int32_t pt_cap, const struct SheetPlan* sheets, hipStream_t st);
// With fill == false and sheets not null the blocks' sheets are planned as well: what launch_sheet_fill reads, and *largest (device
// int32, 0 on entry) = bytes of the largest, INT32_MAX if a block cannot have one.
struct SheetPlan {
    int32_t elem_bytes, map_bytes;
    int32_t* largest;
    int32_t* need;        // [nb]
    uint16_t* first;      // [nb * (kMaxSheetRuns + 1)] first rows of the runs, then the rows of the block
};
hipError_t launch_sheet_fill(const int32_t* block_desc, int32_t nb, const int32_t* rowptr, const uint16_t* lidx, const SheetPlan& p,
                             int32_t stride, unsigned char* sheets, hipStream_t st);
// flag: device int32, must be 0 on entry; set to 1 if any colidx is outside [0, n).
hipError_t launch_validate_columns(const MatrixView& A, int32_t* flag, hipStream_t st);

// y <- alpha*A*x + beta*y for A in COO / CSC / ELL storage (stateless; indices are not checked).
// COO and CSC first scale y by beta, then add every entry's contribution with float atomics.
hipError_t launch_coo(bool bf16, int32_t m, int32_t nnz, const int32_t* row, const int32_t* col, const void* vals,
                      const void* x, float* y, Scalars s, hipStream_t st);
hipError_t launch_csc(bool bf16, int32_t m, int32_t n, int32_t nnz, const int32_t* col_offsets, const int32_t* row,
                      const void* vals, const void* x, float* y, Scalars s, hipStream_t st);
hipError_t launch_ell(bool bf16, int32_t m, int32_t width, const int32_t* col_ids, const void* vals, const void* x,
                      float* y, Scalars s, hipStream_t st);

// Pieces of the COO product for callers that run several of them into one y.
hipError_t launch_scale_y(float* y, int32_t m, float beta, hipStream_t st);  // y <- beta*y (0 when beta == 0)
hipError_t launch_coo_accumulate(bool bf16, int32_t nnz, const int32_t* row, const int32_t* col, const void* vals,
                                 const void* x, float* y, float alpha, hipStream_t st);  // y += alpha*A*x, atomics

// Column-blocked regrouping (analysis).  Block of column c = c >> shift; C blocks.  ntiles =
// column_block_tiles(nnz).  count: tile_counts[b*ntiles + t].  scatter: tile_base = exclusive
// prefix sums of tile_counts in that order; writes row, column within block, source position
// and value of every regrouped entry.
int32_t column_block_tiles(int32_t nnz);
hipError_t launch_column_block_count(const MatrixView& A, int shift, int C, int32_t* tile_counts, hipStream_t st);
hipError_t launch_column_block_scatter(const MatrixView& A, int shift, int C, const int32_t* tile_base, int32_t* cb_row,
                                       int32_t* cb_col, int32_t* cb_src, void* cb_vals, hipStream_t st);
// cb_vals[k] = vals[cb_src[k]] for the nnz regrouped entries (the caller's values may have changed).
hipError_t launch_column_block_values(const MatrixView& A, const int32_t* cb_src, void* cb_vals, hipStream_t st);

// The row-wise product with x gathered in column order, of a MERGE or ADAPTIVE handle (device arrays owned by the handle).
constexpr size_t kGatherMaxLds = 160 * 1024 - 8192;  // LDS of a chunk; the rest is the kernel's own
constexpr int32_t kGatherMaxSlots = (1 << 15) - 8;   // a place in a chunk takes 15 bits, one more is the padding's
struct GatherTiles {
    int32_t* chunk_desc;  // [2*(num_chunks+1)] pairs (first row, first entry)
    uint32_t* words;      // [num_chunks * stride * 256] a chunk's entries by column: place in the chunk, column less the group's first
    int32_t* base;        // [num_chunks * stride] first column of each group of 256
    int32_t* cut_range;   // [2*(num_chunks+1)] (see finish_cut); null: no chunk cuts a row (ADAPTIVE)
    CutScratch cut;
    int32_t num_chunks, stride, slots;
    int32_t group;  // 1, or 8: entries, places and columns above are groups of eight (a WINDOWED handle of a group-aligned bf16 matrix)
    size_t lds;
};
constexpr int32_t kGatherGroupSlots = 4096;              // most groups of a chunk
constexpr size_t kGatherGroupLds = kGatherMaxLds / 2;    // two workgroups to a compute unit
// Fewest entries.  Windows / gathered, us call by call: 3.2 M in rows of 8 groups 6.1 / 5.5, 3.8 M of 6 6.2 / 6.4, 5.1 M of 16 7.6 / 6.5, of 4 10.0 / 8.0,
// 5.8 M of 6 and of 12 8.5 / 7.4 and 8.4 / 7.1, 8 M of 10 10.7 / 8.2.
constexpr int64_t kGatherGroupEntries = 1 << 22;
size_t gather_group_lds(int32_t groups, int32_t rows);
// LDS slots of the largest chunk (desc: HOST array), and the LDS bytes of a workgroup for them and at most `rows` rows.
int32_t gather_slots(bool bf16, const int32_t* desc, int64_t P);
size_t gather_lds(bool bf16, int32_t slots, int32_t rows);
// Analysis time: fills words and base, and found (device, zeroes before): whether they cannot express the matrix, and the 128-byte lines of x that
// the chunk with the most of them touches, that all chunks touch, and that all stretches of 1024 consecutive entries of a chunk touch (an x of more than
// 16384 lines: intervals of several lines, so that there are at most as many).
enum { kGatherBad, kGatherMostLines, kGatherLines, kGatherStretchLines, kGatherFound };
hipError_t launch_gather_build(const MatrixView& A, const GatherTiles& t, int32_t* found, hipStream_t st);
hipError_t launch_gather(const GatherTiles& t, const MatrixView& A, const void* x, float* y, Scalars s, hipStream_t st, hipEvent_t done);

// The two-pass plan (device arrays owned by the handle).
struct TwoPhase {
    int32_t shift;              // column blocks of 2^shift columns (of 2^shift groups' columns when group == 8)
    int32_t group;              // 1, or 8: a slot stands for a group of eight entries (group-aligned matrix)
    int32_t num_pieces;         // multiply pass: workgroups
    int32_t num_chunks;         // reduce pass: merge-path chunks
    size_t reduce_lds;          // two_phase_reduce_lds() of the largest chunk
    const int32_t* piece_c;     // [num_pieces]   column block of each piece
    const int32_t* piece_g;     // [num_pieces+1] first group of each piece (pieces are contiguous)
    const uint16_t* tp_col;     // [slots] column within the block; padding: 2^shift
    const void* tp_val;         // [slots] values in the handle's dtype; padding: 0
    const int32_t* tp_from;     // [slots/4] group of the multiply order that each group of the reduce order is fed by
    const uint16_t* tp_pos;     // [slots] reduce order: CSR position within the chunk; padding: 0xFFFF
    const int32_t* chunk_desc;  // [2*(num_chunks+1)] pairs (rows finished, entries taken)
    const int32_t* chunk_g;     // [num_chunks+1] first group of each chunk in the reduce order
    float* prod;                // [slots] scratch: the products between the two passes, in the multiply order
    const int32_t* cut_range;   // [2*(num_chunks+1)] per cut that falls inside a row: first and last chunk of that row (else -1)
    CutScratch cut;             // [num_chunks]
};
constexpr int kTpMaxShift = 15;  // column blocks of at most 32768 columns (16-bit columns, one more value for padding)
size_t two_phase_reduce_lds(int32_t entries, int32_t rows);
hipError_t launch_two_phase(const TwoPhase& t, const MatrixView& A, const void* x, float* y, Scalars s, hipStream_t st, hipEvent_t done);
// Analysis time.  Scratch of the regrouping (device, T = C*P tiles): all of it is temporary.
struct TwoPhaseTables {
    int32_t* padded;       // [T]    slots of tile t = c*P + p (entries rounded up to whole groups of four)
    int32_t* base1;        // [T]    slots before it in the multiply order
    int32_t* within;       // [T]    slots of its chunk in the column blocks before its own
    int32_t* in_chunk;     // [P+1]  slots of every chunk, then 0
    int32_t* chunk_first;  // [P+1]  slots before every chunk in the reduce order, then all slots
    int32_t* block_first;  // [C+1]  slots before every column block in the multiply order, then all slots
    int32_t* scan_sums;    // [two_phase_scan_blocks(T)] scratch of the prefix sums
};
int64_t two_phase_scan_blocks(int64_t count);
// Counts every chunk's entries per column block and derives every table above, and chunk_g[P+1] (first group of
// every chunk in the reduce order).  Integer arithmetic only: the result does not depend on scheduling.
hipError_t launch_two_phase_tables(const MatrixView& A, int shift, int32_t C, int32_t P, const int32_t* chunk_desc,
                                   const TwoPhaseTables& w, int32_t* chunk_g, hipStream_t st);
// Fills the padding and places every entry (CSR order kept inside a tile).
// group == 8: A is the matrix of groups (its colidx the groups' columns) and no value is placed.
hipError_t launch_two_phase_place(const MatrixView& A, int shift, int32_t C, int32_t P, const TwoPhaseTables& w,
                                  const int32_t* chunk_desc, int64_t slots, int group, uint16_t* tp_col, void* tp_val,
                                  int32_t* tp_src, int32_t* tp_from, uint16_t* tp_pos, hipStream_t st);
// tp_val[s] = vals[tp_src[s]] wherever tp_src[s] >= 0; group == 8: A is the caller's matrix, a slot holds the eight values of
// group tp_src[s].
hipError_t launch_two_phase_values(const MatrixView& A, const int32_t* tp_src, void* tp_val, int64_t slots, int group,
                                   hipStream_t st);
// gcol[g] = colidx[8g] / 8; *flag (cleared by the caller) is set when some group of eight entries is not an aligned run
// of eight consecutive columns.
hipError_t launch_two_phase_groups(const int32_t* colidx, int32_t ngroups, int32_t* gcol, int32_t* flag, hipStream_t st);

// The sliced ELL plan.  slice_ptr[ns+1]: slots before each slice of kSellHeight rows (a slice takes width * kSellHeight
// slots, stored column by column).  fill: column, source position and value of every slot (-1, -1, 0 for padding).
constexpr int kSellHeight = 64;
hipError_t launch_sell_fill(const MatrixView& A, const int32_t* slice_ptr, int32_t ns, int32_t* sell_col, int32_t* sell_src,
                            void* sell_val, hipStream_t st);
// sell_val[s] = vals[sell_src[s]] wherever sell_src[s] >= 0.
hipError_t launch_sell_values(const MatrixView& A, const int32_t* sell_src, void* sell_val, int64_t slots, hipStream_t st);
hipError_t launch_sell(const MatrixView& A, const int32_t* slice_ptr, int32_t ns, const int32_t* sell_col, const void* sell_val,
                       const void* x, float* y, Scalars s, hipStream_t st);

// Cross-lane reduction self-check on one wavefront.  in: device float[64], lane l contributes in[l].
// out: device float[14*64]; out[gi*64 + l] = sum over lane l's aligned group of G = 2^gi lanes,
// gi = 0..6 from the compile-time variant, then the same seven again from the run-time variant.
hipError_t launch_reduce_selftest(const float* in, float* out, hipStream_t st);

const char* scalar_kernel_name();
const char* vector_kernel_name();
const char* gather_kernel_name();
const char* gather_group_kernel_name();
const char* tile_kernel_name();  // kernel of the adaptive and merge plans
const char* windowed_kernel_name(WindowKernel k);
const char* spmm_kernel_name();
const char* sell_kernel_name();

}  // namespace spmv
