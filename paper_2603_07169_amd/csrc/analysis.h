// Host-side analysis of the CSR row structure: statistics, length bins, row blocks,
// merge-path splits, plan.  Integer work only; O(m) plus O(P log m).
#pragma once
#include <cstdint>
#include <vector>

#include "spmv_mi355.h"

namespace spmv {

constexpr int kDefaultItemsPerChunk = 2048;
constexpr int kMaxBlockNnz = 8192;
constexpr int kMaxRowsMax = 1024;
constexpr int kMaxItemsPerChunk = 8192;

struct Analysis {
    spmv_analysis_info_t info{};
    int32_t bin_count[SPMV_NUM_BINS]{};
    int32_t bin_offset[SPMV_NUM_BINS + 1]{};
    std::vector<int32_t> bin_rows;    // [m]
    std::vector<int32_t> row_blocks;  // [nb+1]
    std::vector<int32_t> mp_row;      // [P+1]
    std::vector<int32_t> mp_nz;       // [P+1]
    // How scattered the columns are, from the count pass of the x windows (-1: not counted): the distinct
    // 16-byte x vectors of the row blocks, summed, and the entries of the blocks that were counted
    // (all but single rows longer than block_nnz).
    int64_t x_vectors_counted = -1;
    int64_t entries_counted = 0;
    // AUTO found the matrix group-aligned and takes the two-pass plan on its groups: the groups' columns (device memory,
    // nnz / 8 numbers, released once the plan is built)
    bool two_phase_on_groups = false;
    int32_t* d_group_cols = nullptr;
};

// Range-checks the parameters and fills in the defaults that do not depend on the matrix
// (block_nnz / rows_max left at 0 are resolved by analyze_rowptr from the mean row length).
// Returns SPMV_OK or SPMV_ERR_INVALID_ARG.
spmv_status_t resolve_params(const spmv_analyze_params_t* in, spmv_analyze_params_t* out);

// Row-block shape for a matrix of m rows and nnz entries when the caller gives none.
void default_tile_shape(int64_t m, int64_t nnz, int32_t* block_nnz, int32_t* rows_max);

// rowptr is a HOST array of m+1 entries.  Returns SPMV_OK, SPMV_ERR_BAD_STRUCTURE or SPMV_ERR_ALLOC.
// want_bin_rows: also build out->bin_rows (the one output only the BINNED plan's kernels read: 4 bytes a row that
// every other plan can do without until somebody reads the analysis back; bin_count / bin_offset are always filled).
spmv_status_t analyze_rowptr(int64_t m, int64_t n, int64_t nnz, const int32_t* rowptr,
                             const spmv_analyze_params_t& params, Analysis* out, bool want_bin_rows);
// The same list on its own (rowptr: HOST array of m+1 checked entries).  May throw std::bad_alloc.
void bin_rows_of(int64_t m, const int32_t* rowptr, std::vector<int32_t>* rows);

// Columns per block of the column-blocked plan (4 MiB of x), and whether the automatic plan
// takes it: only in place of ADAPTIVE / MERGE, with x beyond two blocks, at most 16 blocks and
// at least 2^22 entries.
int64_t column_block_width(spmv_dtype_t dtype);
// scattered: at least three distinct x vectors per four counted entries (x_vectors_counted < 0, nothing counted: no).
bool columns_scattered(int64_t x_vectors_counted, int64_t entries_counted);
bool column_block_sizes_ok(int64_t n, int64_t nnz, spmv_dtype_t dtype);
bool column_block_choice(int64_t n, int64_t nnz, spmv_dtype_t dtype, int32_t plan, int64_t x_vectors_counted, int64_t entries_counted);

// Merge-path splits every ipc steps: rows finished and entries taken at each split (P+1 of each).
void merge_path_splits(int64_t m, int64_t nnz, const int32_t* rowptr, int64_t ipc, std::vector<int32_t>* rows,
                       std::vector<int32_t>* entries);

// The two-pass plan.
constexpr int kTwoPhaseItems = 8192;               // merge-path steps per chunk of the reduce pass
constexpr int kTwoPhaseSnap = SPMV_TP_SNAP;         // rows of at most this many entries are never cut by a chunk
constexpr int kTwoPhasePieceGroups = 16384;        // most groups of four slots a workgroup of the multiply pass takes
constexpr int kTwoPhasePieceFloor = 2048;          // pieces are not made smaller than this to fill the device
constexpr int kTwoPhaseWaves = 2;                  // rounds of resident workgroups the multiply pass is cut for, where the matrix is large enough
constexpr int64_t kTwoPhaseMaxTiles = 1 << 24;     // most (column block, chunk) pairs
int two_phase_shift(int64_t n);                    // log2 of the columns per block
// Sizes alone: x of 256 KiB or more, 3 * 2^21 entries or more, tiles few and dense enough.
bool two_phase_sizes_ok(int64_t m, int64_t n, int64_t nnz, spmv_dtype_t dtype);
// The whole rule: the sizes, a row-wise plan to replace, and scattered columns (at least three distinct x vectors
// per four counted entries; x_vectors_counted < 0, nothing counted, says no).
bool two_phase_choice(int64_t m, int64_t n, int64_t nnz, spmv_dtype_t dtype, int32_t plan, int64_t x_vectors_counted,
                      int64_t entries_counted);
// Whether x is gathered in column order (spmv_gather_kernel) by k chunks to a compute unit, where AUTO has arrived at a row-wise plan.
// us, tile kernel / in column order:
//   - ADAPTIVE, FP32, call by call and out of a graph: rows of 8, 393 k entries 4.1 / 4.8 and 3.9 / 4.9, 480 k 4.75 / 4.75 and 4.7 / 4.8, 640 k 5.3 / 5.5 and
//     5.5 / 5.6, 800 k 6.0 / 5.9 and 6.1 / 6.1; of 9, 400 k 4.45 / 4.2 and 4.3 / 4.3, 600 k 5.2 / 4.7; of 16, 400 k 4.15 / 4.15 and 4.0 / 4.3, 460 k 4.35 / 4.3 and 4.25 / 4.45,
//     600 k 4.9 / 4.7 and 4.9 / 4.9, 780 k 5.5 / 5.2, 1.6 M 10.7 / 7.9, 3.2 M 19.5 / 14.5; of 24, 400 k 4.05 / 4.05 and 4.0 / 4.1, 600 k 4.65 / 4.35; of 40, 460 k 4.05 / 3.95 and 4.1 / 4.05;
//     of 5, 500 k 4.7 / 4.75, 600 k 5.25 / 5.0, 20 000 columns 4.3 / 4.0 and 4.6 / 4.0.  From 131 072 rows on the tile kernel takes more than eight tiles to a compute unit: 131 000 of 4
//     5.05 / 5.4, 131 200 of 4 5.3 / 4.9, 140 000 of 3 5.6 / 4.8, of 5 6.9 / 5.6, 250 000 of 2 6.4 / 5.6.  An x of 2048 or 4000 columns: 480 k 3.9 / 3.95 and 3.75 / 4.0, 600 k rows of 16
//     4.6 / 4.2 and 4.5 / 4.3, 655 k 4.2 / 4.2 and 4.0 / 4.2.  bf16: rows of 8, 320 k 4.3 / 4.3, 393 k 4.15 / 4.05 and 3.9 / 4.0, 480 k 4.6 / 3.95; of 16, 320 k 4.0 / 4.3, 416 k 4.05 / 3.85
//     and 3.9 / 3.7, 800 k 5.1 / 4.05, 1.6 M 9.0 / 5.4, 3.2 M 16.9 / 8.8; 2048 columns, 480 k 3.95 / 3.75 and 3.9 / 3.75, 655 k 4.15 / 3.9 and 4.0 / 3.9.
//     Rows are not cut there, so the longest may take half a chunk.  Long rows in bf16 whose x a unit's own cache holds (12 000 columns): 3000 rows of 1000 7.5 / 7.9,
//     of 1500 9.5 / 10.5, 2000 of 2400 10.6 / 11.1, 5000 of 1000 10.6 / 11.1; 9000 of 500 11.4 / 10.6, 12 000 of 300 9.75 / 8.65; 3000 of 1000 in 50 000 columns 9.9 / 8.0.
//   - MERGE, power-law rows: 92 k entries 8.6 / 5.7 and 8.4 / 5.5, 626 k 10.6 / 7.4 and 10.1 / 6.8, 2.6 M 20.2 / 16.6 and 18.6 / 13.3; 20 000 rows
//     of 3 and one of 1500, 61 k entries, 4.8 / 5.7 and 4.5 / 5.2.  A row that many small chunks cut is put together by one lane of the last:
//     3 rows of 40 000 in chunks of 512 8.4 / 14.0; 5 of 16 000 7.1 / 7.8; 13 000 rows of 5 and one of 16 000 6.3 / 7.3, one of 9000 6.0 / 6.3, one of 4000 6.6 / 5.1; 25 600 and
//     one of 16 000 (chunks of 660 steps) 6.6 / 7.2, 50 000 of 3 and one of 16 000 (840) 7.35 / 6.7; 300 000 rows of 5 and one of 200 000, 26 chunks, 21.8 / 13.2.
//     Where the pieces are so many that they go to cut_rows_kernel: 900 rows of 9000 21.7 / 23.3, scattered 23.6 / 26.1; bf16, 1200 of 9000 23.4 / 24.9, 600 of 16 000
//     24.4 / 25.5; rows over several chunks, 60 of 100 000 22.8 / 20.5, bf16, 120 of 100 000 29.9 / 25.1 (gather_leaves_pieces).
bool gather_choice(int64_t m, int64_t n, int64_t nnz, int32_t plan, bool bf16, int64_t max_len, int32_t cus, int k);
// Whether that stays so once the lines of x are known (kGatherFound).  A compute unit takes a line from the L2s in about 1 ns.  The tile kernel asks for
// about the lines that stretches of 1024 entries touch; a unit with a chunk of the gathered product for those that its chunk touches, and all
// wait for the chunk with the most.  So lines are saved where neighbouring rows share few, and lost where they share most (a stencil, a narrow
// band) and a few long or scattered rows fall into one chunk.  Over 229 matrices of 0.15 to 9 M entries what the gathered product gains goes with the lines
// saved to a compute unit, 0.7 to 0.8 ns each; the plan on cut rows gains 2 us by itself, the other one loses 0.2 us (FP32) or 0.6 us (bf16) for 1000 rows.
// us, tile kernel / in column order, lines saved:
//   - MERGE, one row of 9000 in a 27-point stencil: 64 000 rows 7.9 / 7.4, -1030, 125 000 9.4 / 10.5, -3300, 216 000 bf16 10.9 / 13.2, -2900; 640 000 rows of 5
//     and one of 9000 11.8 / 17.3, -7000; a band of 150 000 x 16 and a row of 2500 in every 5000 12.3 / 10.2, -1450, of 300 000, bf16, 15.1 / 14.0, -1220;
//     of 100 000 x 40 and one row, bf16, 9.5 / 10.2, -1290.
//   - ADAPTIVE, 2-D grid with 64 scattered rows: 360 000 rows 6.3 / 7.2, -2150, 640 000 8.6 / 13.1, -2180; with a row of 300 in every 300: 360 000 8.6 / 10.0, 40,
//     bf16 7.0 / 8.8, 80, 640 000 bf16 11.2 / 13.2, 180; bands of 300 000 x 5, FP32, 4000 wide 5.8 / 5.7, 580, bf16, 10 000 wide 5.2 / 5.6, 720, 40 000 wide
//     6.4 / 5.7, 2150; 490 000 rows of 5 in no order 13.3 / 12.3, 790, bf16 12.7 / 11.6, 1400.
//   - Short calls are bound by other things: 200 000 rows of 5 and 64 scattered 5.6 / 5.1, -2040, a 27-point stencil of 64 000 and 64 scattered rows 8.0 / 6.6,
//     -1370, bf16 7.1 / 5.7; 200 000 rows of 5 and a row of 300 in every 300 (4700 entries and 790 rows to a unit) 6.0 / 6.1.
// Given up for it: 640 000 rows of 5 and a row of 300 in every 300, FP32, 13.7 us instead of 14.3; 100 000 x 40 with a row of 2500 in every 5000, bf16, 9.7 instead of 10.1.
bool gather_pays(int64_t m, int64_t nnz, int32_t plan, bool bf16, int32_t cus, int64_t chunks, int64_t most_lines, int64_t lines, int64_t stretch_lines);
constexpr int64_t kGatherAlways = 7680;  // entries and four times rows to a compute unit up to which the lines are not looked at
// Whether the groups of eight of a WINDOWED matrix of m rows and `groups` groups are gathered by cus compute units.  Windows / gathered, us: rows of one group,
// 600 000 6.7 to 8.6 / 6.2 to 9.0, 1.5 M 12.5 / 13.5, 16.0 / 18.9 (scattered); of two, 600 000 9.2 / 8.0, 12.9 / 11.7, 1.5 M 17.2 / 18.1, 24.4 / 24.5, 21.5 / 18.7; of three,
// 600 000 12.8 / 11.8, 17.9 / 18.3; of four, 400 000 19.4 / 9.3, 20.7 / 13.5.
bool gather_groups_choice(int64_t m, int64_t groups, int32_t cus);
inline bool gather_leaves_pieces(int64_t m, int64_t chunks) { return 8 * m <= chunks; }
constexpr int64_t kGatherSmallX = 32 * 1024;  // bytes of x that a compute unit's own cache holds
constexpr int64_t kGatherMinItems = 512;  // fewest steps of a chunk: a wavefront's worth or two of every load
// Rows of at most this many entries are not cut by chunks of `items` steps.  A cut costs a chunk 1 to 2 us that show where it is short, a row
// kept whole makes its chunk the longest.  512 / 2048 entries, power-law rows, FP32: 20 000 rows (chunks of 700 steps) 5.85 / 5.11 us, 50 000 6.74 / 6.30,
// 100 000 (3500 steps) 7.89 / 8.22, 333 333 (11 700) 16.8 / 16.7 and, with other rows, 16.9 / 18.0.  A chunk of fewer steps may be left empty by it.
constexpr int64_t kGatherSnap = 2048;
int64_t gather_snap(int32_t plan, int64_t max_len, int64_t items);
// Whether every row is a whole number of groups of eight entries, as a plan that is laid out over the groups needs it.  Grouped window positions
// do not say so: they ask it of the row blocks only, and of the entries of a group only that their positions follow one another.
bool rows_of_groups(int64_t m, const int32_t* rowptr);
// The pieces of the multiply pass from where the column blocks start in the multiply order (block_first[C+1], in slots,
// the last entry = all slots): every block's groups cut evenly into the fewest pieces of at most piece_groups.
// The two-pass plan on groups of eight entries (a group-aligned matrix: every row starts at a multiple of eight entries and
// every group of eight is an aligned run of eight consecutive columns).  The matrix of groups has m rows, ceil(n / 8)
// columns and nnz / 8 entries; its column blocks hold 2^two_phase_group_shift columns (64 KB of x either way).
constexpr int kTpGroup = 8;
int two_phase_group_shift(spmv_dtype_t dtype);
// The chunks of the two-pass plan: the merge path cut every ipc steps, a cut that falls inside a row of at most snap
// entries (some of its entries taken, the row not finished) moved back to that row's first entry, the next ipc steps
// counted from there (snap < ipc).
void merge_path_splits_snapped(int64_t m, int64_t nnz, const int32_t* rowptr, int64_t ipc, int64_t snap, std::vector<int32_t>* rows,
                               std::vector<int32_t>* entries);
void two_phase_pieces(int64_t C, const int32_t* block_first, int32_t piece_groups, std::vector<int32_t>* piece_c,
                      std::vector<int32_t>* piece_g);
// AUTO's rule for the two-pass plan on groups of eight (a group-aligned matrix; plan = what the row-length rule chose):
// x of 1 MiB or more, the matrix of groups within the two-pass plan's size conditions, scattered groups (three distinct
// x vectors or more per four that the counted entries would fill).
bool grouped_two_phase_choice(int64_t m, int64_t n, int64_t nnz, spmv_dtype_t dtype, int32_t plan, bool group_aligned,
                              int64_t x_vectors_counted, int64_t entries_counted);
// The cap on a piece's groups for a device that keeps `resident` workgroups of the multiply pass at once.  A launch of a
// few more pieces than that leaves the device nearly idle while the last ones run (519 pieces on 512 places: 92 us
// instead of 71 on the 1 M-row block-clustered matrix), so the cap is the smallest one with which the column blocks make
// at most k * resident pieces, k the fewest rounds that kTwoPhasePieceGroups allows - at least `waves` rounds where
// pieces of kTwoPhasePieceFloor groups or more remain; never below kTwoPhasePieceFloor.
int32_t two_phase_piece_groups(int64_t C, const int32_t* block_first, int32_t resident, int32_t waves);

// Sums and maximises the blocks' x vector counts; true when the automatic plan should serve x
// from the windows: every block within SPMV_MAX_X_VECTORS, and the fixed-stride address lists
// (one slot per block and possible vector) no longer than a quarter of the entries.
bool window_choice(const int32_t* nv, int64_t nb, int64_t nnz, int64_t* total, int32_t* largest);

// The kernel a product of the WINDOWED plan runs from: the positions of its entries, the packed runs of its row patterns, or the blocks'
// sheets.  From the sheets where every block has one (sheet_stride > 0), vals, colidx and x allow 16-byte copies and two sets of a
// block's buffers leave a compute unit room for two workgroups at least: each product for itself, since x and beta (a y that is kept
// is held in the buffers too) are the call's.
enum class WindowKernel { positions, runs, sheets };
constexpr int64_t kStreamMaxLds = 64 * 1024;  // LDS of a workgroup that works from sheets, at most
// LDS bytes of the values, and of all that is held, of a block of at most staged_max entries and rows_max rows.
int64_t stream_val_bytes(int elem_bytes, int32_t staged_max);
int64_t stream_buf_bytes(int elem_bytes, int32_t staged_max, int32_t rows_max, int32_t x_vectors, int32_t sheet_stride, bool y_kept);
WindowKernel window_kernel(int elem_bytes, int32_t staged_max, int32_t rows_max, int32_t x_vectors, int32_t sheet_stride, bool has_runs,
                           bool vec_ok, bool y_kept);

// The row length (at most 64) whose rows hold half of the entries or more, 0 if there is none: of all rows, or, beyond kSampledRows of
// them, of as many spread over the matrix by a multiplicative hash (counting all rows' lengths took 1.2 of 9.7 ms of analysis on 4 M rows;
// rows at a fixed step would meet a grid's lines).  rowptr is a HOST array.
constexpr int64_t kSampledRows = 4096;
int32_t common_row_length(int64_t m, const int32_t* rowptr);

// Whether a windowed matrix gets sheets at all; common_len: common_row_length().  Not where the kernel that works from them was slower than the one it stands in for
// (us per product out of a graph, every row of one length, sheets / packed runs, and beside them what a neighbouring length takes).
//   - Rows that begin on the same LDS banks, read a row per lane, or half a row: FP32 64 entries 5.3 / 3.9 (1 M entries), 16.4 / 8.7
//     (6 M), 50.1 / 22.6 (24 M; 62 entries 19.7 / 20.0); 48 entries 4.2 / 3.9, 8.2 / 7.7, 20.8 / 20.7 (52: 3.7 / 3.9, 6.8 / 7.3); 32
//     entries in small blocks 4.8 / 3.9 (28: 3.3 / 4.0), while blocks of 128 of them break even, 10.5 / 10.5 and 30.7 / 31.6; bf16 64
//     entries in small blocks 4.5 / 3.7 (62: 3.9 / 4.0), in blocks of 64 6.7 / 7.0; 16 entries in blocks of 256 5.6 / 4.7, 15.0 / 12.3 (20:
//     12.0 / 16.9), in blocks of 64 3.4 / 3.7.  Scattered columns in rows of 64, which have sheets of sixteen lists: FP32 5.1 / 3.7,
//     bf16 5.3 / 3.7 from the positions; of 61: 4.1 / 4.4, 3.9 / 4.1.
//   - Rows of 32 entries or more in so few blocks that a compute unit gets one (bf16: two), where a lane's walk along a row is what the
//     product waits for: 250 k entries FP32 40 / 48 / 56 / 62 entries 2.9 / 3.1 / 3.0 / 3.1 against 2.8 / 2.9 / 2.6 / 2.8, bf16 36 / 40 / 56 / 62
//     3.0 / 3.2 / 3.3 / 3.6 against 2.6 / 2.8 / 2.8 / 3.1; 500 k entries FP32 3.4 / 3.7 / 3.6 / 3.8 against 3.5 / 3.5 / 3.6 / 3.7, bf16 3.4 / 3.5 / 3.8 /
//     4.1 against 3.3 / 3.3 / 3.5 / 3.4; 1 M entries FP32 3.9 / - / 4.0 / 4.0 against 4.1 / - / 4.2 / 4.5, bf16 3.6 / 3.6 / 3.9 / 4.0 against 4.0 / 3.9 / 3.9 / 4.3.
bool sheets_pay(int elem_bytes, int64_t m, int64_t nnz, int64_t nb, int32_t block_nnz, int32_t rows_max, int32_t common_len, int32_t cus);
// Lanes of the sheets' kernel that share a row (1 or 2); places: workgroups that a compute unit holds by their LDS.  Two where that is
// ten wavefronts or fewer and rows have 16 entries or more (27 points FP32 46.8 -> 45.3 us, 49 points bf16 32.0 -> 26.0; elsewhere two cost:
// 27 points bf16 25.8 -> 27.1, 5 points 10.6 -> 15.4), and for FP32 rows of 24 entries in large blocks, which meet on the banks whole but
// not halved (3 M / 12 M entries 4.9 -> 4.3 / 12.6 -> 11.5 us).
int stream_lanes(int elem_bytes, int64_t m, int64_t nnz, int32_t rows_max, int places, int32_t common_len);

// The chunks as the merge-path kernels take them: pairs (mp_row[p], mp_nz[p]) with every split that falls inside a row of at most
// `snap` entries moved back to the row's first entry.  May throw std::bad_alloc.
void merge_chunk_desc(int64_t m, const int32_t* rowptr, const std::vector<int32_t>& mp_row, const std::vector<int32_t>& mp_nz,
                      int64_t snap, std::vector<int32_t>* desc);
// Per split of the two-pass plan: the first and the last chunk of the row it cuts, or -1, -1.  rowptr as the splits were made
// with.  May throw std::bad_alloc.
void cut_ranges(int64_t m, const int32_t* rowptr, const std::vector<int32_t>& rows, const std::vector<int32_t>& entries,
                std::vector<int32_t>* ranges);

// Row order of the sparse-times-dense kernel: inside every window of SPMV_SPMM_WINDOW consecutive
// rows, the row ids by decreasing min(ceil(len / 4), 64), rows of equal key ascending.  rowptr is
// a HOST array of m+1 checked entries.  May throw std::bad_alloc.
constexpr int kSpmmMaxKey = 64;
void spmm_row_order(int64_t m, const int32_t* rowptr, std::vector<int32_t>* rows);

// Packed layout of the sparse-times-dense kernel.  Group g holds the rows at positions 16g .. 16g+15
// of `rows` and is stored as ceil(longest row / 16) blocks of 16 rows x 16 entries.
// desc[2g] = blocks of the groups before g, desc[2g+1] = ceil(longest row of g / 4); one closing
// pair (all blocks, 0).  Returns whether the packed copy is to be built: at most twice as many
// slots (256 per block) as the matrix has entries, and at most kSpmmMaxBlocks blocks.  May throw
// std::bad_alloc.
constexpr int64_t kSpmmMaxBlocks = int64_t{1} << 22;
bool spmm_packed_layout(int64_t m, int64_t nnz, const int32_t* rowptr, const int32_t* rows, std::vector<int32_t>* desc,
                        int64_t* num_blocks);

// Layout of the pairs form of the sparse-times-dense product: rows by decreasing length inside every window of
// SPMV_SPMM_WINDOW consecutive rows (lengths from kSpmmPairMaxKey on count as equal; ties ascending), groups of 32
// positions stored as max(1, ceil(longest row / 4)) blocks of 32 rows x 4 entries.  desc[2g] = blocks of the groups before
// g, desc[2g+1] = max(1, ceil(longest row / 2)); one closing pair (all blocks, 1).  Returns whether the form is to be kept
// next to the packed copy described by packed_desc: it takes more rows to a group, so where lengths differ inside the groups
// it pads more.  Beyond 1.25 times the packed copy's slots (matrices of a few dozen rows, or with a few rows 30 times as long
// as the others) it would be picked only for C that is not 16-byte aligned (40 rows x 333 columns 11.7 -> 9.9 us, 200 rows
// 22.1 -> 13.4), for 90 us more of analysis.  May throw std::bad_alloc.
constexpr int kSpmmPairMaxKey = 1023;
bool spmm_pair_layout(int64_t m, const int32_t* rowptr, const std::vector<int32_t>& packed_desc, std::vector<int32_t>* rows,
                      std::vector<int32_t>* desc, int64_t* num_blocks);

// What the choice between the packed copy and the pairs form knows of either's groups: a workgroup deals its groups to its
// 16 wavefronts in turn, and the rows lie in decreasing length inside windows of SPMV_SPMM_WINDOW rows, so with the rows in S
// parts a wavefront keeps meeting the same places of the windows.  place[e]: the steps of a group, averaged over the groups
// a wavefront meets at its worst place when gcd(S, groups per window / 16) = 2^e.
struct GroupSteps {
    int64_t groups = 0;
    double steps = 0;    // of all groups; a group without entries takes one
    double longest = 0;  // of any group
    double place[5] = {0, 0, 0, 0, 0};
};
// desc: pairs (first block, steps) of the groups, and a closing pair; rows_per_group: 16 or 32.
GroupSteps spmm_group_steps(const std::vector<int32_t>& desc, int rows_per_group);
// About the steps of the wavefront that has most of them, with the groups in S parts.
double spmm_busiest(const GroupSteps& g, int64_t S);
// Into how many parts the rows are cut, per slice of 16 columns: the packed copy's and the pairs form's kernels.
int spmm_packed_splits(int64_t slices, int64_t groups);
int spmm_pair_splits(int64_t slices, int64_t groups, int64_t blocks);
// Whether a product with K columns of C runs from the pairs form, where a handle has both.  vec_ok: B's and C's addresses
// and leading dimensions allow 16-byte accesses.
bool spmm_pairs_choice(const GroupSteps& packed, const GroupSteps& pairs, int64_t pair_blocks, int64_t m, int64_t K, bool vec_ok);

}  // namespace spmv
