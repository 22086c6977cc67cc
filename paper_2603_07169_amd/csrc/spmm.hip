// gfx950 kernel for the sparse-times-dense product C <- alpha*A*B + beta*C (paper App. C task 13).
#include <hip/hip_runtime.h>

#include "analysis.h"
#include "device_common.h"
#include "kernels.h"

namespace spmv {
namespace {

constexpr int kSpmmWG = 1024;  // 16 wavefronts per workgroup (one workgroup per CU: its B slice fills the LDS)
constexpr int kSpmmKT = 16;    // columns of B and C a workgroup owns (4 lanes x float4 per row)
constexpr int kSpmmNB = 2048;  // rows of B held in LDS at a time (2048 x 16 floats = 128 KB)

// ------------------------------------------------------------------------------------------
// C <- alpha*A*B + beta*C with A in CSR (FP32), B (n x K) and C (m x K) dense, row-major
// (paper App. C task 13).  Every stored entry a_ij adds a_ij * B[j, :] to C[i, :], so the
// operation reads a K-wide row of B per entry: nnz * K * 4 bytes in all, far more than B itself
// or than C.  Those reads are kept on chip: a workgroup owns kSpmmKT = 16 columns of B and C,
// copies that slice of B (up to kSpmmNB = 2048 rows: 128 KB) into LDS once and then walks over
// all its rows of A.  Four lanes (a DPP quad) serve a row, one float4 of the slice each; a
// wavefront serves 16 rows at a time, for as long as the longest of them lasts: the rows can be
// handed out in an order that puts rows of like length side by side (built at analysis time on
// request).  The quad reads its row's entries straight from memory, 16 bytes per lane and load;
// an entry is then handed to the other three lanes with a quad broadcast that rides on the
// multiply-add, and each lane adds value * B-row piece out of LDS.  Row ids, row bounds and
// entries of the coming groups are fetched while the current one is multiplied.
// B wider than the LDS block is taken in several passes over A, accumulating into C.
struct SpmmArgs {
    const int32_t* rowptr;
    const int32_t* colidx;
    const void* vals;     // float or bf16 bit patterns (the kernel's storage type)
    const int32_t* rows;  // row order (SORTED kernels), else unused
    const void* B;        // same storage type as vals
    float* C;
    int64_t ldb, ldc;
    int32_t m, n, K, nnz;
    int32_t row_splits;  // split y takes every row_splits-th group of 16 rows, from group y on
    int32_t vec_ok;      // B and C 16-byte aligned, ldb and ldc multiples of 4
    float alpha, beta;
};

template <int S>
__device__ __forceinline__ int quad_bcast(int v) {  // every lane gets the value of lane S of its quad
    return __builtin_amdgcn_update_dpp(0, v, S * 0x55, 0xF, 0xF, true);
}

// acc += (val of lane S of the quad) * b: the quad broadcast rides on the multiply-add itself.
// All 64 lanes are active wherever this is used.
template <int S>
__device__ __forceinline__ void fma_quad(float& acc, float val, float b) {
    if constexpr (S == 0)
        asm("v_fmac_f32_dpp %0, %1, %2 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf bound_ctrl:1" : "+v"(acc) : "v"(val), "v"(b));
    else if constexpr (S == 1)
        asm("v_fmac_f32_dpp %0, %1, %2 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf bound_ctrl:1" : "+v"(acc) : "v"(val), "v"(b));
    else if constexpr (S == 2)
        asm("v_fmac_f32_dpp %0, %1, %2 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf bound_ctrl:1" : "+v"(acc) : "v"(val), "v"(b));
    else
        asm("v_fmac_f32_dpp %0, %1, %2 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf bound_ctrl:1" : "+v"(acc) : "v"(val), "v"(b));
}

// 4-byte aligned vectors of four: a row's entries start anywhere in colidx / vals.
typedef int32_t i32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2_a2 __attribute__((ext_vector_type(2), aligned(2)));

__device__ __forceinline__ f32x4 widen4(u32x2_t b) {  // four bf16 values, little-endian pairs
    return f32x4{__uint_as_float(b[0] << 16), __uint_as_float(b[0] & 0xFFFF0000u), __uint_as_float(b[1] << 16),
                 __uint_as_float(b[1] & 0xFFFF0000u)};
}
// Four consecutive stored values from element k on (any alignment the element type allows), as floats.
__device__ __forceinline__ f32x4 load4_any(const float* p, int64_t k) { return *reinterpret_cast<const f32x4_a4*>(p + k); }
__device__ __forceinline__ f32x4 load4_any(const uint16_t* p, int64_t k) { return widen4(*reinterpret_cast<const u32x2_a2*>(p + k)); }
// Four consecutive values from a 16-byte (float) or 8-byte (bf16) aligned address.
__device__ __forceinline__ f32x4 load4_aligned(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load4_aligned(const uint16_t* p) { return widen4(*reinterpret_cast<const u32x2_t*>(p)); }

// Copies rows cb0 .. cb0+nbk-1 of the slice of B (columns k0 .. k0+kw-1) to the LDS block Bs[row][16] as floats.
template <typename E>
__device__ __forceinline__ void stage_b_block(const E* B, int64_t ldb, int cb0, int nbk, int k0, int kw, bool vec_ok, float* Bs,
                                              int tid) {
    for (int idx = tid; idx < nbk * 4; idx += kSpmmWG) {
        const int j = idx >> 2, qq = idx & 3;
        const E* src = B + static_cast<size_t>(cb0 + j) * ldb + k0 + 4 * qq;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (vec_ok && 4 * qq + 4 <= kw) {
            v = load4_aligned(src);
        } else {
            for (int t = 0; t < 4; ++t)
                if (4 * qq + t < kw) v[t] = widen(src[t]);
        }
        *reinterpret_cast<f32x4*>(Bs + j * kSpmmKT + 4 * qq) = v;
    }
}

// SINGLE: B has at most kSpmmNB rows, so one block holds all of it and cb0 is 0 throughout.
// SORTED: the wavefronts take their rows from a.rows (rows of like length side by side) instead
// of in natural order.
template <typename T, bool SINGLE, bool SORTED>
__global__ __launch_bounds__(kSpmmWG) void spmm_csr_kernel(const SpmmArgs a) {
    using E = typename T::elem;
    const E* const a_vals = static_cast<const E*>(a.vals);
    constexpr int KT = kSpmmKT, NB = kSpmmNB, RPW = 16, WAVES = kSpmmWG / 64;
    constexpr int U = 8;  // entries per lane and chunk: a chunk covers 32 entries of a row
    static_assert(KT == 16, "four lanes per row, one float4 each");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float* Bs = reinterpret_cast<float*>(smem_raw);  // [NB + 1][KT]; row NB stays zero
    const unsigned char* const Bq = smem_raw + 16 * (threadIdx.x & 3);  // this lane's float4 of row 0
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = lane & 3;      // which float4 of the slice, and which entries of the row (4q .. 4q+3, 16+4q .. 16+4q+3)
    const int rsub = lane >> 2;  // which of the wavefront's 16 rows

    // Workgroup ids are handed to the 8 dies round-robin.  Die j takes a contiguous run of
    // (slice, split) pairs, so that the slices whose pieces of a row of C lie side by side are
    // written through the same L2.
    const int n_slices = (a.K + KT - 1) / KT;
    int pair;
    {
        const int nb = gridDim.x, per = nb / kXcds, rem = nb % kXcds;
        const int die = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
        pair = die * per + (die < rem ? die : rem) + slot;
    }
    const int slice = pair % n_slices, split = pair / n_slices;
    const int k0 = slice * KT;
    const int kw = a.K - k0 < KT ? a.K - k0 : KT;  // live columns of this slice
    const bool full4 = a.vec_ok && 4 * q + 4 <= kw;  // this lane's float4 lies wholly inside the slice

    if (a.nnz == 0) {  // C <- beta*C; the main path below may then assume that A has entries
        const int row_lo = static_cast<int>(static_cast<int64_t>(a.m) * split / a.row_splits);
        const int row_hi = static_cast<int>(static_cast<int64_t>(a.m) * (split + 1) / a.row_splits);
        for (int r = row_lo + tid / 4; r < row_hi; r += kSpmmWG / 4) {
            float* dst = a.C + static_cast<size_t>(r) * a.ldc + k0 + 4 * q;
            for (int t = 0; t < 4; ++t)
                if (4 * q + t < kw) dst[t] = a.beta != 0.f ? a.beta * dst[t] : 0.f;
        }
        return;
    }
    if (tid < KT) Bs[NB * KT + tid] = 0.f;  // the row that entries without a partner in this block point to

    // Rows are dealt out in groups of 16 positions of the row order.  Workgroup (slice, split y of S)
    // takes the groups y, y + S, y + 2S, ..: with the rows sorted by length every split gets its
    // share of the long ones.  Its wavefronts take those in turn.  All slices walk through the
    // rows in the same order, so a row of C is written, piece by piece, within a short time.
    const int S = a.row_splits, y = split;
    const int total_groups = (a.m + RPW - 1) / RPW;
    const int n_groups = total_groups > y ? (total_groups - y + S - 1) / S : 0;
    auto pos_of = [&](int j) {  // position of this lane's row in the wavefront's j-th group; m or more: none
        if (j >= n_groups) return a.m;
        return (y + S * j) * RPW + rsub;
    };
    // A lane without a row takes the last row again (and stores nothing): no select on loaded
    // values anywhere, so nothing tempts the compiler into a branch with a wait behind it.
    auto load_id = [&](int j) {
        int p = pos_of(j);
        p = p < a.m ? p : a.m - 1;
        return SORTED ? a.rows[p] : p;
    };
    auto load_row = [&](int r, int& rs, int& len) {  // first entry and length of row r
        const int32_t* rp = a.rowptr + r;
        rs = rp[0];
        len = rp[1] - rs;
    };

    for (int cb0 = 0; cb0 < (SINGLE ? 1 : a.n); cb0 += NB) {
        const int nbk = a.n - cb0 < NB ? a.n - cb0 : NB;  // rows of B in this block
        if (cb0 > 0) __syncthreads();                     // the previous block is no longer read
        stage_b_block(static_cast<const E*>(a.B), a.ldb, cb0, nbk, k0, kw, a.vec_ok != 0, Bs, tid);
        __syncthreads();

        // A chunk is 32 consecutive entries of the lane's row from entry c0 on; lane q of the quad
        // holds entries 4q .. 4q+3 (slots 0..3) and 16+4q .. 16+4q+3 (slots 4..7) of it, two 16-byte
        // loads per array.  issue() only requests them, so the loads stay in flight while something
        // else is multiplied; a lane reads on past the end of its row (into the next rows) and
        // finish() sorts that out.  Only near the end of the arrays (the last rows of the matrix)
        // are the reads clamped one by one.
        auto issue = [&](int rs, int c0, int (&col)[U], float (&val)[U]) {
            const int kq = rs + c0 + 4 * q;
            if (!__builtin_amdgcn_ballot_w64(kq + 20 > a.nnz)) {
                const i32x4_a4 ca = *reinterpret_cast<const i32x4_a4*>(a.colidx + kq);
                const i32x4_a4 cb = *reinterpret_cast<const i32x4_a4*>(a.colidx + kq + 16);
                const f32x4 va = load4_any(a_vals, kq);
                const f32x4 vb = load4_any(a_vals, kq + 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    col[e] = ca[e];
                    col[4 + e] = cb[e];
                    val[e] = va[e];
                    val[4 + e] = vb[e];
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int t = kq + 16 * (u >> 2) + (u & 3);
                    const int k = t < a.nnz ? t : a.nnz - 1;
                    col[u] = a.colidx[k];
                    val[u] = widen(a_vals[k]);
                }
            }
        };
        // Column -> byte offset of the B row in the LDS block.  Entries past the row's end, or with a
        // column outside this block, point at the zero row; the former also get the value 0 (they
        // belong to another row, whose value need not be finite).
        auto finish = [&](int len, int c0, int (&col)[U], float (&val)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool live = c0 + 16 * (u >> 2) + 4 * q + (u & 3) < len;
                unsigned c = static_cast<unsigned>(col[u] - (SINGLE ? 0 : cb0));  // a column before the block wraps to a huge number
                c = c < static_cast<unsigned>(NB) ? c : static_cast<unsigned>(NB);
                c = live ? c : static_cast<unsigned>(NB);
                col[u] = static_cast<int>(c * (KT * 4));
                val[u] = live ? val[u] : 0.f;
            }
        };

        // Three stages in flight: row ids three groups ahead, row bounds two ahead, entries one ahead.
        int gi = wave;
        int r = load_id(gi), r_n = load_id(gi + WAVES), r_nn = load_id(gi + 2 * WAVES);
        int rs, len, rs_n, len_n;
        load_row(r, rs, len);
        load_row(r_n, rs_n, len_n);
        int col[U], coln[U];
        float val[U], valn[U];
        issue(rs, 0, col, val);
        finish(len, 0, col, val);
        while (gi < n_groups) {
            issue(rs_n, 0, coln, valn);
            int rs_nn, len_nn;
            load_row(r_nn, rs_nn, len_nn);
            int r_nnn = load_id(gi + 3 * WAVES);

            float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f, acc3 = 0.f;
            for (int c0 = 0;; c0 += 4 * U) {
                // Step st takes entries c0 + 4 st .. c0 + 4 st + 3 of every row: slots 4 (st / 4) .. + 3
                // of lane st % 4 of the quad.  Two steps per trip.
#define SPMM_STEP_LOADS(B0, ST)                                                                                  \
    B0[0] = *reinterpret_cast<const f32x4*>(Bq + quad_bcast<(ST) % 4>(col[4 * ((ST) / 4) + 0]));                \
    B0[1] = *reinterpret_cast<const f32x4*>(Bq + quad_bcast<(ST) % 4>(col[4 * ((ST) / 4) + 1]));                \
    B0[2] = *reinterpret_cast<const f32x4*>(Bq + quad_bcast<(ST) % 4>(col[4 * ((ST) / 4) + 2]));                \
    B0[3] = *reinterpret_cast<const f32x4*>(Bq + quad_bcast<(ST) % 4>(col[4 * ((ST) / 4) + 3]));
#define SPMM_STEP_FMAS(B0, ST)                                                 \
    _Pragma("unroll") for (int e = 0; e < 4; ++e) {                            \
        fma_quad<(ST) % 4>(acc0, val[4 * ((ST) / 4) + e], B0[e][0]);           \
        fma_quad<(ST) % 4>(acc1, val[4 * ((ST) / 4) + e], B0[e][1]);           \
        fma_quad<(ST) % 4>(acc2, val[4 * ((ST) / 4) + e], B0[e][2]);           \
        fma_quad<(ST) % 4>(acc3, val[4 * ((ST) / 4) + e], B0[e][3]);           \
    }
#define SPMM_TWO_STEPS(ST)                                                                     \
    if (__builtin_amdgcn_ballot_w64(c0 + 4 * (ST) < len)) {                                    \
        f32x4 b0[4], b1[4];                                                                    \
        SPMM_STEP_LOADS(b0, ST) SPMM_STEP_LOADS(b1, (ST) + 1)                                  \
        SPMM_STEP_FMAS(b0, ST) SPMM_STEP_FMAS(b1, (ST) + 1)                                    \
    } else {                                                                                   \
        break;                                                                                 \
    }
                do {  // left by the first pair of steps that no row of the wavefront reaches
                    SPMM_TWO_STEPS(0) SPMM_TWO_STEPS(2) SPMM_TWO_STEPS(4) SPMM_TWO_STEPS(6)
                } while (false);
#undef SPMM_TWO_STEPS
#undef SPMM_STEP_FMAS
#undef SPMM_STEP_LOADS
                if (!__builtin_amdgcn_ballot_w64(c0 + 4 * U < len)) break;
                issue(rs, c0 + 4 * U, col, val);  // rows longer than a chunk: fetched on demand
                finish(len, c0 + 4 * U, col, val);
            }

            // What the next round needs is settled before C is touched: nothing that is loaded is
            // then still awaited when the loop comes round, and the store below stays in flight.
            finish(len_n, 0, coln, valn);
            asm volatile("" : "+v"(rs_nn), "+v"(len_nn), "+v"(r_nnn));

            if (pos_of(gi) < a.m && 4 * q < kw) {
                float* dst = a.C + static_cast<size_t>(r) * a.ldc + k0 + 4 * q;
                const bool first = cb0 == 0;
                const bool reads_c = !first || a.beta != 0.f;
                const float scale_c = first ? a.beta : 1.f;
                const f32x4 acc = {acc0, acc1, acc2, acc3};
                if (full4) {
                    f32x4 out = a.alpha * acc;
                    if (reads_c) out += scale_c * *reinterpret_cast<const f32x4*>(dst);
                    __builtin_nontemporal_store(out, reinterpret_cast<f32x4*>(dst));  // written once, not read again soon
                } else {
                    for (int t = 0; t < 4; ++t)
                        if (4 * q + t < kw) dst[t] = a.alpha * acc[t] + (reads_c ? scale_c * dst[t] : 0.f);
                }
            }
            gi += WAVES;
            r = r_n;
            r_n = r_nn;
            r_nn = r_nnn;
            rs = rs_n;
            len = len_n;
            rs_n = rs_nn;
            len_n = len_nn;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                col[u] = coln[u];
                val[u] = valn[u];
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// The same product from a packed copy of A (built at analysis time on request).  The rows are
// taken in the length-sorted order; group g (16 rows) is stored as ceil(longest row / 16) blocks,
// a block being what one load of the wavefront fetches: lane (row rsub, quad lane q) owns the four
// slots of the entries ranked 16b + 4q .. 16b + 4q + 3 in its row's order (below), columns and values in arrays of their
// own.  The order inside a row deals the entries out by column residue modulo 4, turned by the row's position: B's rows
// lie 64 bytes apart in LDS, four to a cycle of the banks, and the 16 rows a wavefront reads at once then fall on the
// four quarters in turn (bank-conflict cycles -44 % against storage order).  Slots past a row's end hold the value 0
// and a column that maps to the zero row.  Against
// reading CSR directly: every load is aligned and fully coalesced, columns take 2 bytes while
// n <= 32768, no row bounds are fetched, no entry needs a validity test, and the number of steps
// of a group is a scalar from its descriptor.
struct SpmmPackedArgs {
    const int32_t* desc;  // pairs (first block, steps of 4 entries) per group, one closing pair
    const void* pcol;     // [blocks + 1][64 lanes][4]: uint16 or int32; the last block is padding only
    const float* pval;    // [blocks + 1][64][4]
    const int32_t* rows;  // [m] the row order
    const void* B;        // float or bf16 bit patterns
    float* C;
    int64_t ldb, ldc;
    int32_t m, n, K, num_groups;
    int32_t row_splits, vec_ok;
    float alpha, beta;
};

// Column number a padding slot holds: the zero row itself when all of B fits one block, else a
// number no block of B contains.
template <typename CT>
__host__ __device__ inline CT packed_pad_column(int n) {
    return n <= kSpmmNB ? static_cast<CT>(kSpmmNB) : static_cast<CT>(-1);
}

template <typename CT, typename E>
__global__ __launch_bounds__(64) void spmm_pack_kernel(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                       const E* __restrict__ vals, const int32_t* __restrict__ rows,
                                                       const int32_t* __restrict__ desc, int m, int n, CT* __restrict__ pcol,
                                                       float* __restrict__ pval, int32_t* __restrict__ psrc) {
    const int g = blockIdx.x, lane = threadIdx.x, rsub = lane >> 2, q = lane & 3;
    const int first = desc[2 * g], nblocks = desc[2 * g + 2] - first;
    const int pos = 16 * g + rsub;
    int rs = 0, len = 0;
    if (pos < m) {
        const int r = rows[pos];
        rs = rowptr[r];
        len = rowptr[r + 1] - rs;
    }
    const CT pad = packed_pad_column<CT>(n);
    // padding first: the slots past the row's end
    for (int b = 0; b < nblocks; ++b) {
        const size_t slot0 = (static_cast<size_t>(first + b) * 64 + lane) * 4;
        for (int e = 0; e < 4; ++e) {
            if (16 * b + 4 * q + e >= len) {
                pcol[slot0 + e] = pad;
                pval[slot0 + e] = 0.f;
                if (psrc) psrc[slot0 + e] = -1;
            }
        }
    }
    // The row's entries, one lane per row.  Entry e, the j-th of the row's entries with its column residue, has the key
    // 4 j + d with d = (column - pos) mod 4; its rank is the number of entries with a smaller key: of the entries with
    // difference dd, those numbered below j (and number j itself when dd < d), as far as there are any.
    if (q == 0 && len > 0) {
        int cnt[4] = {0, 0, 0, 0};
        for (int k = 0; k < len; ++k) ++cnt[(colidx[rs + k] - pos) & 3];
        int seen[4] = {0, 0, 0, 0};
        for (int k = 0; k < len; ++k) {
            const int c = colidx[rs + k];
            const int d = (c - pos) & 3;
            const int j = seen[d]++;
            int t = 0;
#pragma unroll
            for (int dd = 0; dd < 4; ++dd) {
                const int below = j + (dd < d ? 1 : 0);
                t += cnt[dd] < below ? cnt[dd] : below;
            }
            const size_t slot = ((static_cast<size_t>(first + (t >> 4)) * 64 + 4 * rsub + ((t >> 2) & 3)) * 4) + (t & 3);
            pcol[slot] = static_cast<CT>(c);
            pval[slot] = widen(vals[rs + k]);
            if (psrc) psrc[slot] = rs + k;
        }
    }
}

// One block of the packed copy as a lane holds it.
template <typename CT>
struct PackedBlock;
template <>
struct PackedBlock<uint16_t> {
    unsigned c01, c23;  // four 16-bit columns
    f32x4 v;
    // block: the same in every lane (a scalar base address), lane: the only per-lane part of the address
    __device__ __forceinline__ void load(const void* pcol, const float* pval, int block, int lane) {
        const uint16_t* cb = static_cast<const uint16_t*>(pcol) + static_cast<size_t>(block) * 256;
        const float* vb = pval + static_cast<size_t>(block) * 256;
        const uint2 c = *reinterpret_cast<const uint2*>(cb + static_cast<unsigned>(4 * lane));
        c01 = c.x;
        c23 = c.y;
        v = *reinterpret_cast<const f32x4*>(vb + static_cast<unsigned>(4 * lane));
    }
    __device__ __forceinline__ unsigned col(int e) const {
        const unsigned w = e < 2 ? c01 : c23;
        return (e & 1) ? w >> 16 : w & 0xFFFFu;
    }
    __device__ __forceinline__ void touch() { asm volatile("" : "+v"(c01), "+v"(c23), "+v"(v)); }
};
template <>
struct PackedBlock<int32_t> {
    i32x4 c;
    f32x4 v;
    __device__ __forceinline__ void load(const void* pcol, const float* pval, int block, int lane) {
        c = *reinterpret_cast<const i32x4*>(static_cast<const int32_t*>(pcol) + static_cast<size_t>(block) * 256 + static_cast<unsigned>(4 * lane));
        v = *reinterpret_cast<const f32x4*>(pval + static_cast<size_t>(block) * 256 + static_cast<unsigned>(4 * lane));
    }
    __device__ __forceinline__ unsigned col(int e) const { return static_cast<unsigned>(c[e]); }
    __device__ __forceinline__ void touch() { asm volatile("" : "+v"(c), "+v"(v)); }
};

template <typename T, bool SINGLE, typename CT>
__global__ __launch_bounds__(kSpmmWG) void spmm_packed_kernel(const SpmmPackedArgs a) {
    using E = typename T::elem;
    constexpr int KT = kSpmmKT, NB = kSpmmNB, RPW = 16, WAVES = kSpmmWG / 64;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float* Bs = reinterpret_cast<float*>(smem_raw);  // [NB + 1][KT]; row NB stays zero
    const unsigned char* const Bq = smem_raw + 16 * (threadIdx.x & 3);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // the same in every lane: what depends on it alone stays in scalar registers
    const int q = lane & 3, rsub = lane >> 2;

    // die-aware numbering of the (slice, split) pairs, as in spmm_csr_kernel
    const int n_slices = (a.K + KT - 1) / KT;
    int pair;
    {
        const int nb = gridDim.x, per = nb / kXcds, rem = nb % kXcds;
        const int die = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
        pair = die * per + (die < rem ? die : rem) + slot;
    }
    const int slice = pair % n_slices, split = pair / n_slices;
    const int k0 = slice * KT;
    const int kw = a.K - k0 < KT ? a.K - k0 : KT;
    const bool full4 = a.vec_ok && 4 * q + 4 <= kw;
    if (tid < KT) Bs[NB * KT + tid] = 0.f;

    const int S = a.row_splits, y = split;
    const int n_groups = a.num_groups > y ? (a.num_groups - y + S - 1) / S : 0;  // this workgroup's
    // (first block, steps) of the wavefront's j-th group; past the end: the closing pair (all blocks, 0)
    auto load_desc = [&](int j, int& first, int& nsteps) {
        const int g = j < n_groups ? y + S * j : a.num_groups;
        first = a.desc[2 * g];
        nsteps = a.desc[2 * g + 1];
    };

    for (int cb0 = 0; cb0 < (SINGLE ? 1 : a.n); cb0 += NB) {
        const int nbk = a.n - cb0 < NB ? a.n - cb0 : NB;
        if (cb0 > 0) __syncthreads();
        stage_b_block(static_cast<const E*>(a.B), a.ldb, cb0, nbk, k0, kw, a.vec_ok != 0, Bs, tid);
        __syncthreads();

        // column -> byte offset of the B row in the LDS block; padding and columns of other blocks -> zero row
        auto offsets = [&](const PackedBlock<CT>& blk, int (&off)[4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                unsigned c = blk.col(e);
                if constexpr (!SINGLE) {
                    c -= static_cast<unsigned>(cb0);  // a column before the block wraps to a huge number
                    c = c < static_cast<unsigned>(NB) ? c : static_cast<unsigned>(NB);
                }
                off[e] = static_cast<int>(c * (KT * 4));
            }
        };

        int j = wave;
        int first, nsteps, first_n, nsteps_n;  // first_n, nsteps_n: as loaded (vector registers), one group ahead
        load_desc(j, first, nsteps);
        load_desc(j + WAVES, first_n, nsteps_n);
        first = __builtin_amdgcn_readfirstlane(first);
        nsteps = __builtin_amdgcn_readfirstlane(nsteps);
        PackedBlock<CT> cur;
        cur.load(a.pcol, a.pval, first, lane);
        while (j < n_groups) {
            // the next group's pair arrived a group ago; as scalars, block numbers and step counts cost no vector work
            const int first_nu = __builtin_amdgcn_readfirstlane(first_n);
            const int nsteps_nu = __builtin_amdgcn_readfirstlane(nsteps_n);
            const int pos = (y + S * j) * RPW + rsub;
            const int r = a.rows[pos < a.m ? pos : a.m - 1];
            float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f, acc3 = 0.f;
            const int nblocks = nsteps > 0 ? (nsteps + 3) / 4 : 1;  // a group of empty rows: one pass that multiplies nothing
            for (int b = 0; b < nblocks; ++b) {
                // the next block of the wavefront's stream: the group's next one, else the next group's first
                const int next_block = b + 1 < nblocks ? first + b + 1 : first_nu;
                PackedBlock<CT> nxt;
                nxt.load(a.pcol, a.pval, next_block, lane);
                const int steps = nsteps - 4 * b;  // steps of this block still to do (4 or more: all four)
                int off[4];
                offsets(cur, off);
#define SPMM_STEP_LOADS(B0, J)                                                   \
    B0[0] = *reinterpret_cast<const f32x4*>(Bq + quad_bcast<J>(off[0]));         \
    B0[1] = *reinterpret_cast<const f32x4*>(Bq + quad_bcast<J>(off[1]));         \
    B0[2] = *reinterpret_cast<const f32x4*>(Bq + quad_bcast<J>(off[2]));         \
    B0[3] = *reinterpret_cast<const f32x4*>(Bq + quad_bcast<J>(off[3]));
#define SPMM_STEP_FMAS(B0, J)                          \
    _Pragma("unroll") for (int e = 0; e < 4; ++e) {    \
        fma_quad<J>(acc0, cur.v[e], B0[e][0]);         \
        fma_quad<J>(acc1, cur.v[e], B0[e][1]);         \
        fma_quad<J>(acc2, cur.v[e], B0[e][2]);         \
        fma_quad<J>(acc3, cur.v[e], B0[e][3]);         \
    }
                // step J takes the four slots of lane J of every quad.  All LDS reads of the block go out
                // first, so the multiply-adds of the early steps run while the later rows arrive.
                {
                    f32x4 b0[4], b1[4], b2[4], b3[4];
                    switch (steps >= 4 ? 4 : steps) {
                        case 4:
                            SPMM_STEP_LOADS(b0, 0) SPMM_STEP_LOADS(b1, 1) SPMM_STEP_LOADS(b2, 2) SPMM_STEP_LOADS(b3, 3)
                            SPMM_STEP_FMAS(b0, 0) SPMM_STEP_FMAS(b1, 1) SPMM_STEP_FMAS(b2, 2) SPMM_STEP_FMAS(b3, 3)
                            break;
                        case 3:
                            SPMM_STEP_LOADS(b0, 0) SPMM_STEP_LOADS(b1, 1) SPMM_STEP_LOADS(b2, 2)
                            SPMM_STEP_FMAS(b0, 0) SPMM_STEP_FMAS(b1, 1) SPMM_STEP_FMAS(b2, 2)
                            break;
                        case 2:
                            SPMM_STEP_LOADS(b0, 0) SPMM_STEP_LOADS(b1, 1) SPMM_STEP_FMAS(b0, 0) SPMM_STEP_FMAS(b1, 1)
                            break;
                        case 1:
                            SPMM_STEP_LOADS(b0, 0) SPMM_STEP_FMAS(b0, 0)
                            break;
                        default:
                            break;
                    }
                }
#undef SPMM_STEP_FMAS
#undef SPMM_STEP_LOADS
                nxt.touch();  // arrived before anything is stored: the loop never waits behind a store
                cur = nxt;
            }

            if (pos < a.m && 4 * q < kw) {
                float* dst = a.C + static_cast<size_t>(r) * a.ldc + k0 + 4 * q;
                const bool first_pass = cb0 == 0;
                const bool reads_c = !first_pass || a.beta != 0.f;
                const float scale_c = first_pass ? a.beta : 1.f;
                const f32x4 acc = {acc0, acc1, acc2, acc3};
                if (full4) {
                    f32x4 out = a.alpha * acc;
                    if (reads_c) out += scale_c * *reinterpret_cast<const f32x4*>(dst);
                    __builtin_nontemporal_store(out, reinterpret_cast<f32x4*>(dst));  // written once, not read again soon
                } else {
                    for (int t = 0; t < 4; ++t)
                        if (4 * q + t < kw) dst[t] = a.alpha * acc[t] + (reads_c ? scale_c * dst[t] : 0.f);
                }
            }
            j += WAVES;
            first = first_nu;
            nsteps = nsteps_nu;
            load_desc(j + WAVES, first_n, nsteps_n);
        }
    }
}


// ------------------------------------------------------------------------------------------
// The product for B of at most 2048 rows, from a second packed form of A ("pairs"): two lanes per row, eight columns each.
//
// Bound: the LDS feeds one B value per multiply-add and the vector units issue one multiply-add per B value, so both are
// near their limit at once and what counts is everything besides.  Measured on this chip, a 128-bit LDS read of a wavefront
// goes out in four phases of 16 lanes and a phase takes as many cycles as the most used of its 256-byte bank row's slots
// has addresses: 4.5 cycles without conflicts, 8.8 for quads reading random 64-byte rows.
//   - Two lanes per row instead of four: the address add of an entry serves eight multiply-adds of a lane instead of four
//     (9 vector instructions per entry and 512 products; the four-lane kernel needs 10 and spent 16 with its overheads),
//     and a group's fixed cost (descriptor, row numbers, epilogue) falls on 32 rows instead of 16.
//   - B's slice lies in LDS as two halves of eight columns: row j at 512 (j / 8) + 32 (j mod 8), the second half 256 bytes
//     on, so both reads of an entry share one address (the 256 is an instruction offset) and a row occupies one of eight
//     32-byte slots of the banks.  A phase holds eight rows.
//   - The entries of eight rows that share a phase are put, at analysis time, in an order in which as few of a step's eight
//     entries as possible meet in one slot (spmm_pair_pack_kernel): 1.41 cycles per phase on the benchmark's matrices (5.65 LDS
//     cycles per read, counted) against 2.6 for storage order (simulated); padding points at zero rows in slots that are free.
//   - Offsets are stored ready for use (32 bits), so an entry costs no unpacking.
//   - A wavefront works through its blocks as one stream, across the ends of groups: the LDS reads of a step go out before
//     the multiply-adds of the step before, the entries are asked for kPairAhead blocks ahead, an old C a group ahead.  As it is
//     compiled this look-ahead ends with every group: the row number asked for there is moved to another register at once, and the wait
//     for it takes in what was asked for before it, the group's two stores among it (loads and stores share one counter, in order).
// 65536 x 2048 x 4096 at density 0.01, FP32: 432 us with the four-lane kernel, 368 with this one (30 TFLOP/s); without its
// stores of C 287: a row of C is written in 64-byte pieces, one per slice, a quarter of which leave in two requests (1.32 GB
// written for a C of 1.07), and that is what is left over the multiplication, whose LDS and vector units are busy 70 and
// 77 % of the time.  20011 x 2048 x 1000, bf16, C kept: 78 -> 55 us.
// A chain of steps per row is twice as long as the four-lane kernel's and a group twice as large: with few columns of C or
// rows of very different lengths that kernel is the faster one (spmm_pairs_choice).
constexpr int kPairRows = 32;                 // rows of a group: one wavefront, two lanes each
constexpr int kPairZeroRows = 8;              // one zero row per slot, behind the 2048 rows of B
constexpr int kPairLdsBytes = (kSpmmNB + kPairZeroRows) * kSpmmKT * 4;
constexpr int kPairSegment = 256;             // entries of a row that are ordered together

__host__ __device__ inline uint32_t pair_offset(uint32_t j) { return (j >> 3) * 512u + (j & 7u) * 32u; }

// The row of a group that is the i-th (0..7) of those whose lanes share phase s (0..3) of a 128-bit LDS read: the hardware
// takes lanes {0-3, 12-15, 20-27} and {4-11, 16-19, 28-31} of either half of the wavefront together (measured: of lanes that
// read different addresses in one slot, only those of one such set cost a cycle more).
__device__ __forceinline__ int pair_phase_row(int s, int i) {
    const unsigned long long rows = (s & 1) ? 0xFE985432ull : 0xDCBA7610ull;  // four bits each
    return 16 * (s >> 1) + static_cast<int>((rows >> (4 * i)) & 15);
}

struct SpmmPairArgs {
    const int32_t* desc;   // [2 * (num_groups + 1)] pairs (first block, steps of two entries: at least 1), one closing pair
    const uint32_t* ent;   // [blocks + 1][64][4] two byte offsets of B rows in LDS, then the two values
    const int32_t* rows;   // [m] the row order
    const void* B;
    float* C;
    int64_t ldb, ldc;
    int32_t m, n, K, num_groups, row_splits;
    float alpha, beta;
};

typedef float f32x4_a4s __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));

template <int H>
__device__ __forceinline__ int pair_bcast(int v) {  // every lane gets the value of lane H of its pair
    return __builtin_amdgcn_update_dpp(0, v, H == 0 ? 0xA0 : 0xF5, 0xF, 0xF, true);
}

// acc[0..7] += (v of lane H of the pair) * (lo, hi).  The broadcast is a move of its own for eight multiply-adds: riding on
// each of them (as in fma_quad) it saves a ninth of the instructions and measured 8 % slower.
template <int H>
__device__ __forceinline__ void fma_pair(float (&acc)[8], unsigned v, f32x4 lo, f32x4 hi) {
    const float w = __int_as_float(pair_bcast<H>(static_cast<int>(v)));
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        acc[t] = __builtin_fmaf(w, lo[t], acc[t]);
        acc[4 + t] = __builtin_fmaf(w, hi[t], acc[4 + t]);
    }
}

constexpr int kPairAhead = 7;  // 3, 5 and 7 measure the same (see above: every group's end waits for what is on its way)

// C32: every byte offset into C fits 32 bits, and row numbers and the row stride 24.
template <typename T, bool READ_C, bool C32>
__global__ __launch_bounds__(kSpmmWG) void spmm_pair_kernel(const SpmmPairArgs a) {
    using E = typename T::elem;
    constexpr int KT = kSpmmKT, WAVES = kSpmmWG / 64;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane & 1, rsub = lane >> 1;
    const unsigned char* const Bh = smem_raw + 16 * h;

    // die-aware numbering of the (slice, split) pairs, as in spmm_csr_kernel
    const int n_slices = (a.K + KT - 1) / KT;
    const int pair = xcd_remap(blockIdx.x, gridDim.x);
    const int slice = pair % n_slices, split = pair / n_slices;
    const int k0 = slice * KT;
    const int kw = a.K - k0 < KT ? a.K - k0 : KT;

    const int S = a.row_splits;
    const int n_groups = a.num_groups > split ? (a.num_groups - split + S - 1) / S : 0;  // this workgroup's
    auto group_of = [&](int jj) { return jj < n_groups ? split + S * jj : a.num_groups; };
    auto load_desc = [&](int jj, int& first, int& steps) {
        const int g = group_of(jj);
        first = a.desc[2 * g];
        steps = a.desc[2 * g + 1];
    };
    // the stream's reading end: block `at`, `left` blocks of its group from there on, the next group's pair on its way
    int jr = wave, at, left, first_n, steps_n;
    load_desc(jr, at, left);
    load_desc(jr + WAVES, first_n, steps_n);
    at = __builtin_amdgcn_readfirstlane(at);
    int todo = __builtin_amdgcn_readfirstlane(left);  // steps of two entries the group being multiplied still has to do
    left = (todo + 1) >> 1;
    auto load_block = [&](u32x4v& e) {
        e = (reinterpret_cast<const u32x4v*>(a.ent) + static_cast<size_t>(at) * 64)[static_cast<unsigned>(lane)];
        ++at;
        if (--left == 0) {
            at = __builtin_amdgcn_readfirstlane(first_n);
            left = (__builtin_amdgcn_readfirstlane(steps_n) + 1) >> 1;
            jr += WAVES;
            load_desc(jr + WAVES, first_n, steps_n);
        }
    };
    u32x4v e[kPairAhead + 1];
#pragma unroll
    for (int i = 0; i < kPairAhead; ++i) load_block(e[i]);

    // the slice of B: eight loads in flight per lane, then the LDS stores
    {
        const E* const B = static_cast<const E*>(a.B) + k0;
        constexpr int UB = 8;
        for (int base = tid; base < a.n * 4; base += UB * kSpmmWG) {
            f32x4 v[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int idx = base + u * kSpmmWG;
                const int row = idx >> 2, c = 4 * (idx & 3);
                v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (row < a.n) {
                    const E* src = B + static_cast<size_t>(row) * a.ldb + c;
                    if (c + 4 <= kw) {
                        v[u] = load4_any(src, 0);
                    } else {
                        for (int t = 0; t < 4; ++t)
                            if (c + t < kw) v[u][t] = widen(src[t]);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int idx = base + u * kSpmmWG;
                const int row = idx >> 2, qq = idx & 3;
                if (row < a.n) *reinterpret_cast<f32x4*>(smem_raw + pair_offset(row) + 256 * (qq >> 1) + 16 * (qq & 1)) = v[u];
            }
        }
        if (tid < 4 * kPairZeroRows) {
            const int row = kSpmmNB + (tid >> 2), qq = tid & 3;
            *reinterpret_cast<f32x4*>(smem_raw + pair_offset(row) + 256 * (qq >> 1) + 16 * (qq & 1)) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __syncthreads();
    int j = wave;
    if (j >= n_groups) return;

    // what the end of the group being multiplied needs: its row numbers, and the next group's steps
    const bool upper = (lane & 2) != 0;
    const int c = 4 * (lane & 3);
    auto load_row = [&](int jj) {
        const unsigned pos = static_cast<unsigned>(split + S * jj) * kPairRows + static_cast<unsigned>(rsub);
        return a.rows[pos < static_cast<unsigned>(a.m) ? pos : static_cast<unsigned>(a.m - 1)];
    };
    char* const C0 = reinterpret_cast<char*>(a.C + k0);
    auto pieces_of_c = [&](int row, char* (&dst)[2]) {  // this lane's piece of C in the rows of the quad's first and second pair
        if constexpr (C32) {
            const int at_row = static_cast<int>(__umul24(static_cast<unsigned>(row), static_cast<unsigned>(a.ldc) * 4u));
            dst[0] = C0 + (static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, at_row, 0x44, 0xF, 0xF, true)) + 4u * static_cast<unsigned>(c));  // quad_perm [0,1,0,1]
            dst[1] = C0 + (static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, at_row, 0xEE, 0xF, 0xF, true)) + 4u * static_cast<unsigned>(c));  // quad_perm [2,3,2,3]
        } else {
            dst[0] = C0 + 4 * (static_cast<size_t>(__builtin_amdgcn_update_dpp(0, row, 0x44, 0xF, 0xF, true)) * a.ldc + c);
            dst[1] = C0 + 4 * (static_cast<size_t>(__builtin_amdgcn_update_dpp(0, row, 0xEE, 0xF, 0xF, true)) * a.ldc + c);
        }
    };
    int r, r_n, todo_n;
    f32x4 old[2];
    auto whole = [&](int jj) { return kw == KT && (split + S * jj + 1) * kPairRows <= a.m; };  // the same for all lanes: whole rows and whole columns
    auto begin_group = [&]() {  // r: the row of this lane's pair
        if constexpr (READ_C) {
            if (whole(j)) {  // the old C travels while the group is multiplied
                char* dst[2];
                pieces_of_c(r, dst);
                old[0] = *reinterpret_cast<f32x4_a4s*>(dst[0]);
                old[1] = *reinterpret_cast<f32x4_a4s*>(dst[1]);
            }
        }
        r_n = load_row(j + WAVES);
        todo_n = a.desc[2 * group_of(j + WAVES) + 1];
    };
    r = load_row(j);
    begin_group();

    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x4 ra[4], rb[4];
    auto reads = [&](f32x4(&R)[4], unsigned off) {  // both reads of an entry share one address
        const unsigned char* const p0 = Bh + pair_bcast<0>(static_cast<int>(off));
        const unsigned char* const p1 = Bh + pair_bcast<1>(static_cast<int>(off));
        R[0] = *reinterpret_cast<const f32x4*>(p0);
        R[1] = *reinterpret_cast<const f32x4*>(p0 + 256);
        R[2] = *reinterpret_cast<const f32x4*>(p1);
        R[3] = *reinterpret_cast<const f32x4*>(p1 + 256);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto fmas = [&](const f32x4(&R)[4], unsigned val) {
        fma_pair<0>(acc, val, R[0], R[1]);
        fma_pair<1>(acc, val, R[2], R[3]);
        __builtin_amdgcn_sched_barrier(0);
    };
    reads(ra, e[0][0]);
    for (;;) {
#pragma unroll
        for (int i = 0; i <= kPairAhead; ++i) {
            u32x4v& now = e[i];
            u32x4v& next = e[(i + 1) % (kPairAhead + 1)];
            load_block(e[(i + kPairAhead) % (kPairAhead + 1)]);
            if (todo > 1) reads(rb, now[1]);  // (the last block of a group of an odd number of steps holds one)
            fmas(ra, now[2]);
            reads(ra, next[0]);
            if (todo > 1) fmas(rb, now[3]);
            todo -= 2;
            if (todo <= 0) {
                // A lane holds columns 4h .. 4h+3 and 8+4h .. 8+4h+3 of its row.  The two rows of a quad trade halves, so that
                // a store takes 64 bytes of a row from four lanes (with 32-byte pieces the product took 994 us instead of 421).
                f32x4 piece[2];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float give = upper ? acc[t] : acc[4 + t];
                    const float got = dpp_move<0x4E>(give);  // quad_perm [2,3,0,1]
                    piece[0][t] = upper ? got : acc[t];
                    piece[1][t] = upper ? acc[4 + t] : got;
                    acc[t] = acc[4 + t] = 0.f;
                }
                if (a.alpha != 1.f) {
                    piece[0] *= a.alpha;
                    piece[1] *= a.alpha;
                }
                char* dst[2];
                pieces_of_c(r, dst);
                if (whole(j)) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        if constexpr (READ_C) piece[u] += a.beta * old[u];
                        __builtin_nontemporal_store(static_cast<f32x4_a4s>(piece[u]), reinterpret_cast<f32x4_a4s*>(dst[u]));  // written once, not read again soon
                    }
                } else {
                    const int pos_even = (split + S * j) * kPairRows + (rsub & ~1);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        if (pos_even + u >= a.m) continue;
                        float* const p = reinterpret_cast<float*>(dst[u]);
                        if (c + 4 <= kw) {
                            if constexpr (READ_C) piece[u] += a.beta * static_cast<f32x4>(*reinterpret_cast<f32x4_a4s*>(p));
                            __builtin_nontemporal_store(static_cast<f32x4_a4s>(piece[u]), reinterpret_cast<f32x4_a4s*>(p));
                        } else {
                            for (int t = 0; t < 4; ++t)
                                if (c + t < kw) p[t] = READ_C ? piece[u][t] + a.beta * p[t] : piece[u][t];
                        }
                    }
                }
                j += WAVES;
                if (j >= n_groups) return;
                todo = __builtin_amdgcn_readfirstlane(todo_n);
                r = r_n;
                begin_group();
            }
        }
    }
}

// The largest of the 64 lanes' values (all active), as a scalar: permutes inside rows of 16 lanes, then every row hands its
// maximum on to the next, so that lane 63 ends up with the largest.
__device__ __forceinline__ int wave_max(int v) {
    auto step = [&](int other) { v = other > v ? other : v; };
    step(__builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
    step(__builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
    step(__builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    step(__builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false));  // row_mirror
    step(__builtin_amdgcn_update_dpp(INT32_MIN, v, 0x142, 0xA, 0xF, false));  // row_bcast15: rows 0, 2 to rows 1, 3
    step(__builtin_amdgcn_update_dpp(INT32_MIN, v, 0x143, 0xC, 0xF, false));  // row_bcast31: row 1 to rows 2, 3
    return __builtin_amdgcn_readlane(v, 63);
}

// Fills the pairs form: one wavefront per eight rows that share a phase of the LDS (pair_phase_row) and per stretch of
// kPairSegment entries (blockIdx.y, in strides).  Lane (r, c) = (lane / 8, lane mod 8) stands for row r's entries whose B row
// falls into slot c.  Steps are filled one after another: in a step every row that still has entries takes one of them,
// picked by a greedy matching - the (row, slot) with the fewest rows already in that slot, then the most entries left for the
// slot (less twice the row's number of other choices, plus twice the entries the row itself has there).
// src: the entry a slot holds, or -1.
// Bound: a chain of up to eight picks per step, each a maximum over the wavefront, one wavefront to itself.  So nothing but
// the pick stands in that chain: the entries lie in LDS slot by slot, which rows and slots are still open are scalar masks,
// and what a row took is written after the step's last pick.  With a load of the column inside the chain and the stretches
// one after another: 228 us for 65536 rows of 20 entries, 502 for 3000 of up to 200, 4900 for 64 of 2000; now 102, 196, 250.
__global__ __launch_bounds__(64) void spmm_pair_pack_kernel(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                            const int32_t* __restrict__ rows, const int32_t* __restrict__ desc, int m,
                                                            uint32_t* __restrict__ ent, int32_t* __restrict__ src) {
    __shared__ __align__(16) uint16_t cols[8][kPairSegment];  // the stretch's columns in storage order (from 2048 on: 2048)
    __shared__ uint32_t list[8][kPairSegment];                // the same slot by slot: column and place in the stretch
    const int lane = threadIdx.x, r = lane >> 3, c = lane & 7;
    const int set = blockIdx.x, g = set >> 2;
    const int first = desc[2 * g], blocks = desc[2 * g + 2] - first;
    const int in_group = pair_phase_row(set & 3, r);
    const int pos = kPairRows * g + in_group;
    int rs = 0, len = 0;
    if (pos < m) {
        const int row = rows[pos];
        rs = rowptr[row];
        len = rowptr[row + 1] - rs;
    }
    auto put = [&](int t, uint32_t offset, int k) {  // this lane's row, position t
        const size_t s = (static_cast<size_t>(first) + (t >> 2)) * 64 + 2 * in_group + (t & 1);
        ent[4 * s + ((t >> 1) & 1)] = offset;
        src[2 * s + ((t >> 1) & 1)] = k;
    };
    const int64_t positions = 4 * static_cast<int64_t>(blocks);
    const int64_t stride = static_cast<int64_t>(gridDim.y) * kPairSegment;
    for (int64_t start = static_cast<int64_t>(blockIdx.y) * kPairSegment; start < positions; start += stride) {
        const int t0 = static_cast<int>(start);
        int left = len - t0;  // of this row, in this stretch
        left = left < 0 ? 0 : (left > kPairSegment ? kPairSegment : left);
        for (int i = c; i < left; i += 8) {
            const uint32_t col = static_cast<uint32_t>(colidx[rs + t0 + i]);
            cols[r][i] = static_cast<uint16_t>(col < static_cast<uint32_t>(kSpmmNB) ? col : static_cast<uint32_t>(kSpmmNB));
        }
        __syncthreads();
        auto walk = [&](auto&& mine) {  // the row's entries in slot c, in storage order
            for (int i = 0; i < left; i += 8) {
                const u32x4v w = *reinterpret_cast<const u32x4v*>(&cols[r][i]);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t col = (w[u >> 1] >> (16 * (u & 1))) & 0xFFFFu;
                    if (i + u < left && static_cast<int>(col & 7u) == c) mine(i + u, col);
                }
            }
        };
        int cnt = 0;
        walk([&](int, uint32_t) { ++cnt; });
        int begin = cnt;  // exclusive prefix over the row's eight lanes
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
            const int up = __shfl_up(begin, d, 8);
            if (c >= d) begin += up;
        }
        begin -= cnt;
        {
            int at = begin;
            walk([&](int i, uint32_t col) { list[r][at++] = col << 16 | static_cast<uint32_t>(i); });
        }
        int total = cnt;  // entries left for slot c in all rows
#pragma unroll
        for (int d = 8; d < 64; d <<= 1) total += __shfl_xor(total, d);
        __syncthreads();
        uint32_t next = cnt > 0 ? list[r][begin] : 0;  // the entry this lane takes next
        const int stretch = positions - t0 < kPairSegment ? static_cast<int>(positions - t0) : kPairSegment;
        for (int t = 0; t < stretch; ++t) {
            unsigned long long live = __builtin_amdgcn_ballot_w64(cnt > 0);  // (row, slot) pairs that can still be picked in this step
            unsigned long long picked = 0;
            // the row's slots that have entries and are not taken in this step
            unsigned open = ((r < 4 ? static_cast<unsigned>(live) : static_cast<unsigned>(live >> 32)) >> (8 * (r & 3))) & 0xFFu;
            // score of the pair, 26 bits; a slot that is taken once more, and so has an entry less, comes after every one taken less often
            int score = ((1 << 16) + 16 + total + 2 * cnt - 2 * __popc(open)) * 64 + lane;
            while (live != 0) {
                const int win = wave_max(__builtin_amdgcn_inverse_ballot_w64(live) ? score : -1) & 63;
                const int wc = win & 7;
                picked |= 1ull << win;
                live &= ~(0xFFull << (win & 56));
                score += static_cast<int>((open >> wc) & 1u) << 7;  // one slot less to choose from
                open &= ~(1u << wc);
                score = c == wc ? score - ((1 << 12) + 1) * 64 : score;
            }
            const unsigned long long column = picked >> c & 0x0101010101010101ull;
            total -= __popcll(column);
            const bool won = __builtin_amdgcn_inverse_ballot_w64(picked);
            if (won) {
                put(t0 + t, pair_offset(next >> 16), rs + t0 + static_cast<int>(next & 0xFFFFu));
                ++begin;
                --cnt;
                if (cnt > 0) next = list[r][begin];
            }
            // rows without an entry here: zero rows in slots nobody reads, ascending (as many are free as rows remain)
            const unsigned long long empty = __builtin_amdgcn_ballot_w64(c == 0 && t >= left);
            if (empty != 0 && c == 0 && t >= left) {
                unsigned taken = static_cast<unsigned>(picked | picked >> 32);
                taken |= taken >> 16;
                unsigned free_slots = ~(taken | taken >> 8) & 0xFFu;
                for (int below = __popcll(empty & ((1ull << lane) - 1)); below > 0; --below) free_slots &= free_slots - 1;
                put(t0 + t, pair_offset(kSpmmNB + __ffs(free_slots) - 1), -1);
            }
        }
        __syncthreads();
    }
}

// The values of the packed copy (PAIRS = false): out[s] = vals[src[s]]; of the pairs form: out[4 q + 2 + i] = vals[src[2 q + i]]; 0 in
// padding.  65536 rows of 20 entries: 9 us each, packing the copy anew takes 50.
template <typename E, bool PAIRS>
__global__ __launch_bounds__(kWG) void spmm_values_kernel(const E* __restrict__ vals, const int32_t* __restrict__ src,
                                                          uint32_t* __restrict__ out, int64_t slots) {
    for (int64_t s = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x; s < slots; s += static_cast<int64_t>(gridDim.x) * kWG) {
        const int k = src[s];
        out[PAIRS ? 4 * (s >> 1) + 2 + (s & 1) : s] = k >= 0 ? __float_as_uint(widen(vals[k])) : 0u;
    }
}

}  // namespace

// Base addresses and leading dimensions must allow them.
bool spmm_vec_ok(bool bf16, const void* B, int64_t ldb, const float* C, int64_t ldc) {
    return reinterpret_cast<uintptr_t>(B) % (bf16 ? 8 : 16) == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0 && ldb % 4 == 0 &&
           ldc % 4 == 0;
}

namespace {

template <auto KERNEL, typename Args>
hipError_t launch_spmm_k(dim3 grid, dim3 block, size_t lds, hipStream_t st, const Args& a) {
    const hipError_t e = allow_lds<KERNEL>(lds);
    return e == hipSuccess ? launch_kernel(KERNEL, grid, block, lds, st, a) : e;
}

template <typename T>
hipError_t launch_spmm_t(const SpmmArgs& a, bool single, bool sorted, dim3 grid, size_t lds, hipStream_t st) {
    const dim3 block(kSpmmWG);
    if (sorted) return single ? launch_spmm_k<spmm_csr_kernel<T, true, true>>(grid, block, lds, st, a) : launch_spmm_k<spmm_csr_kernel<T, false, true>>(grid, block, lds, st, a);
    return single ? launch_spmm_k<spmm_csr_kernel<T, true, false>>(grid, block, lds, st, a) : launch_spmm_k<spmm_csr_kernel<T, false, false>>(grid, block, lds, st, a);
}

template <typename T>
hipError_t launch_spmm_packed_t(const SpmmPackedArgs& a, bool col16, bool single, dim3 grid, size_t lds, hipStream_t st) {
    const dim3 block(kSpmmWG);
    if (!col16) return launch_spmm_k<spmm_packed_kernel<T, false, int32_t>>(grid, block, lds, st, a);
    return single ? launch_spmm_k<spmm_packed_kernel<T, true, uint16_t>>(grid, block, lds, st, a)
                  : launch_spmm_k<spmm_packed_kernel<T, false, uint16_t>>(grid, block, lds, st, a);
}

template <typename CT>
hipError_t launch_spmm_pack_t(const MatrixView& A, const int32_t* rows, const int32_t* desc, int32_t num_groups, CT* pcol, float* pval,
                              int32_t* psrc, hipStream_t st) {
    if (A.bf16)
        launch_kernel((spmm_pack_kernel<CT, uint16_t>), dim3(num_groups), dim3(64), 0, st, A.rowptr, A.colidx,
                           static_cast<const uint16_t*>(A.vals), rows, desc, A.m, A.n, pcol, pval, psrc);
    else
        launch_kernel((spmm_pack_kernel<CT, float>), dim3(num_groups), dim3(64), 0, st, A.rowptr, A.colidx,
                           static_cast<const float*>(A.vals), rows, desc, A.m, A.n, pcol, pval, psrc);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_spmm(const MatrixView& A, const int32_t* rows, const void* B, int64_t ldb, float* C, int64_t ldc,
                       int32_t K, Scalars s, hipStream_t st) {
    if (A.m <= 0 || K <= 0) return hipSuccess;
    SpmmArgs a{};
    a.rowptr = A.rowptr;
    a.colidx = A.colidx;
    a.vals = A.vals;
    a.rows = rows;
    a.B = B;
    a.C = C;
    a.ldb = ldb;
    a.ldc = ldc;
    a.m = A.m;
    a.n = A.n;
    a.K = K;
    a.nnz = A.nnz;
    a.alpha = s.alpha;
    a.beta = s.beta;
    a.vec_ok = spmm_vec_ok(A.bf16, B, ldb, C, ldc) ? 1 : 0;
    const int slices = ceil_div(K, kSpmmKT);
    // one workgroup fits a CU (its B slice takes most of the LDS): aim at one per CU or more
    int splits = slices >= 256 ? 1 : ceil_div(256, slices);
    const int max_splits = ceil_div(A.m, 16);
    if (splits > max_splits) splits = max_splits;
    a.row_splits = splits;
    const size_t lds = sizeof(float) * (kSpmmNB + 1) * kSpmmKT;  // the B block and one zero row
    const dim3 grid(slices * splits);
    const bool single = A.n <= kSpmmNB;
    return A.bf16 ? launch_spmm_t<BF16>(a, single, rows != nullptr, grid, lds, st)
                  : launch_spmm_t<F32>(a, single, rows != nullptr, grid, lds, st);
}

hipError_t launch_spmm_pack(const MatrixView& A, const int32_t* rows, const int32_t* desc, int32_t num_groups, bool col16,
                            void* pcol, float* pval, int32_t* psrc, hipStream_t st) {
    if (num_groups <= 0) return hipSuccess;
    return col16 ? launch_spmm_pack_t(A, rows, desc, num_groups, static_cast<uint16_t*>(pcol), pval, psrc, st)
                 : launch_spmm_pack_t(A, rows, desc, num_groups, static_cast<int32_t*>(pcol), pval, psrc, st);
}

hipError_t launch_spmm_packed(const MatrixView& A, const PackedRows& P, const void* B, int64_t ldb, float* C, int64_t ldc,
                              int32_t K, Scalars s, hipStream_t st) {
    if (A.m <= 0 || K <= 0) return hipSuccess;
    SpmmPackedArgs a{};
    a.desc = P.desc;
    a.pcol = P.pcol;
    a.pval = P.pval;
    a.rows = P.rows;
    a.B = B;
    a.C = C;
    a.ldb = ldb;
    a.ldc = ldc;
    a.m = A.m;
    a.n = A.n;
    a.K = K;
    a.num_groups = P.num_groups;
    a.alpha = s.alpha;
    a.beta = s.beta;
    a.vec_ok = spmm_vec_ok(A.bf16, B, ldb, C, ldc) ? 1 : 0;
    const int slices = ceil_div(K, kSpmmKT);
    const int splits = spmm_packed_splits(slices, P.num_groups);
    a.row_splits = splits;
    const size_t lds = sizeof(float) * (kSpmmNB + 1) * kSpmmKT;
    const dim3 grid(slices * splits);
    return A.bf16 ? launch_spmm_packed_t<BF16>(a, P.col16, A.n <= kSpmmNB, grid, lds, st)
                  : launch_spmm_packed_t<F32>(a, P.col16, A.n <= kSpmmNB, grid, lds, st);
}

namespace {

template <typename T, bool READ_C, bool C32>
hipError_t launch_spmm_pair_k(const SpmmPairArgs& a, dim3 grid, hipStream_t st) {
    return launch_spmm_k<spmm_pair_kernel<T, READ_C, C32>>(grid, dim3(kSpmmWG), kPairLdsBytes, st, a);
}

template <typename T>
hipError_t launch_spmm_pair_t(const SpmmPairArgs& a, dim3 grid, hipStream_t st) {
    const bool c32 = a.m <= (1 << 24) && a.ldc < (1 << 22) && static_cast<int64_t>(a.m) * a.ldc * 4 <= (int64_t{1} << 32);
    if (c32) return a.beta != 0.f ? launch_spmm_pair_k<T, true, true>(a, grid, st) : launch_spmm_pair_k<T, false, true>(a, grid, st);
    return a.beta != 0.f ? launch_spmm_pair_k<T, true, false>(a, grid, st) : launch_spmm_pair_k<T, false, false>(a, grid, st);
}

int capped_grid(int64_t items) {
    const int64_t g = (items + kWG - 1) / kWG;
    return static_cast<int>(g > 8192 ? 8192 : (g < 1 ? 1 : g));
}

}  // namespace

hipError_t launch_spmm_pair_pack(const MatrixView& A, const PairRows& P, hipStream_t st) {
    if (P.num_groups <= 0) return hipSuccess;
    // a stretch of a long row is a workgroup of its own, as far as that does not make much more than 65536 of them
    const int64_t stretches = (2 * static_cast<int64_t>(P.longest_steps) + kPairSegment - 1) / kPairSegment;
    const int64_t most = 16384 / P.num_groups;
    const int per_row = static_cast<int>(stretches < most ? stretches : (most > 1 ? most : 1));
    launch_kernel(spmm_pair_pack_kernel, dim3(4 * P.num_groups, per_row), dim3(64), 0, st, A.rowptr, A.colidx, P.rows, P.desc, A.m, P.ent, P.src);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? launch_spmm_pair_values(A, P, st) : e;
}

namespace {

template <bool PAIRS>
hipError_t launch_spmm_values(const MatrixView& A, const int32_t* src, uint32_t* out, int64_t slots, hipStream_t st) {
    if (slots <= 0) return hipSuccess;
    if (A.bf16)
        launch_kernel((spmm_values_kernel<uint16_t, PAIRS>), dim3(capped_grid(slots)), dim3(kWG), 0, st,
                           static_cast<const uint16_t*>(A.vals), src, out, slots);
    else
        launch_kernel((spmm_values_kernel<float, PAIRS>), dim3(capped_grid(slots)), dim3(kWG), 0, st,
                           static_cast<const float*>(A.vals), src, out, slots);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_spmm_pair_values(const MatrixView& A, const PairRows& P, hipStream_t st) {
    return launch_spmm_values<true>(A, P.src, P.ent, P.num_blocks * 128, st);
}

hipError_t launch_spmm_packed_values(const MatrixView& A, const int32_t* psrc, float* pval, int64_t slots, hipStream_t st) {
    return launch_spmm_values<false>(A, psrc, reinterpret_cast<uint32_t*>(pval), slots, st);
}

hipError_t launch_spmm_pair(const MatrixView& A, const PairRows& P, const void* B, int64_t ldb, float* C, int64_t ldc, int32_t K,
                            Scalars s, hipStream_t st) {
    if (A.m <= 0 || K <= 0) return hipSuccess;
    if (A.n > kSpmmNB) return hipErrorInvalidValue;
    const int slices = ceil_div(K, kSpmmKT);
    const int splits = spmm_pair_splits(slices, P.num_groups, P.num_blocks);
    const SpmmPairArgs a{P.desc, P.ent, P.rows, B, C, ldb, ldc, A.m, A.n, K, P.num_groups, splits, s.alpha, s.beta};
    const dim3 grid(slices * splits);
    return A.bf16 ? launch_spmm_pair_t<BF16>(a, grid, st) : launch_spmm_pair_t<F32>(a, grid, st);
}

const char* spmm_kernel_name() { return "spmm_csr_kernel"; }
const char* spmm_packed_kernel_name() { return "spmm_packed_kernel"; }
const char* spmm_pair_kernel_name() { return "spmm_pair_kernel"; }

}  // namespace spmv
