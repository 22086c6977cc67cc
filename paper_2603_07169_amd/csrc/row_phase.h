// The row phase of the tile kernels: the entries of a tile sit in LDS and teams of lanes take one
// row (segment) each.  Shared by the CSR tile kernels.  Internal linkage.
#pragma once
#include <type_traits>

#include "device_common.h"

namespace spmv {
namespace {

constexpr int kMaxDeferred = 136;  // segments far longer than the tile's mean that can be set aside per tile

// Column type of a tile whose staged values are finished products: nothing is gathered, the row
// phase only adds.  cols and x are then null pointers that are never read.
struct NoGather {};
// The same for the sums of groups of eight entries: a batch of them is added up in 64 bits and rounded once.
struct GroupSums {};
// Column type of a tile whose x values stand in LDS at their entries' slots: slot j multiplies x[j].  cols is then a null pointer.
struct AtSlot {};

// B entries of one segment for one lane of a team of G lanes: staged slots j, j+G, .., j+(B-1)G.
// Three bursts of independent accesses, each issued back to back: column indices out of LDS,
// x out of memory, matrix values out of LDS.  G and B are compile-time so that every LDS
// access is the lane's base address plus an immediate offset, and nothing is predicated:
// the row phase is bound by instruction issue, so instructions per entry are what counts.
template <int B, int G, typename I, typename E>
__device__ __forceinline__ float gather_batch(const I* cols, const E* vals, const E* x, int j) {
    unsigned c[B];
    E xv[B];
    E av[B];
#pragma unroll
    for (int u = 0; u < B; ++u) c[u] = static_cast<unsigned>(cols[j + u * G]);
#pragma unroll
    for (int u = 0; u < B; ++u) xv[u] = x[c[u]];
#pragma unroll
    for (int u = 0; u < B; ++u) av[u] = vals[j + u * G];
    float acc = 0.f;
#pragma unroll
    for (int u = 0; u < B; ++u) acc += widen(av[u]) * widen(xv[u]);
    return acc;
}

template <int B, int G>
__device__ __forceinline__ float gather_batch(const NoGather*, const float* vals, const float*, int j) {
    float p[B];
#pragma unroll
    for (int u = 0; u < B; ++u) p[u] = vals[j + u * G];
    // in a tree: fewer roundings in a row than one after another (4 M-row power law, two passes: 7.2e-8 -> 6.8e-8 off the 64-bit result)
#pragma unroll
    for (int d = 1; d < B; d *= 2)
#pragma unroll
        for (int u = 0; u + d < B; u += 2 * d) p[u] += p[u + d];
    return p[0];
}

template <int B, int G>
__device__ __forceinline__ float gather_batch(const GroupSums*, const float* vals, const float*, int j) {
    float p[B];
#pragma unroll
    for (int u = 0; u < B; ++u) p[u] = vals[j + u * G];
    double acc = p[0];
#pragma unroll
    for (int u = 1; u < B; ++u) acc += p[u];
    return static_cast<float>(acc);
}

template <int B, int G, typename E>
__device__ __forceinline__ float gather_batch(const AtSlot*, const E* vals, const E* x, int j) {
    E xv[B], av[B];
#pragma unroll
    for (int u = 0; u < B; ++u) xv[u] = x[j + u * G];
#pragma unroll
    for (int u = 0; u < B; ++u) av[u] = vals[j + u * G];
    float acc = 0.f;
#pragma unroll
    for (int u = 0; u < B; ++u) acc += widen(av[u]) * widen(xv[u]);
    return acc;
}

// Partial dot product of the staged entries [b, e) of one segment, taken by lane `tl` of a team
// of G lanes: entry j of the segment goes to lane j mod G.  Neighbouring teams work on
// neighbouring rows, so for banded or stencil-like rows the lanes of a gather instruction fall
// into a handful of cache lines.  The lane's entries are taken in batches of 8, then 4, 2, 1.
template <int G, typename I, typename E>
__device__ __forceinline__ float segment_dot(const I* cols, const E* vals, const E* x, int b, int e, int tl) {
    // chunks of gathered x hold rows several times as long as a tile's: their batches are added in 64 bits
    std::conditional_t<std::is_same_v<I, AtSlot>, double, float> acc = 0;
    int j = b + tl;
    int cnt = (e - j + G - 1) / G;  // entries this lane takes (<= 0 when the segment is shorter than the team)
    for (; cnt >= 8; cnt -= 8, j += 8 * G) acc += gather_batch<8, G>(cols, vals, x, j);
    if (cnt >= 4) {
        acc += gather_batch<4, G>(cols, vals, x, j);
        j += 4 * G;
        cnt -= 4;
    }
    if (cnt >= 2) {
        acc += gather_batch<2, G>(cols, vals, x, j);
        j += 2 * G;
        cnt -= 2;
    }
    if (cnt >= 1) acc += gather_batch<1, G>(cols, vals, x, j);
    return static_cast<float>(acc);
}

// Where the row phase of a tile sends its results.
struct RowOut {
    float* y;
    const float* y0;  // LDS: y0[i] = old y of row r0+i when beta != 0 (fetched while the tile was loading)
    float alpha, beta;
    float* cut_sums;  // merge path only, LDS: [0] the finished part of a first row that began in an earlier chunk, [1] the sum of the cut-off piece
    bool head_cut;    // merge path only: the chunk's first row began in an earlier chunk and its part goes to cut_sums
};

// Where the parts of rows that are cut by chunk boundaries are put together (finish_cut).
struct CutOut {
    float* carry_val;          // [chunks] the sum of the piece a chunk cuts off at its end
    unsigned* arrivals;        // [chunks] 0 between runs
    const int32_t* cut_range;  // [2*(chunks+1)] per cut: first and last chunk of the row it cuts; null: they follow from rowptr and items
    const int32_t* rowptr;
    int items;                 // merge-path steps between cuts
    int32_t* carry_row;        // [chunks] not null: the pieces are left to cut_rows_kernel, with the row each belongs to (-1: none)
};

// A row in pieces: the chunks p0 .. p1 - 1 cut it at their ends and chunk p1 finishes it.  Every one of them leaves its part
// in memory - p0 .. p1 - 1 their sums in carry_val, p1 the finished part in y - and counts itself in arrivals[p0]; whoever
// comes last adds the carries to y in chunk order, so the result does not depend on who that is.  The counter wraps to 0 with the
// last arrival, so nothing has to be cleared between runs.  What one die writes another reads: the accesses are agent-scope
// atomics, which go past the dies' own L2s, and the part is in place (vmcnt 0) before its arrival is counted.
// A kernel behind the tiles that adds the carries (cut_rows_kernel) takes 1 to 3 us a run, this less than can be measured for a few
// dozen rows; but every chunk that takes part stays on for a store, an atomic and a load that other dies must see, so where many
// do the kernel is the cheaper way (use_cut_rows_kernel).
__device__ __forceinline__ void finish_cut(const RowOut& o, const CutOut& c, int r, int part, bool head, float value) {
    int p0, p1;
    if (c.cut_range) {
        const int cut = head ? part : part + 1;
        p0 = c.cut_range[2 * cut];
        p1 = c.cut_range[2 * cut + 1];
    } else {  // step r + rowptr[r] takes the row's first entry, step r + rowptr[r+1] finishes it
        p0 = static_cast<int>((static_cast<int64_t>(r) + c.rowptr[r]) / c.items);
        p1 = static_cast<int>((static_cast<int64_t>(r) + c.rowptr[r + 1]) / c.items);
    }
    __hip_atomic_store(head ? o.y + r : c.carry_val + part, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const unsigned last = static_cast<unsigned>(p1 - p0);
    if (atomicInc(c.arrivals + p0, last) != last) return;
    asm volatile("" ::: "memory");
    double s = 0;  // a row's parts in 64 bits: one that is cut many times would else be rounded at its full size as often
    for (int q = p0; q < p1; q += 8) {
        float part_sum[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            part_sum[u] = __hip_atomic_load(c.carry_val + (q + u < p1 ? q + u : q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (q + u < p1) s += part_sum[u];
    }
    const float y = static_cast<float>(__hip_atomic_load(o.y + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + o.alpha * s);
    __hip_atomic_store(o.y + r, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Row phase of a tile whose entries sit in LDS (cols[], vals[]); seg[i] .. seg[i+1] bounds the
// slots of segment i.  cols[] indexes x[]: global column numbers into the x vector in memory,
// or 16-bit positions into the tile's x window in LDS.  Segments 0 .. nr-1 are the rows r0 .. r0+nr-1 and go to y.  With MERGE
// there is one more segment, the piece of row r0+nr that the chunk cuts off: its sum is the
// chunk's carry (left in cut_sums for finish_cuts).  Teams of G lanes take one segment each;
// segments longer than defer_len are set aside and taken by whole wavefronts afterwards.
// Entered by the whole workgroup with *n_deferred == 0; contains one barrier.
template <bool MERGE, int WG, int G, typename I, typename E>
__device__ __forceinline__ void tile_rows_g(const I* cols, const E* vals, const E* x, const int* seg, int nr, int r0,
                                            const RowOut& o, int* deferred, int* n_deferred, int tid) {
    const int nseg = nr + (MERGE ? 1 : 0);
    constexpr int defer_len = 32 * G > 64 ? 32 * G : 64;
    constexpr int teams = WG / G;
    const int team = tid / G;
    const int tl = tid % G;

    auto emit = [&](int i, float s) {
        if (!MERGE || i < nr) {  // without the extra segment the test costs the windowed kernel 2 to 4 %
            const float v = epilogue(s, o.alpha, o.beta, o.y0, i);
            if (!(MERGE && i == 0 && o.head_cut)) o.y[r0 + i] = v;
            else o.cut_sums[0] = v;
        } else {
            o.cut_sums[1] = s;
        }
    };

    for (int base = 0; base < nseg; base += teams) {
        const int i = base + team;
        float acc = 0.f;
        bool mine = false;
        if (i < nseg) {
            const int b = seg[i], e = seg[i + 1];
            if (e - b <= defer_len) {
                mine = true;
                acc = segment_dot<G>(cols, vals, x, b, e, tl);
            } else if (tl == 0) {
                deferred[atomicAdd(n_deferred, 1)] = i;
            }
        }
        acc = group_sum<G>(acc);  // every lane takes part
        if (mine && tl == 0) emit(i, acc);
    }
    __syncthreads();

    const int nd = *n_deferred;
    const int lane = tid & 63;
    for (int d = tid >> 6; d < nd; d += WG / 64) {
        const int i = deferred[d];
        const int b = seg[i], e = seg[i + 1];
        float acc = segment_dot<64>(cols, vals, x, b, e, lane);
        acc = group_sum<64>(acc);
        if (lane == 0) emit(i, acc);
    }
}

// Lanes per row from the tile's mean segment length: the largest power of two G <= 64 with
// 16*G <= mean + 15.  Small teams keep the lanes of a gather on
// neighbouring rows, which is what makes the gathers of banded matrices coalesce.
template <bool MERGE, int WG, typename I, typename E>
__device__ __forceinline__ void tile_rows(const I* cols, const E* vals, const E* x, const int* seg, int nr, int r0,
                                          int tile_nnz, const RowOut& o, int* deferred, int* n_deferred,
                                          int tid) {
    const int nseg = nr + (MERGE ? 1 : 0);
    // With mean = floor(tile_nnz / nseg):  k < mean  <=>  (k + 1) * nseg <= tile_nnz  and
    // k > mean  <=>  k * nseg > tile_nnz, so the choice needs no division.
    int G = 1;
    while (G < 64 && nseg > 0 && (16 * G + 1) * nseg <= tile_nnz) G <<= 1;
    if (sizeof(I) == 2 && nseg > 0 && tile_nnz >= 64 * nseg) {
        // x comes out of LDS (16-bit window positions) and mean >= 64: long rows get about four
        // entries per lane.  Fewer rows then share a wavefront, and rows whose length is a multiple
        // of the 128-byte bank cycle would otherwise have all their teams on the same LDS banks.
        G = 64;
        while (4 * G * nseg > tile_nnz) G >>= 1;
    }
    if constexpr (std::is_same_v<I, NoGather> || std::is_same_v<I, GroupSums> || (std::is_same_v<I, AtSlot> && sizeof(E) == 4)) {
        // Rows of one length that is a multiple of four put the lanes of G = 1 on a few LDS banks (16 entries: four of 64): about
        // four entries per lane instead.  16 M groups in rows of 16: the reduce pass 27 -> 22 us; with rows of mixed lengths, whose
        // starts spread over the banks by themselves, more lanes per row cost 2 us on the 4 M-row power law.  x gathered in column order,
        // FP32, 100 000 rows of 16: 8.3 -> 6.7 us; 300 000 in bf16, where a lane reads half as far: 11.3 with one lane, 12.4 with four.
        const int len = __builtin_amdgcn_readfirstlane(nr > 0 ? seg[1] - seg[0] : 0);
        const int half = __builtin_amdgcn_readfirstlane(seg[nr >> 1] - seg[0]), all = __builtin_amdgcn_readfirstlane(seg[nr] - seg[0]);
        if (len >= 8 && (len & 3) == 0 && all == nr * len && half == (nr >> 1) * len) {
            G = 64;
            while (4 * G > len) G >>= 1;
        }
    }
    switch (G) {
        case 1: tile_rows_g<MERGE, WG, 1>(cols, vals, x, seg, nr, r0, o, deferred, n_deferred, tid); break;
        case 2: tile_rows_g<MERGE, WG, 2>(cols, vals, x, seg, nr, r0, o, deferred, n_deferred, tid); break;
        case 4: tile_rows_g<MERGE, WG, 4>(cols, vals, x, seg, nr, r0, o, deferred, n_deferred, tid); break;
        case 8: tile_rows_g<MERGE, WG, 8>(cols, vals, x, seg, nr, r0, o, deferred, n_deferred, tid); break;
        case 16: tile_rows_g<MERGE, WG, 16>(cols, vals, x, seg, nr, r0, o, deferred, n_deferred, tid); break;
        case 32: tile_rows_g<MERGE, WG, 32>(cols, vals, x, seg, nr, r0, o, deferred, n_deferred, tid); break;
        default: tile_rows_g<MERGE, WG, 64>(cols, vals, x, seg, nr, r0, o, deferred, n_deferred, tid); break;
    }
}

// After the row phase of a merge-path chunk (entered by the whole workgroup): hands over its first row's part, if that began
// in an earlier chunk, and the piece cut off at its end, if there is one.  One lane each, in different wavefronts.
__device__ __forceinline__ void finish_cuts(const RowOut& o, const CutOut& c, const int* seg, int nr, int r0, int part, int tid) {
    const bool tail_cut = seg[nr + 1] > seg[nr];
    if (c.carry_row) {
        __syncthreads();
        if (tid == 0) {
            c.carry_row[part] = tail_cut ? r0 + nr : -1;
            c.carry_val[part] = o.cut_sums[1];
        }
        return;
    }
    if (!o.head_cut && !tail_cut) return;
    __syncthreads();
    if (tid == 0 && o.head_cut) finish_cut(o, c, r0, part, true, o.cut_sums[0]);
    if (tid == 64 && tail_cut) finish_cut(o, c, r0 + nr, part, false, o.cut_sums[1]);
}

}  // namespace
}  // namespace spmv
