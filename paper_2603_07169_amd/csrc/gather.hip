// gfx950 kernels for the row-wise product with x gathered in column order: MERGE and ADAPTIVE handles and, on groups of eight, WINDOWED ones, where
// analysis.h's gather_choice, gather_pays and gather_groups_choice say so from the entries, the row lengths and the lines of x that are touched.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "analysis.h"
#include "device_common.h"
#include "kernels.h"
#include "row_phase.h"

namespace spmv {
namespace {

constexpr int kGatherWG = 1024;        // lanes of a workgroup
constexpr int kGatherWords = 256;      // words of a group: a wavefront's load of 16 bytes a lane
constexpr int kGatherPosBits = 15;     // low bits of a word: the entry's place in its chunk; above them its column less the group's first
constexpr int kGatherDeferred = 512;   // rows far longer than the mean that a chunk can set aside (a chunk holds less than 2^15 entries)
constexpr int kGatherGroupWG = 512;    // lanes of a workgroup on groups of eight
constexpr int kGatherBuckets = 16384;  // column intervals the entries of a chunk are sorted by, at most

struct GatherArgs {
    const int32_t* chunk_desc;  // [2*(P+1)] first row and first entry of each chunk
    const uint32_t* words;      // [P * stride * 256]
    const int32_t* base;        // [P * stride] first column of each group
    const int32_t* rowptr;
    const void* vals;
    const void* x;
    float* y;
    const int32_t* cut_range;  // [2*(P+1)] (see finish_cut)
    CutScratch cut;
    int32_t stride;  // groups of words per chunk
    int32_t cap;     // slots of a chunk in LDS; padding words point at the one behind them
    int32_t nnz;
    int32_t vec_ok;  // vals is 16-byte aligned
    float alpha, beta;
};

// One workgroup per chunk of the merge path (MERGE; without cut rows for the ADAPTIVE plan), about as many chunks as compute units.
//   1. The chunk's values are copied to LDS as they lie in CSR, past the registers.  At the same time its columns are read in
//      ascending order, x is gathered in that order, and every value of x is put at its entry's place in CSR order.
//   2. The row phase of the tile kernels, with both operands in LDS.
// Bound: a gather of x out of a die's L2 brings a line of 128 bytes for 2 or 4 that are used, and the tile kernel asks for
// one line per entry (340 MB for 2.7 M entries, 17 TB/s).  In column order the entries that share a line stand in the same
// instruction, which asks for the line once; how often that happens grows with the entries a chunk holds, hence chunks as large
// as the LDS allows, one to a compute unit (power law 333 333 rows, FP32, 1 / 2 / 3 / 4 chunks to a compute unit: 14.3 / 15.9 / 17.3 /
// 17.7 us, the tile kernel 18.5; 300 000 rows of 16, bf16: 11.4 / 14.7 / 16.3 / 17.9, the tile kernel 22.8).
// A lane's four words are 64 places apart, so that an instruction's 64 gathers are neighbours in the order.  A word is four bytes as colidx
// is: the place, and the column less the first of 256 neighbours.  Chunks have a fixed stride in `words`, so that the words are
// asked for at once and not after the chunk's bounds have come.  Values are read where the caller keeps them.
// 512 lanes: the same up to 8000 entries a chunk, 10 to 20 % slower on 12000 and more.
// The pieces of rows that the chunk's ends cut are summed first, so that their way through memory (finish_cut: three round trips) runs
// beside the row phase: power law 333 333 rows 18.3 -> 16.6 us FP32, 14.8 -> 13.3 bf16.  Rows of more than 1024 entries in pieces for all
// wavefronts: 17.1 and 13.8.  (Timed call by call on three matrices in turn: tile kernel 20.2 and 18.6.)
template <typename T, bool MERGE, int U>
__global__ __launch_bounds__(kGatherWG) void spmv_gather_kernel(const GatherArgs a) {
    using E = typename T::elem;
    constexpr int VEC = T::VEC, WG = kGatherWG, WAVES = WG / 64;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ int deferred[kGatherDeferred];
    __shared__ int n_deferred;
    __shared__ float part_sums[kGatherWG / 64];  // of the pieces that the chunk's ends cut: its first row's in the first half, its last row's in the second
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int part = xcd_remap(blockIdx.x, gridDim.x);
    const E* const x = static_cast<const E*>(a.x);
    const u32x4* const words = reinterpret_cast<const u32x4*>(a.words) + static_cast<size_t>(part) * a.stride * 64;
    const int32_t* const base = a.base + static_cast<size_t>(part) * a.stride;

    u32x4 w[U];
    int first[U];
    auto ask = [&](int g0) {  // the wavefront's groups of one round; past the chunk's: the last again, whose words are then not used
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = g0 + wave + u * WAVES;
            const int held = g < a.stride ? g : a.stride - 1;
            w[u] = __builtin_nontemporal_load(words + held * 64 + lane);
            first[u] = base[held];
        }
    };
    ask(0);

    const int r0 = a.chunk_desc[2 * part];
    const int k0 = a.chunk_desc[2 * part + 1];
    const int nr = a.chunk_desc[2 * part + 2] - r0;
    const int k1 = a.chunk_desc[2 * part + 3];
    const int k0a = k0 & ~(VEC - 1);
    const int span = k1 - k0a;
    const int nseg = nr + (MERGE ? 1 : 0);
    const bool first_row_began = MERGE && a.rowptr[r0] < k0;  // in an earlier chunk
    E* const vals_l = reinterpret_cast<E*>(smem_raw);  // [cap]
    E* const x_l = vals_l + a.cap;                     // [cap + VEC]
    int* const seg = reinterpret_cast<int*>(x_l + a.cap + VEC);
    float* const y0_l = reinterpret_cast<float*>(seg + nseg + 1);

    const int rp0 = a.rowptr[r0 + (tid < nr ? tid : nr)];
    const float y0v = (a.beta != 0.f && tid < nr) ? a.y[r0 + tid] : 0.f;
    int whole = 0;  // vectors of vals that lie in the array as a whole
    if (a.vec_ok) {
        const int held = (span + VEC - 1) / VEC, there = (a.nnz - k0a) / VEC;
        whole = held < there ? held : there;
        const uint32_t to = lds_address(vals_l);
        const unsigned char* const from = static_cast<const unsigned char*>(a.vals) + sizeof(E) * static_cast<size_t>(k0a);
        for (int v = 64 * wave; v < whole; v += WG)
            if (lane < whole - v) copy16_to_lds_nt(to + 16 * v, from + 16 * static_cast<size_t>(v), 16u * static_cast<unsigned>(lane));
    }
    for (int i = whole * VEC + tid; i < span; i += WG)
        if (k0a + i >= k0) vals_l[i] = static_cast<const E*>(a.vals)[k0a + i];

    for (int g0 = 0;;) {
        E xv[U][4];
        unsigned at[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                xv[u][i] = x[static_cast<unsigned>(first[u]) + (w[u][i] >> kGatherPosBits)];
                at[u][i] = w[u][i] & ((1u << kGatherPosBits) - 1);
            }
        const int here = g0;
        g0 += U * WAVES;
        const bool more = g0 < a.stride;
        if (more) ask(g0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (here + wave + u * WAVES < a.stride) {
#pragma unroll
                for (int i = 0; i < 4; ++i) x_l[at[u][i]] = xv[u][i];
            }
        if (!more) break;
    }

    auto bound = [&](int v) {
        v = v < k0 ? k0 : v;
        v = v > k1 ? k1 : v;
        return v - k0a;
    };
    if (tid == 0) {
        n_deferred = 0;
        if (MERGE) seg[nseg] = k1 - k0a;
    }
    if (tid <= nr) seg[tid] = bound(rp0);
    if (tid < nr) y0_l[tid] = y0v;
    for (int i = tid + WG; i <= nr; i += WG) seg[i] = bound(a.rowptr[r0 + i]);
    if (a.beta != 0.f)
        for (int i = tid + WG; i < nr; i += WG) y0_l[i] = a.y[r0 + i];
    wait_all_and_barrier();

    int done = 0;  // rows taken before the row phase
    if constexpr (MERGE) {
        const bool head_cut = !a.cut.carry_row && nr > 0 && first_row_began;
        const bool tail_cut = seg[nr + 1] > seg[nr];
        if (head_cut || tail_cut) {
            float sum = 0.f;
            const bool tail = wave >= WAVES / 2;
            if (tail ? tail_cut : head_cut) {
                const int b = tail ? seg[nr] : seg[0], e = tail ? seg[nr + 1] : seg[1];
                sum = group_sum<64>(segment_dot<WG / 2>(static_cast<const AtSlot*>(nullptr), vals_l, x_l, b, e, tid % (WG / 2)));
            }
            if (lane == 0) part_sums[wave] = sum;
            __syncthreads();
            const RowOut o{a.y, y0_l, a.alpha, a.beta, nullptr, head_cut};
            const CutOut c{a.cut.carry_val, a.cut.arrivals, a.cut_range, nullptr, 0, a.cut.carry_row};
            auto sum_of = [&](int v0) {
                double s = 0;
                for (int v = v0; v < v0 + WAVES / 2; ++v) s += part_sums[v];
                return static_cast<float>(s);
            };
            // the last two wavefronts, which have no rows to spare for a last sweep
            if (tid == WG - 128 && head_cut) {
                finish_cut(o, c, r0, part, true, epilogue(sum_of(0), a.alpha, a.beta, y0_l, 0));
            }
            if (tid == WG - 64 && tail_cut) {
                const float s = sum_of(WAVES / 2);
                if (a.cut.carry_row) a.cut.carry_val[part] = s;
                else finish_cut(o, c, r0 + nr, part, false, s);
            }
            done = head_cut ? 1 : 0;
        }
        if (a.cut.carry_row && tid == WG - 64) a.cut.carry_row[part] = tail_cut ? r0 + nr : -1;
    }
    const RowOut o{a.y, y0_l + done, a.alpha, a.beta, nullptr, false};
    tile_rows<false, WG>(static_cast<const AtSlot*>(nullptr), vals_l, x_l, seg + done, nr - done, r0 + done, seg[nr] - seg[done], o, deferred, &n_deferred, tid);
}

// The same for a group-aligned matrix in bf16 (every row a whole number of groups of eight entries, every group an aligned run of eight
// columns; a WINDOWED handle), with groups in the place of entries: x is gathered, and kept in LDS, in runs of eight; a lane multiplies a group by
// its run with one 16-byte read of either, its values asked for before x is; the row phase adds up the groups' sums.
// Bound: the window kernel copies about every run of x anew for each block of 32 rows, in no order (address units 80 % busy).  Two
// chunks of half the LDS to a compute unit, so that one gathers while the other multiplies.  Windows / this, us out of a graph: 100 000 rows of
// 10 runs 10.4 / 7.9, 200 000 of 8 15.4 / 11.8, 200 000 of 16 25.9 / 19.2, 400 000 of 10 34.7 / 26.3, 500 000 of 16 57.9 / 46.2, 1 M of 5 42.9 / 37.0.  With
// 1024 lanes and all of the LDS 7.3, 10.9, 21.0, 29.7, 57.6, 41.3.  FP32, whose runs take twice the LDS: 200 000 of 16 42.4 / 41.6, 1 M of 5
// 65.8 / 80.3; it stays with the windows.
__global__ __launch_bounds__(kGatherGroupWG) void spmv_gather_group_kernel(const GatherArgs a) {
    constexpr int WG = kGatherGroupWG, WAVES = WG / 64, U = 2, PER_LANE = kGatherGroupSlots / WG;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ int deferred[kMaxDeferred];
    __shared__ int n_deferred;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int part = xcd_remap(blockIdx.x, gridDim.x);
    const u32x4* const x = static_cast<const u32x4*>(a.x);
    const u32x4* const words = reinterpret_cast<const u32x4*>(a.words) + static_cast<size_t>(part) * a.stride * 64;
    const int32_t* const base = a.base + static_cast<size_t>(part) * a.stride;

    u32x4 w[U];
    int first[U];
    auto ask = [&](int g0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = g0 + wave + u * WAVES;
            const int held = g < a.stride ? g : a.stride - 1;
            w[u] = __builtin_nontemporal_load(words + held * 64 + lane);
            first[u] = base[held];
        }
    };
    ask(0);
    const int r0 = a.chunk_desc[2 * part];
    const int k0 = a.chunk_desc[2 * part + 1];
    const int nr = a.chunk_desc[2 * part + 2] - r0;
    const int groups = a.chunk_desc[2 * part + 3] - k0;
    u32x4* const x_l = reinterpret_cast<u32x4*>(smem_raw);            // [cap + 1]
    float* const sums = reinterpret_cast<float*>(x_l + a.cap + 1);    // [cap]
    int* const seg = reinterpret_cast<int*>(sums + a.cap);            // [nr + 1]
    float* const y0_l = reinterpret_cast<float*>(seg + nr + 1);

    u32x4 v[PER_LANE];
#pragma unroll
    for (int u = 0; u < PER_LANE; ++u) {
        const int i = tid + u * WG;
        if (i < groups) v[u] = __builtin_nontemporal_load(static_cast<const u32x4*>(a.vals) + static_cast<size_t>(k0) + i);
    }
    for (int i = tid; i <= nr; i += WG) seg[i] = (a.rowptr[r0 + i] >> 3) - k0;
    if (tid == 0) n_deferred = 0;
    if (a.beta != 0.f)
        for (int i = tid; i < nr; i += WG) y0_l[i] = a.y[r0 + i];

    for (int g0 = 0;;) {
        u32x4 xv[U][4];
        unsigned at[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                xv[u][i] = x[static_cast<unsigned>(first[u]) + (w[u][i] >> kGatherPosBits)];
                at[u][i] = w[u][i] & ((1u << kGatherPosBits) - 1);
            }
        const int here = g0;
        g0 += U * WAVES;
        const bool more = g0 < a.stride;
        if (more) ask(g0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (here + wave + u * WAVES < a.stride) {
#pragma unroll
                for (int i = 0; i < 4; ++i) x_l[at[u][i]] = xv[u][i];
            }
        if (!more) break;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER_LANE; ++u) {
        const int i = tid + u * WG;
        if (i < groups) {
            const u32x4 xs = x_l[i];
            // Two chains of four products, exact in binary32 as they are: 2.1 roundings at the sum's full size for the eight, against 4.4 in one chain
            // and 3 in a tree of pairs.  With the row phase adding groups in 64 bits (GroupSums) rows of 4 / 6 / 10 / 16 groups are 2.4, 3.2, 3.6 and
            // 4.4e-8 off the 64-bit result, with the windows 2.7, 3.3, 4.0 and 4.6, with these chains and binary32 2.7, 3.4, 4.1, 4.6.
            float four[2];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                float acc = 0.f;
#pragma unroll
                for (int t = 2 * half; t < 2 * half + 2; ++t) {
                    acc = __builtin_fmaf(__uint_as_float(v[u][t] << 16), __uint_as_float(xs[t] << 16), acc);
                    acc = __builtin_fmaf(__uint_as_float(v[u][t] & 0xFFFF0000u), __uint_as_float(xs[t] & 0xFFFF0000u), acc);
                }
                four[half] = acc;
            }
            sums[i] = four[0] + four[1];
        }
    }
    __syncthreads();
    const RowOut o{a.y, y0_l, a.alpha, a.beta, nullptr, false};
    tile_rows<false, WG>(static_cast<const GroupSums*>(nullptr), sums, static_cast<const float*>(nullptr), seg, nr, r0, groups, o, deferred, &n_deferred, tid);
}

// Analysis: one workgroup per chunk sorts its entries by column interval (counts, prefix sums, places handed out with a counter per
// interval, all in LDS) and writes the chunk's words.  Inside an interval - at least a line of x - the order does not matter, to
// the gathers no more than to the result.  found[kGatherBad] is set where a column is out of range or too far from its group's first, or where
// eight entries that are to be one are not an aligned run of eight columns (colidx is 16-byte aligned then).  The rest of found is what
// gather_pays looks at: the intervals that chunks touch and, unless the entries are groups, those that stretches of 1024 entries touch.
__global__ __launch_bounds__(kGatherWG) void gather_build_kernel(const int32_t* __restrict__ colidx, const int32_t* __restrict__ chunk_desc,
                                                                 int n, int shift, int gs, int vec, int stride, int cap,
                                                                 uint32_t* __restrict__ words, int32_t* __restrict__ base, int32_t* found) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int WG = kGatherWG;
    int* const place = reinterpret_cast<int*>(smem_raw);  // [buckets]
    const int buckets = ((n - 1) >> shift) + 1;
    __shared__ int group_first[(1 << kGatherPosBits) / kGatherWords];
    __shared__ int wave_sums[WG / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = blockIdx.x;
    const int k0 = chunk_desc[2 * part + 1], k1 = chunk_desc[2 * part + 3];
    const int k0a = k0 & ~(vec - 1);
    const int entries = k1 - k0;
    bool bad = false;
    auto column = [&](int k) { return colidx[static_cast<size_t>(k) << gs] >> gs; };  // gs: 3 where the entries are groups of eight, else 0
    auto bucket_of = [&](int c) {
        if (c < 0 || c >= n) {
            bad = true;
            c = 0;
        }
        return c >> shift;
    };
    for (int i = tid; i < buckets; i += WG) place[i] = 0;
    __syncthreads();
    int stretch_lines = 0, lines = 0;
    if (gs == 0) {
        for (int s = 0; s * WG < entries; ++s) {
            const int k = k0 + s * WG + tid;
            if (k < k1 && atomicMax(place + bucket_of(column(k)), s + 1) <= s) ++stretch_lines;
            __syncthreads();
        }
        for (int i = tid; i < buckets; i += WG) place[i] = 0;
        __syncthreads();
    }
    for (int k = k0 + tid; k < k1; k += WG) atomicAdd(place + bucket_of(column(k)), 1);
    if (gs != 0)
        for (int k = k0 + tid; k < k1; k += WG) {
            const i32x4* const eight = reinterpret_cast<const i32x4*>(colidx) + 2 * static_cast<size_t>(k);
            const i32x4 lo = eight[0], hi = eight[1];
            bool run = (lo[0] & 7) == 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) run = run && lo[i] == lo[0] + i && hi[i] == lo[0] + 4 + i;
            bad = bad || !run;
        }
    __syncthreads();
    // exclusive prefix sums: a lane takes a run of buckets
    const int run = (buckets + WG - 1) / WG, b0 = tid * run, b1 = b0 + run < buckets ? b0 + run : buckets;
    int mine = 0;
    for (int b = b0; b < b1; ++b) {
        mine += place[b];
        lines += place[b] != 0;
    }
    int before = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(before, d);
        if (lane >= d) before += up;
    }
    if (lane == 63) wave_sums[wave] = before;
    __syncthreads();
    int at = before - mine;
    for (int v = 0; v < wave; ++v) at += wave_sums[v];
    for (int b = b0; b < b1; ++b) {
        const int count = place[b];
        place[b] = at;
        for (int g = (at + kGatherWords - 1) / kGatherWords; g * kGatherWords < at + count; ++g) group_first[g] = b << shift;
        at += count;
    }
    __syncthreads();
    for (int g = tid; g < stride; g += WG)
        base[static_cast<size_t>(part) * stride + g] = g * kGatherWords < entries ? group_first[g] : 0;
    uint32_t* const out = words + static_cast<size_t>(part) * stride * kGatherWords;
    auto put = [&](int i, uint32_t word) { out[(i & ~(kGatherWords - 1)) + 4 * (i & 63) + ((i >> 6) & 3)] = word; };
    for (int i = entries + tid; i < stride * kGatherWords; i += WG) put(i, static_cast<uint32_t>(cap));
    for (int k = k0 + tid; k < k1; k += WG) {
        const int c = column(k);
        const int i = atomicAdd(place + bucket_of(c), 1);
        const uint32_t off = static_cast<uint32_t>(c - group_first[i / kGatherWords]);
        if (off >= 1u << (32 - kGatherPosBits)) bad = true;
        put(i, off << kGatherPosBits | static_cast<uint32_t>(k - k0a));
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) found[kGatherBad] = 1;  // plain store: every writer writes 1
    // place is no longer needed
    __syncthreads();
    if (tid < 2) place[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        lines += __shfl_xor(lines, d);
        stretch_lines += __shfl_xor(stretch_lines, d);
    }
    if (lane == 0) {
        atomicAdd(place, lines);
        atomicAdd(place + 1, stretch_lines);
    }
    __syncthreads();
    if (tid == 0) {
        atomicMax(found + kGatherMostLines, place[0]);
        atomicAdd(found + kGatherLines, place[0]);
        atomicAdd(found + kGatherStretchLines, place[1]);
    }
}

template <typename T, bool MERGE, int U>
hipError_t launch_gather_u(const GatherArgs& a, int32_t P, size_t lds, hipStream_t st, hipEvent_t done) {
    const hipError_t e = allow_lds<spmv_gather_kernel<T, MERGE, U>>(lds);
    return e == hipSuccess ? launch_with_event(spmv_gather_kernel<T, MERGE, U>, dim3(P), dim3(kGatherWG), lds, st, done, a) : e;
}

template <typename T, bool MERGE>
hipError_t launch_gather_t(const GatherArgs& a, int32_t P, size_t lds, hipStream_t st, hipEvent_t done) {
    // groups a wavefront asks for at once: all of them up to four, beyond that as many rounds of equal size (92 groups, three at a time 21.0, four 21.9 us)
    constexpr int WAVES = kGatherWG / 64;
    const int rounds = (a.stride + 4 * WAVES - 1) / (4 * WAVES);
    switch ((a.stride + rounds * WAVES - 1) / (rounds * WAVES)) {
        case 1: return launch_gather_u<T, MERGE, 1>(a, P, lds, st, done);
        case 2: return launch_gather_u<T, MERGE, 2>(a, P, lds, st, done);
        case 3: return launch_gather_u<T, MERGE, 3>(a, P, lds, st, done);
        default: return launch_gather_u<T, MERGE, 4>(a, P, lds, st, done);
    }
}

}  // namespace

size_t gather_group_lds(int32_t groups, int32_t rows) {
    return 16 * (static_cast<size_t>(groups) + 1) + 4 * static_cast<size_t>(groups) + 4 * (2 * static_cast<size_t>(rows) + 1);
}

int32_t gather_slots(bool bf16, const int32_t* chunk_desc, int64_t P) {
    const int vec = bf16 ? BF16::VEC : F32::VEC;
    int32_t most = vec;
    for (int64_t p = 0; p < P; ++p) {
        const int32_t held = chunk_desc[2 * p + 3] - (chunk_desc[2 * p + 1] & ~(vec - 1));
        if (held > most) most = held;
    }
    return (most + vec - 1) & ~(vec - 1);
}

size_t gather_lds(bool bf16, int32_t slots, int32_t rows) {
    const size_t e = bf16 ? 2 : 4, vec = bf16 ? BF16::VEC : F32::VEC;
    return e * (2 * static_cast<size_t>(slots) + vec) + 4 * (2 * static_cast<size_t>(rows) + 2);
}

hipError_t launch_gather_build(const MatrixView& A, const GatherTiles& t, int32_t* found, hipStream_t st) {
    const int gs = t.group == 8 ? 3 : 0;
    const int n = t.group == 8 ? A.n / 8 : A.n;  // whole runs of eight: the kernel reads all of a run
    int shift = (A.bf16 ? 6 : 5) - gs;  // log2 of the columns (runs of columns) of a line of x
    while (((n - 1) >> shift) + 1 > kGatherBuckets) ++shift;
    const size_t lds = sizeof(int) * std::max<size_t>(((n - 1) >> shift) + 1, 2);
    const hipError_t e = allow_lds<gather_build_kernel>(lds);
    if (e != hipSuccess) return e;
    return launch_kernel(gather_build_kernel, dim3(t.num_chunks), dim3(kGatherWG), lds, st, A.colidx, t.chunk_desc, n, shift, gs,
                         t.group == 8 ? 1 : (A.bf16 ? BF16::VEC : F32::VEC), t.stride, t.slots, t.words, t.base, found);
}

hipError_t launch_gather(const GatherTiles& t, const MatrixView& A, const void* x, float* y, Scalars s, hipStream_t st, hipEvent_t done) {
    const GatherArgs a{t.chunk_desc, t.words, t.base, A.rowptr, A.vals, x, y, t.cut_range, t.cut, t.stride, t.slots, A.nnz, A.vec_ok ? 1 : 0, s.alpha, s.beta};
    if (t.group == 8) {
        const hipError_t e = allow_lds<spmv_gather_group_kernel>(t.lds);
        return e == hipSuccess ? launch_kernel(spmv_gather_group_kernel, dim3(t.num_chunks), dim3(kGatherGroupWG), t.lds, st, a) : e;
    }
    if (!t.cut_range) return A.bf16 ? launch_gather_t<BF16, false>(a, t.num_chunks, t.lds, st, done) : launch_gather_t<F32, false>(a, t.num_chunks, t.lds, st, done);
    hipEvent_t const last = t.cut.carry_row ? nullptr : done;
    const hipError_t e = A.bf16 ? launch_gather_t<BF16, true>(a, t.num_chunks, t.lds, st, last) : launch_gather_t<F32, true>(a, t.num_chunks, t.lds, st, last);
    return e == hipSuccess && t.cut.carry_row ? launch_cut_rows(t.cut, t.num_chunks, y, s.alpha, st, done) : e;
}

const char* gather_group_kernel_name() { return "spmv_gather_group_kernel"; }
const char* gather_kernel_name() { return "spmv_gather_kernel"; }

}  // namespace spmv
