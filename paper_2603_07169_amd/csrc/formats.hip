// gfx950 kernels for y <- alpha*A*x + beta*y with A in COO, CSC and ELL storage (paper App. C
// tasks 8, 10, 14).
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "kernels.h"

namespace spmv {
namespace {

constexpr int kEllTileSlots = 4096;  // most slots a workgroup of the ELL tile kernel stages
constexpr int kCscLdsRows = 16384;  // CSC: up to this many rows a workgroup keeps a private y in LDS (64 KB)

// ------------------------------------------------------------------------------------------
// y <- alpha*A*x + beta*y for A in the other storage layouts of the benchmark (App. C tasks 8,
// 10, 14).  ELL rows are independent and are reduced like CSR rows.  COO and CSC entries arrive
// grouped by nothing (COO) or by column (CSC), so their contributions are added to y with
// hardware float atomics after y has been scaled by beta in a kernel of its own; sums therefore
// depend on the order in which the atomics land (results agree to rounding, not bit for bit).
__global__ __launch_bounds__(kWG) void scale_y_kernel(float* __restrict__ y, int m, float beta) {
    for (int i = blockIdx.x * kWG + threadIdx.x; i < m; i += gridDim.x * kWG) y[i] = beta == 0.f ? 0.f : beta * y[i];
}

// Four consecutive entries per lane and trip.  A lane first sums the runs of equal row numbers
// among its own four; runs that lie wholly inside go to y with one hardware float atomic each.
// Its last run (its only one, if all four rows agree) may go on in the next lanes and its first may
// continue the previous lane's: those are joined across the wavefront with a segmented scan over
// the lanes' last-run sums, so a row held by consecutive entries (the whole row, for row-sorted
// input) costs one atomic per wavefront it touches instead of one per entry.
// shift: the arrays are read in aligned groups of four starting `shift` (0..3) entries before
// `row`; vec: those groups may be fetched with one 16-byte (8-byte for bf16 values) load each.
template <typename T>
__global__ __launch_bounds__(kWG) void spmv_coo_kernel(const int32_t* __restrict__ row, const int32_t* __restrict__ col,
                                                       const typename T::elem* __restrict__ vals,
                                                       const typename T::elem* __restrict__ x, float* y, int nnz,
                                                       int shift, int vec, float alpha) {
    using E = typename T::elem;
    const int lane = threadIdx.x & 63;
    const int64_t wave = (static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x) >> 6;
    const int64_t n_waves = (static_cast<int64_t>(gridDim.x) * kWG) >> 6;
    const int64_t n_groups = (static_cast<int64_t>(nnz) + shift + 3) / 4;
    for (int64_t gbase = wave * 64; gbase < n_groups; gbase += n_waves * 64) {  // the same trip count for all lanes of a wavefront
        const int64_t e0_64 = 4 * (gbase + lane) - shift;  // first of this lane's four entries; < 0 or >= nnz: none
        int r[4];
        float p[4];
        if (vec && e0_64 >= 0 && e0_64 + 3 < nnz) {
            const int e0 = static_cast<int>(e0_64);
            const i32x4 rv = __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(row + e0));
            const i32x4 cv = __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(col + e0));
            float v[4];
            if constexpr (sizeof(E) == 4) {
                const f32x4 vv = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(vals + e0));
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = vv[i];
            } else {
                typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
                const u32x2 vv = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(vals + e0));
                v[0] = __uint_as_float(vv[0] << 16);
                v[1] = __uint_as_float(vv[0] & 0xFFFF0000u);
                v[2] = __uint_as_float(vv[1] << 16);
                v[3] = __uint_as_float(vv[1] & 0xFFFF0000u);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                r[i] = rv[i];
                p[i] = alpha * (v[i] * widen(x[cv[i]]));
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t e = e0_64 + i;
                const bool live = e >= 0 && e < nnz;
                r[i] = live ? row[e] : -1;
                p[i] = live ? alpha * (widen(vals[e]) * widen(x[col[e]])) : 0.f;
            }
        }
        // runs inside the lane: the first is kept as the head, the last as the tail, others go out at once
        const int head_row = r[0];
        float head_sum = 0.f;
        bool single = true;  // no row change seen yet: the run in hand is still the first
        int tail_row = r[0];
        float tail_sum = p[0];
#pragma unroll
        for (int i = 1; i < 4; ++i) {
            if (r[i] != tail_row) {
                if (single) {
                    head_sum = tail_sum;
                    single = false;
                } else if (tail_row >= 0) {
                    unsafeAtomicAdd(y + tail_row, tail_sum);
                }
                tail_row = r[i];
                tail_sum = p[i];
            } else {
                tail_sum += p[i];
            }
        }
        // chains of last runs: a lane joins the chain of the lane before it when all its entries have that lane's last row
        const int prev_tail_row = __shfl_up(tail_row, 1, 64);
        const int next_head_row = __shfl_down(head_row, 1, 64);
        const bool follows = lane > 0 && head_row == prev_tail_row;
        float chain = tail_sum;
        bool head = !(single && follows);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const float cc = __shfl_up(chain, d, 64);
            const int hh = __shfl_up(static_cast<int>(head), d, 64);
            if (lane >= d && !head) {
                chain += cc;
                head = hh != 0;
            }
        }
        const float chain_before = __shfl_up(chain, 1, 64);
        if (!single && head_row >= 0) unsafeAtomicAdd(y + head_row, follows ? head_sum + chain_before : head_sum);
        if (tail_row >= 0 && (lane == 63 || next_head_row != tail_row)) unsafeAtomicAdd(y + tail_row, chain);
    }
}

// A team of G lanes per column: its entries all multiply the same x[j] and go to different rows.
template <typename T, int G>
__global__ __launch_bounds__(kWG) void spmv_csc_kernel(const int32_t* __restrict__ col_offsets,
                                                       const int32_t* __restrict__ row,
                                                       const typename T::elem* __restrict__ vals,
                                                       const typename T::elem* __restrict__ x, float* y, int n, float alpha) {
    const int64_t j64 = (static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x) / G;
    const int tl = threadIdx.x % G;
    if (j64 >= n) return;
    const int j = static_cast<int>(j64);
    const float xj = alpha * widen(x[j]);
    const int e1 = col_offsets[j + 1];
    for (int e = col_offsets[j] + tl; e < e1; e += G) unsafeAtomicAdd(y + row[e], widen(vals[e]) * xj);
}

// The same for matrices with few rows, where the atomics of thousands of columns would queue up
// on the same few addresses of y: a workgroup adds its columns into a private copy of y in LDS
// and sends every row's total to memory once.  Few workgroups, so few atomics per address.
// gridDim.y workgroups share a stretch of columns, each with its own stretch of the rows.
constexpr int kCscLdsWG = 512;      // lanes of a workgroup of spmv_csc_lds_kernel
constexpr int kCscLdsBlocks = 128;  // most workgroups it is launched with
template <typename T, int G>
__global__ __launch_bounds__(kCscLdsWG) void spmv_csc_lds_kernel(const int32_t* __restrict__ col_offsets,
                                                           const int32_t* __restrict__ row,
                                                           const typename T::elem* __restrict__ vals,
                                                           const typename T::elem* __restrict__ x, float* y, int m, int n,
                                                           float alpha) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float* ly = reinterpret_cast<float*>(smem_raw);  // [hi - lo]
    // blockIdx.y: the stretch of rows this workgroup adds up; entries of other rows are read and passed over
    const int lo = static_cast<int>(static_cast<int64_t>(m) * blockIdx.y / gridDim.y);
    const int hi = static_cast<int>(static_cast<int64_t>(m) * (blockIdx.y + 1) / gridDim.y);
    for (int i = threadIdx.x; i < hi - lo; i += kCscLdsWG) ly[i] = 0.f;
    __syncthreads();
    const int tl = threadIdx.x % G;
    for (int j = (blockIdx.x * kCscLdsWG + threadIdx.x) / G; j < n; j += gridDim.x * (kCscLdsWG / G)) {
        const float xj = alpha * widen(x[j]);
        const int e1 = col_offsets[j + 1];
        for (int e = col_offsets[j] + tl; e < e1; e += G) {
            const int r = row[e];
            if (r >= lo && r < hi) atomicAdd(ly + (r - lo), widen(vals[e]) * xj);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < hi - lo; i += kCscLdsWG) {
        const float v = ly[i];
        if (v != 0.f) unsafeAtomicAdd(y + lo + i, v);
    }
}

// A team of G lanes per row of `width` slots; a slot with col_id -1 is padding.
template <typename T, int G>
__global__ __launch_bounds__(kWG) void spmv_ell_kernel(const int32_t* __restrict__ col_ids,
                                                       const typename T::elem* __restrict__ vals,
                                                       const typename T::elem* __restrict__ x, float* y, int m, int width,
                                                       float alpha, float beta) {
    // m * G can pass 2^32 lanes: 64-bit lane number
    const int64_t i64 = (static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x) / G;
    const int tl = threadIdx.x % G;
    const bool live = i64 < m;
    const int i = static_cast<int>(i64);
    float acc = 0.f;
    if (live) {
        const size_t base = static_cast<size_t>(i) * width;
        for (int s = tl; s < width; s += G) {
            const int c = col_ids[base + s];
            if (c >= 0) acc += widen(vals[base + s]) * widen(x[c]);
        }
    }
    acc = group_sum<G>(acc);  // every lane of the wavefront takes part
    if (live && tl == 0) y[i] = epilogue(acc, alpha, beta, y, i);
}


// Four consecutive stored values from slot `at` on, out of LDS, in reads of whole words.
__device__ __forceinline__ f32x4 four_values(const float* vals, int at) {
    f32x4 v;
    __builtin_memcpy(&v, __builtin_assume_aligned(vals + at, 4), 16);
    return v;
}
__device__ __forceinline__ f32x4 four_values(const uint16_t* vals, int at) {
    uint32_t w[3];
    __builtin_memcpy(w, __builtin_assume_aligned(vals + (at & ~1), 4), 12);
    const unsigned shift = 16u * (at & 1);
    const uint32_t lo = __builtin_amdgcn_alignbit(w[1], w[0], shift), hi = __builtin_amdgcn_alignbit(w[2], w[1], shift);
    return f32x4{__uint_as_float(lo << 16), __uint_as_float(lo & 0xFFFF0000u), __uint_as_float(hi << 16), __uint_as_float(hi & 0xFFFF0000u)};
}

// The rows of a staged tile: a wavefront takes 64 / G rows at a time, and its k-th 64 / G lanes every G-th four slots of them from the
// k-th on, K fours in all, so that the lanes of a gather stand for neighbouring rows and, in a band or a stencil, read
// neighbouring x.  (Measured on x in the caches: 64 neighbouring values cost a compute unit 2.4 ns, 32 pairs of neighbours 15, 64 values
// far apart 27.)  All of a lane's gathers are in flight at once; slots past the row's end are treated as padding, whose value and x
// count for nothing, whatever they hold.
template <int G, int K, typename E>
__device__ __forceinline__ void ell_rows(const int* cols_l, int col_stride, const E* vals_l, int val_stride, const E* x, const float* y0_l, float* y,
                                         int nr, int r0, int width, float alpha, float beta, int tid) {
    constexpr int RPW = 64 / G;
    const int lane = tid & 63, part = lane / RPW;
    for (int first = 0; first < nr; first += kWG / G) {
        const int row = first + (tid >> 6) * RPW + lane % RPW;
        const int len = row < nr ? width - 4 * part : 0;
        const int col_at = row < nr ? row * col_stride + 4 * part : 0, val_at = row < nr ? row * val_stride + 4 * part : 0;
        int c[4 * K];
        E xv[4 * K];
#pragma unroll
        for (int q = 0; q < K; ++q) __builtin_memcpy(c + 4 * q, __builtin_assume_aligned(cols_l + col_at + 4 * G * q, 4), 16);
#pragma unroll
        for (int u = 0; u < 4 * K; ++u) {
            c[u] = 4 * G * (u / 4) + u % 4 < len ? c[u] : -1;
            xv[u] = x[static_cast<unsigned>(c[u] < 0 ? 0 : c[u])];
        }
        float acc[2] = {0.f, 0.f};
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const f32x4 v = four_values(vals_l, val_at + 4 * G * q);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u & 1] += (c[4 * q + u] < 0 ? 0.f : v[u]) * (c[4 * q + u] < 0 ? 0.f : widen(xv[4 * q + u]));
        }
        float sum = acc[0] + acc[1];
        if constexpr (G >= 4) sum = add_swap16(sum);
        if constexpr (G >= 2) sum = add_swap32(sum);
        if (row < nr && part == 0) y[r0 + row] = epilogue(sum, alpha, beta, y0_l, row);
    }
}

// ELL rows of moderate width: a workgroup copies the slots of a run of rows (a contiguous stretch of col_ids / vals, since the layout
// is row-major) to LDS as they are, past the registers, and then every lane takes a stretch of a row.  Against a team of lanes
// reading its row straight from memory this keeps the global reads fully coalesced whatever the width.
// Bound: memory (27 points of 128^3: bf16 53.4 us, 6.4 TB/s of the 6.9 a kernel that only reads reaches; FP32 72).  With the slots
// staged through registers and a row's gathers in batches of 8, 4, 2 and 1, each waited for, 67.2 and 96; the copies alone 66, a
// lane's gathers all at once the rest.  Tiles of 3072 or 2048 slots instead of 4096: 53.9, 61.
// rows_per_tile is a multiple of 8, so a tile's first slot is 16-byte aligned in both arrays.
template <typename T>
__global__ __launch_bounds__(kWG, 8) void spmv_ell_tile_kernel(const int32_t* __restrict__ col_ids,
                                                               const typename T::elem* __restrict__ vals,
                                                               const typename T::elem* __restrict__ x, float* y, int m,
                                                               int width, int rows_per_tile, float alpha, float beta,
                                                               int vec_ok) {
    using E = typename T::elem;
    constexpr int VEC = T::VEC;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tid = threadIdx.x;
    const int r0 = xcd_remap(blockIdx.x, gridDim.x) * rows_per_tile;  // a die works through a contiguous stretch of rows
    const int nr = m - r0 < rows_per_tile ? m - r0 : rows_per_tile;
    const size_t k0 = static_cast<size_t>(r0) * width;
    const int span = nr * width;
    // Rows of 32 or 64 slots would all begin on the same LDS banks: 16 bytes are left between them (100000 banded rows of 32, bf16:
    // 13.0 -> 5.6 us).
    const int pad = width % 32 == 0 ? 1 : 0;
    const int col_stride = width + 4 * pad, val_stride = width + VEC * pad;
    int* cols_l = reinterpret_cast<int*>(smem_raw);
    E* vals_l = reinterpret_cast<E*>(smem_raw + sizeof(int) * ((rows_per_tile * col_stride + VEC - 1) & ~(VEC - 1)));
    float* y0_l = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(vals_l) + sizeof(E) * ((rows_per_tile * val_stride + VEC - 1) & ~(VEC - 1)) +
                                           64 * sizeof(E) + 16);  // nr old values of y; a lane reads up to 64 slots past the tile's

    const float y0v = (beta != 0.f && tid < nr) ? y[r0 + tid] : 0.f;
    const int whole = vec_ok ? span & ~(VEC - 1) : 0;  // slots of the tile that whole vectors cover
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto copy = [&](const void* to, const void* from, int vecs, int per_row) {  // whole vectors of 16 bytes; per_row of them to a padded row
        const uint32_t lds = lds_address(to);
        if (!pad) {
            for (int v = 64 * wave; v < vecs; v += kWG)
                if (lane < vecs - v) copy16_to_lds_nt(lds + 16 * v, static_cast<const unsigned char*>(from) + 16 * v, 16u * static_cast<unsigned>(lane));
        } else {  // the gap behind a row is filled with its last vector again
            const int held = vecs + vecs / per_row, step = (1 << 20) / (per_row + 1) + 1;  // v * step >> 20 = v / (per_row + 1) while v < 2^12
            for (int v0 = 64 * wave; v0 < held; v0 += kWG) {
                const int v = v0 + lane, row = v * step >> 20, in_row = v - row * (per_row + 1);
                if (v < held)
                    copy16_to_lds_nt(lds + 16 * v0, from, 16u * static_cast<unsigned>(row * per_row + (in_row < per_row ? in_row : per_row - 1)));
            }
        }
    };
    copy(cols_l, col_ids + k0, whole / 4, width / 4);
    copy(vals_l, vals + k0, whole / VEC, width / VEC);
    for (int off = whole + tid; off < span; off += kWG) {  // what no whole vector covers (everything, if unaligned)
        const int row = pad ? off / width : 0;
        cols_l[off + 4 * pad * row] = col_ids[k0 + off];
        vals_l[off + VEC * pad * row] = vals[k0 + off];
    }
    if (tid < nr) y0_l[tid] = y0v;
    if (beta != 0.f)
        for (int i = tid + kWG; i < nr; i += kWG) y0_l[i] = y[r0 + i];
    wait_all_and_barrier();

#define ELL_ROWS(G, K) ell_rows<G, K>(cols_l, col_stride, vals_l, val_stride, x, y0_l, y, nr, r0, width, alpha, beta, tid)
    if (width <= 4) ELL_ROWS(1, 1);
    else if (width <= 8) ELL_ROWS(1, 2);
    else if (width <= 12) ELL_ROWS(1, 3);
    else if (width <= 16) ELL_ROWS(1, 4);
    else if (width <= 24) ELL_ROWS(2, 3);
    else if (width <= 32) ELL_ROWS(2, 4);
    else if (width <= 48) ELL_ROWS(4, 3);
    else ELL_ROWS(4, 4);
#undef ELL_ROWS
}

}  // namespace

namespace {

int lanes_for_length(int64_t len) {  // smallest power of two G in [2, 64] with 8*G >= len
    int G = 2;
    while (G < 64 && 8 * G < len) G <<= 1;
    return G;
}

template <typename T>
hipError_t launch_coo_t(int32_t m, int32_t nnz, const int32_t* row, const int32_t* col, const void* vals, const void* x,
                        float* y, Scalars s, hipStream_t st) {
    using E = typename T::elem;
    int grid = ceil_div(m, kWG);
    launch_kernel(scale_y_kernel, dim3(grid > 2048 ? 2048 : grid), dim3(kWG), 0, st, y, m, s.beta);
    if (nnz > 0) {
        // the caller's arrays start where they start: whole-vector loads only if all three are aligned as they are
        const bool vec = reinterpret_cast<uintptr_t>(row) % 16 == 0 && reinterpret_cast<uintptr_t>(col) % 16 == 0 &&
                         reinterpret_cast<uintptr_t>(vals) % (4 * sizeof(E)) == 0;
        // Up to 8192 workgroups (four rounds of those the device holds), beyond 16384 stretches of 1024 entries one for every two of
        // them: on 56 M row-sorted entries 127 / 123 / 120 / 118 / 117 / 125 us with 4096 / 8192 / 14000 / 18200 / 27300 / 54435.
        // Against 8192 throughout, FP32: the same up to 20 M entries, 67.4 -> 65.5 us at 24 M, 90 -> 84 at 32, 139 -> 128 at 48,
        // 187 -> 167 at 64 (bf16 146 -> 136).
        const int stretches = ceil_div(nnz, 4 * kWG);
        grid = stretches <= 8192 ? stretches : (stretches <= 16384 ? 8192 : (stretches + 1) / 2);
        launch_kernel((spmv_coo_kernel<T>), dim3(grid), dim3(kWG), 0, st, row, col,
                           static_cast<const E*>(vals), static_cast<const E*>(x), y, nnz, 0, vec ? 1 : 0, s.alpha);
    }
    return hipGetLastError();
}

template <typename T, int G>
hipError_t launch_csc_tg(int32_t m, int32_t n, int32_t nnz, const int32_t* col_offsets, const int32_t* row, const void* vals,
                         const void* x, float* y, Scalars s, hipStream_t st) {
    using E = typename T::elem;
    const int grid = ceil_div(m, kWG);
    launch_kernel(scale_y_kernel, dim3(grid > 2048 ? 2048 : grid), dim3(kWG), 0, st, y, m, s.beta);
    if (n <= 0) return hipGetLastError();
    const int blocks = ceil_div(static_cast<int64_t>(n) * G, kWG);
    if (m <= kCscLdsRows) {
        // A private y per workgroup.  A compute unit retires one LDS float atomic every 1.3 ns whatever the workgroup's
        // size (integer ones every 0.5 ns), so the time to add the entries falls with the number of workgroups, while each
        // workgroup sends one global atomic per row at the end: measured 57 / 31 / 18 / 13 / 15 us with 16 / 32 / 64 / 128 /
        // 256 workgroups on the benchmark's 2048 x 32768 shape (256, 512 or 1024 lanes each: the same).  Up to 2^20 entries
        // entries in columns of eight or more, a second workgroup per stretch of columns takes the other half of the rows:
        // both read every entry of the stretch, each adds half of them, and no row gets more atomics than before
        // (13 -> 10.5 us; with 1.3 entries per column the walk over the columns is what takes the time, and doubling it
        // costs 13.5 -> 15.4 us).
        const int lds_blocks = ceil_div(static_cast<int64_t>(n) * G, kCscLdsWG);
        const int col_blocks = lds_blocks > kCscLdsBlocks ? kCscLdsBlocks : lds_blocks;
        const int parts = (nnz <= (1 << 20) && nnz >= 8 * static_cast<int64_t>(n) && m >= 2) ? 2 : 1;
        launch_kernel((spmv_csc_lds_kernel<T, G>), dim3(col_blocks, parts), dim3(kCscLdsWG), sizeof(float) * (m / parts + 1), st,
                           col_offsets, row, static_cast<const E*>(vals), static_cast<const E*>(x), y, m, n, s.alpha);
    } else {
        launch_kernel((spmv_csc_kernel<T, G>), dim3(blocks), dim3(kWG), 0, st, col_offsets, row,
                           static_cast<const E*>(vals), static_cast<const E*>(x), y, n, s.alpha);
    }
    return hipGetLastError();
}

template <typename T, int G>
hipError_t launch_ell_tg(int32_t m, int32_t width, const int32_t* col_ids, const void* vals, const void* x, float* y,
                         Scalars s, hipStream_t st) {
    using E = typename T::elem;
    return launch_kernel((spmv_ell_kernel<T, G>), dim3(ceil_div(static_cast<int64_t>(m) * G, kWG)), dim3(kWG), 0, st,
                       col_ids, static_cast<const E*>(vals), static_cast<const E*>(x), y, m, width, s.alpha, s.beta);
}

}  // namespace

hipError_t launch_scale_y(float* y, int32_t m, float beta, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    const int grid = ceil_div(m, kWG);
    return launch_kernel(scale_y_kernel, dim3(grid > 2048 ? 2048 : grid), dim3(kWG), 0, st, y, m, beta);
}

hipError_t launch_coo_accumulate(bool bf16, int32_t nnz, const int32_t* row, const int32_t* col, const void* vals,
                                 const void* x, float* y, float alpha, hipStream_t st) {
    if (nnz <= 0) return hipSuccess;
    // The arrays are stretches of the library's own allocations, all three starting the same number of
    // entries into theirs: the (up to three) entries before `row` that complete its first aligned
    // group of four may be read, and are ignored.
    const int shift = static_cast<int>((reinterpret_cast<uintptr_t>(row) / 4) % 4);
    const size_t esz = bf16 ? 2 : 4;
    const bool vec = (reinterpret_cast<uintptr_t>(row) - 4 * shift) % 16 == 0 &&
                     (reinterpret_cast<uintptr_t>(col) - 4 * shift) % 16 == 0 &&
                     (reinterpret_cast<uintptr_t>(vals) - esz * shift) % (4 * esz) == 0;
    int grid = ceil_div(static_cast<int64_t>(nnz) + shift, 4 * kWG);
    if (grid > 8192) grid = 8192;
    if (bf16)
        launch_kernel((spmv_coo_kernel<BF16>), dim3(grid), dim3(kWG), 0, st, row, col, static_cast<const uint16_t*>(vals),
                           static_cast<const uint16_t*>(x), y, nnz, vec ? shift : 0, vec ? 1 : 0, alpha);
    else
        launch_kernel((spmv_coo_kernel<F32>), dim3(grid), dim3(kWG), 0, st, row, col, static_cast<const float*>(vals),
                           static_cast<const float*>(x), y, nnz, vec ? shift : 0, vec ? 1 : 0, alpha);
    return hipGetLastError();
}

hipError_t launch_coo(bool bf16, int32_t m, int32_t nnz, const int32_t* row, const int32_t* col, const void* vals,
                      const void* x, float* y, Scalars s, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    return bf16 ? launch_coo_t<BF16>(m, nnz, row, col, vals, x, y, s, st)
                : launch_coo_t<F32>(m, nnz, row, col, vals, x, y, s, st);
}

hipError_t launch_csc(bool bf16, int32_t m, int32_t n, int32_t nnz, const int32_t* col_offsets, const int32_t* row,
                      const void* vals, const void* x, float* y, Scalars s, hipStream_t st) {
    if (m <= 0) return hipSuccess;
#define SPMV_CSC_CASE(G) \
    case G: return bf16 ? launch_csc_tg<BF16, G>(m, n, nnz, col_offsets, row, vals, x, y, s, st) \
                        : launch_csc_tg<F32, G>(m, n, nnz, col_offsets, row, vals, x, y, s, st);
    switch (lanes_for_length(n > 0 ? (nnz + n - 1) / n : 0)) {
        SPMV_CSC_CASE(2) SPMV_CSC_CASE(4) SPMV_CSC_CASE(8) SPMV_CSC_CASE(16) SPMV_CSC_CASE(32) SPMV_CSC_CASE(64)
    }
#undef SPMV_CSC_CASE
    return hipErrorInvalidValue;
}

namespace {

constexpr int kEllTileMaxWidth = 64;  // widest rows that kernel is used for

template <typename T>
hipError_t launch_ell_tile(int32_t m, int32_t width, const int32_t* col_ids, const void* vals, const void* x, float* y,
                           Scalars s, hipStream_t st) {
    using E = typename T::elem;
    int rows = kEllTileSlots / width;
    rows = rows > kWG ? kWG : rows & ~7;
    // The row phase gives a row G lanes (1 up to 16 slots, 2 up to 32, 4 up to 64) and takes kWG / G rows a sweep.  A last sweep
    // that is less than three quarters full is left to the next tile: of the 144 rows of 27 slots that fit, 16 made a sweep
    // of their own (128^3 rows, FP32 / bf16: 77.2 / 63.6 -> 71.9 / 54.2 us with 128).  1 M banded rows, FP32 / bf16, with the rest and without: width
    // 20 28.4 / 22.1 -> 25.6 / 20.2 us, 40 48.7 / 40.8 -> 48.0 / 37.3, 48 59.0 / 47.4 -> 56.7 / 43.3, 56 72.7 / 58.4 -> 65.9 / 50.4, 60 70.2 / 54.2 -> 70.0 / 54.0; of
    // 420 shapes (60 k to 6 M slots, banded and scattered, widths 1 to 64) none took 3 % more, the best 22 % less.
    int G = 1;
    while (G < 64 && 16 * G < width) G <<= 1;
    const int sweep = kWG / G, rest = rows % sweep;
    if (rows > sweep && 4 * rest < 3 * sweep) rows -= rest;
    const bool vec_ok = reinterpret_cast<uintptr_t>(col_ids) % 16 == 0 && reinterpret_cast<uintptr_t>(vals) % 16 == 0;
    const int pad = width % 32 == 0 ? 1 : 0;
    const size_t lds = sizeof(int) * static_cast<size_t>(rows * (width + 4 * pad) + T::VEC) + sizeof(E) * static_cast<size_t>(rows * (width + T::VEC * pad) + T::VEC) +
                       64 * sizeof(E) + 16 + sizeof(float) * static_cast<size_t>(rows);
    return launch_kernel((spmv_ell_tile_kernel<T>), dim3(ceil_div(m, rows)), dim3(kWG), lds, st, col_ids,
                       static_cast<const E*>(vals), static_cast<const E*>(x), y, m, width, rows, s.alpha, s.beta,
                       vec_ok ? 1 : 0);
}

}  // namespace

hipError_t launch_ell(bool bf16, int32_t m, int32_t width, const int32_t* col_ids, const void* vals, const void* x,
                      float* y, Scalars s, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    // Rows of up to 64 slots go through LDS: read directly they would get teams of at most 8 lanes,
    // whose loads fall into many short pieces.  Wider rows get teams of 16 to 64 lanes, which read
    // 64 to 256 contiguous bytes at a time as it is.
    // Out of a graph, direct / through LDS: 27 wide, 128^3 points bf16 110.5 / 54.2 us, 1 M banded rows FP32 81.4 / 35.7, 200000 scattered ones 35.5 /
    // 26.7; 60 wide, 1 M banded FP32 152.5 / 70.0; 5 wide, 1.5 M banded FP32 19.9 / 13.6.  Where a launch is most of the time direct takes up to a quarter
    // less (30000 rows of 20 2.9 / 3.4, 937 of 64 3.2 / 3.4, 150000 of 4 2.7 / 3.1), which calls one by one do not show (4.1 us of host time each).
    // Rows of one or two slots are direct until memory is what counts: one slot, scattered, FP32 / bf16: 500000 rows 5.6 / 4.3 against 6.3 / 4.9,
    // 1 M 10.7 / 8.6 against 11.3 / 9.2, 4 M 58.9 / 43.5 against 59.2 / 43.2; two slots, 300000 rows 4.8 / 4.4 against 5.3 / 5.0, 500000 8.3 / 6.6 against 8.1 / 6.9.
    const bool narrow = (width == 1 && m <= 3 << 19) || (width == 2 && m <= 3 << 17);
    if (width >= 1 && width <= kEllTileMaxWidth && !narrow)
        return bf16 ? launch_ell_tile<BF16>(m, width, col_ids, vals, x, y, s, st)
                    : launch_ell_tile<F32>(m, width, col_ids, vals, x, y, s, st);
#define SPMV_ELL_CASE(G) \
    case G: return bf16 ? launch_ell_tg<BF16, G>(m, width, col_ids, vals, x, y, s, st) \
                        : launch_ell_tg<F32, G>(m, width, col_ids, vals, x, y, s, st);
    switch (lanes_for_length(width)) {
        SPMV_ELL_CASE(2) SPMV_ELL_CASE(4) SPMV_ELL_CASE(8) SPMV_ELL_CASE(16) SPMV_ELL_CASE(32) SPMV_ELL_CASE(64)
    }
#undef SPMV_ELL_CASE
    return hipErrorInvalidValue;
}

}  // namespace spmv
