// Device-side helpers shared by the kernel files: storage types, cross-lane sums, the alpha/beta
// epilogue.  Everything has internal linkage.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstdint>

#include "lds_grant.h"

namespace spmv {
namespace {

constexpr int kWG = 256;   // threads per workgroup = 4 wavefronts of 64
constexpr int kXcds = 8;   // accelerator dies; workgroup ids are dealt round-robin over them

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct F32 {
    using elem = float;
    static constexpr int VEC = 4;  // elements per 128-bit load of vals
};
struct BF16 {
    using elem = uint16_t;
    static constexpr int VEC = 8;
};

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// ------------------------------------------------------------------------------------------
// Cross-lane sums over aligned groups of G lanes; every lane of the group receives the total.
// Steps 1 and 2 permute inside a quad, 4 and 8 mirror a half row / a row of 16 (valid because
// the lanes being mirrored already agree), 16 swaps inside 32 lanes through the LDS crossbar
// (ds_swizzle, no memory touched), 32 swaps the two wave halves (v_permlane32_swap).
// All 64 lanes must be active.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float add_xor1(float v) { return v + dpp_move<0xB1>(v); }    // quad_perm [1,0,3,2]
__device__ __forceinline__ float add_xor2(float v) { return v + dpp_move<0x4E>(v); }    // quad_perm [2,3,0,1]
__device__ __forceinline__ float add_half_mirror(float v) { return v + dpp_move<0x141>(v); }
__device__ __forceinline__ float add_row_mirror(float v) { return v + dpp_move<0x140>(v); }
__device__ __forceinline__ float add_swap16(float v) {
    return v + __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));  // and 0x1f, xor 0x10
}
__device__ __forceinline__ float add_swap32(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int G>
__device__ __forceinline__ float group_sum(float v) {
    if constexpr (G >= 2) v = add_xor1(v);
    if constexpr (G >= 4) v = add_xor2(v);
    if constexpr (G >= 8) v = add_half_mirror(v);
    if constexpr (G >= 16) v = add_row_mirror(v);
    if constexpr (G >= 32) v = add_swap16(v);
    if constexpr (G >= 64) v = add_swap32(v);
    return v;
}

// Same with G known only at run time (uniform over the workgroup).
__device__ __forceinline__ float group_sum_rt(float v, int G) {
    if (G >= 2) v = add_xor1(v);
    if (G >= 4) v = add_xor2(v);
    if (G >= 8) v = add_half_mirror(v);
    if (G >= 16) v = add_row_mirror(v);
    if (G >= 32) v = add_swap16(v);
    if (G >= 64) v = add_swap32(v);
    return v;
}

__device__ __forceinline__ float epilogue(float acc, float alpha, float beta, const float* y, int r) {
    return beta == 0.f ? alpha * acc : alpha * acc + beta * y[r];
}

// Workgroup ids are handed to the 8 dies round-robin (id % 8).  Each die has its own L2, so
// give die j one contiguous run of logical tiles: its x window then lives in one L2.
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    const int q = nb / kXcds, r = nb % kXcds;
    const int die = bid % kXcds, slot = bid / kXcds;
    return die * q + (die < r ? die : r) + slot;
}

// Copies straight from memory to LDS, past the registers: lane l of the wavefront fetches 16 (4) bytes and they land 16 l (4 l)
// bytes behind `lds`, a byte address that is the same in all lanes.  Lanes that are switched off copy nothing.  The compiler
// does not know these loads: wait_all_and_barrier() waits for all that this wavefront has asked for and for the other wavefronts.
// The compiler does not look into the text either, so the wait states stand in it: one between the move and a copy that reads m0, five
// between a vector instruction that writes a base's scalar registers (none does as the kernels are compiled) and the copy that reads
// them (the move and s_nop 3: 27 points 128^3, bf16 as ELL 53.2 -> 53.5 us, the pattern kernel the same).
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void*)p));
}
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // m0 is reserved and clobbered: the compiler must not keep a value of its own in it across a copy
__device__ __forceinline__ void copy16_to_lds_nt(uint32_t lds, const void* base, uint32_t lane_offset) {  // base the same in all lanes
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(lane_offset), "s"(base) : "m0", "memory");
}
__device__ __forceinline__ void copy16_to_lds(uint32_t lds, const void* src) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "m0", "memory");
}
__device__ __forceinline__ void copy4_to_lds(uint32_t lds, const void* base, uint32_t lane_offset) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(lane_offset), "s"(base) : "m0", "memory");
}
#pragma clang diagnostic pop
// All memory accesses of this wavefront have ended, and all wavefronts of the workgroup have come here.
__device__ __forceinline__ void wait_all_and_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Launches a kernel.  The <<<>>> form hands its configuration to the runtime in a call of its own and fetches it back in another before it
// makes this one: 2.4 us of host time a launch against 2.1, and the error asked for afterwards 0.1 more.
template <typename... P, typename... Q>
hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t st, const Q&... values) {
    return [&](P... p) {
        void* args[] = {const_cast<void*>(static_cast<const void*>(&p))...};
        return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, args, lds, st);
    }(values...);
}

// Lets KERNEL be launched with `lds` bytes of dynamic LDS on the current device.
template <auto KERNEL>
hipError_t allow_lds(size_t lds) {
    static LdsGrant grant;
    return grant(reinterpret_cast<const void*>(KERNEL), lds);
}

// Launches a kernel; done, if not null, is recorded at its end by the dispatch itself.  An event recorded behind the kernel is a
// packet of its own: 2.9 us a run.  In the dispatch, with a device-scope release, it costs nothing on the merge plan (20.4 us
// on 2.7 M power-law entries with or without any fence) and 1.2 us on the two passes (122.7 -> 123.9 us on 32 M entries).
template <typename Args>
hipError_t launch_with_event(void (*kernel)(const Args), dim3 grid, dim3 block, size_t lds, hipStream_t st, hipEvent_t done, const Args& a) {
    if (!done) return launch_kernel(kernel, grid, block, lds, st, a);
    void* args[] = {const_cast<Args*>(&a)};
    return hipExtLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, args, lds, st, nullptr, done, 0);
}

inline int ceil_div(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

}  // namespace
}  // namespace spmv
