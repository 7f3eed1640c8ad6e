// Wave-level pieces shared by the kernels that keep whole tiles on chip (fused_fwd.hip,
// fused_bwd.hip, proj_bwd.hip, ffn.hip): operand types of v_mfma_f32_32x32x16_bf16,
// LDS barrier, buffer resources, transposing LDS reads and exchanges between lane rows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace recblr {
namespace wtile {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s4 lds_s4;

// Workgroup barrier for LDS hand-offs that leaves vector-memory operations in
// flight: __syncthreads() carries a release fence, which waits for every
// outstanding load and store of the wave (a direct-to-LDS prefetch of the
// next tile among them).  Here the wave's own LDS writes are waited for
// (lgkmcnt(0)), and direct-to-LDS loads are waited for explicitly (vmcnt)
// before the barrier that publishes their data; the empty asm statements keep
// the compiler from moving memory accesses across the barrier.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt not waited for
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                             0x00020000);
}

// The lane index, recomputed where it is used: LDS addresses derived from it
// are formed again in each tile (a few vector instructions) instead of being
// kept in registers across the whole loop.
__device__ __forceinline__ int fresh(int lane) {
    asm volatile("" : "+v"(lane));
    return lane;
}

// 8 consecutive-k values of an MFMA operand whose k runs across LDS rows:
// a transposing read hands lane i of each 16-lane block column i of a 4-row x
// 16-column block whose row j the lanes 4 j .. 4 j + 3 address.
__device__ __forceinline__ b8 tr_pair(const char* p0, const char* p1) {
    const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p0);
    const s4 c = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p1);
    return __builtin_bit_cast(b8, __builtin_shufflevector(a, c, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ __forceinline__ f16v mfma(b8 a, b8 b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// One product term set: acc += a b with the planes (hi, lo) each operand has.
template <int PA, int PB>
__device__ __forceinline__ f16v mma(const b8 (&a)[PA], const b8 (&b)[PB], f16v acc) {
    if constexpr (PB == 2) acc = mfma(a[0], b[1], acc);
    if constexpr (PA == 2) acc = mfma(a[1], b[0], acc);
    return mfma(a[0], b[0], acc);
}

// A-operand row of MFMA row R (0..31) in a 32-step block: rows are permuted
// so that lane half h of the 32 x 32 accumulator holds steps 16 h .. 16 h + 15
// in VGPRs 0 .. 15 (the accumulator of row 8 (v / 4) + 4 h + v % 4 is VGPR v).
__device__ __forceinline__ int sigma(int R) { return 16 * ((R >> 2) & 1) + 4 * (R >> 3) + (R & 3); }

// v_permlane16_swap: the odd 16-lane rows of a and the even ones of b trade places.
__device__ __forceinline__ void swap16(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
// The value of the lane in the neighbouring 16-lane row (rows 0 <-> 1, 2 <-> 3).
__device__ __forceinline__ float row_partner(float v, bool odd) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
    return __uint_as_float(odd ? r[0] : r[1]);
}
// The value of the lane 32 away (lower half <-> upper half).
__device__ __forceinline__ float half_partner(float v, bool upper) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
    return __uint_as_float(upper ? r[0] : r[1]);
}

}  // namespace wtile
}  // namespace recblr
