// What the weight-streaming kernels share (gfx950): vector types, bf16 rounding, and a run of a weight stream as a buffer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moespeq {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ inline uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// A run of a weight stream as a buffer: `bytes` bytes from `base` (both wave-uniform).  A load past the run's
// end returns zeros and moves nothing, so a window's loads need no clamps: positions are 32-bit offsets, four
// tiles of 1 KiB under one address register.  (As global loads with clamped 64-bit addresses a tile cost a
// dozen scalar instructions and a branch, and the first window of a workgroup took 5 us to issue.)
typedef __amdgpu_buffer_rsrc_t run_t;
__device__ inline run_t make_run(const char *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00027000);
}
constexpr int kNonTemporal = 2;
__device__ inline u32x4 run_load16(run_t r, uint32_t off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kNonTemporal));
}
__device__ inline uint32_t run_load4(run_t r, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kNonTemporal); }
__device__ inline uint32_t run_load2(run_t r, uint32_t off) { return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, kNonTemporal); }

}  // namespace

}  // namespace moespeq
