// Small device helpers shared by the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace pk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// fp32 -> bf16 bits, round to nearest even: one v_cvt_pk_bf16_f32 per pair.  (Rounding by hand, an add
// and a shift on the bit patterns, takes ten vector instructions per pair.)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{lo, hi}, bf16x2));
}

__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
    return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
    return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// 16 bytes to memory through the L2, not left in it: the end of a launch waits for nothing that is still there, and beside work that
// streams at the rate of the memory a line evicted later, alone, costs it many times its own time (64 workgroups' 4.4 MB beside 1.15 GB of reads: 13 us).
// For stores of whole lines only: a line put together from several instructions goes to memory once for each.
constexpr int kWriteThrough = 16;                  // cache policy of a buffer store
// The same at an address of each lane's own; no builtin makes such a store of 16 bytes.  The compiler does not know what the statement reads: two wait states keep
// the instruction behind it from writing the data registers too early, and data must not come straight from an MFMA.
__device__ __forceinline__ void write_through(void* p, const u32x4& x) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(x) : "memory");
}

}  // namespace pk
