// Storage codecs of the distributions.
//
// FP64 and FP32 store values as they are.  FP16 and BF16 store shifted and
// scaled populations, (f - shift) * scale, rounded to nearest-even; loads
// invert that in FP32.  The shift removes the large part of a population that
// its reader can rebuild on its own (w_j times its own phi of the step before,
// for h); the scale (a power of two) lifts the small remainder out of the
// FP16 subnormal range.  BF16 rounding is to nearest-even and keeps NaNs quiet.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pulbm {

// Round to nearest-even, NaNs quiet: one instruction of this GPU
// (v_cvt_pk_bf16_f32), which gives the upper 16 bits that adding 0x7fff + bit 16
// gives, for every binary32 value.  Written out, with its branch for NaNs, it
// took six (128^3, 46 of them to a node: step 178 / 173 us).  The branch that is
// never taken ends the basic block where that one did: the compiler contracts a
// product and a sum into an FMA within a block only, and 2-byte storage carries
// the different rounding of the merged blocks into the results (167 us).
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    const uint16_t r = __builtin_bit_cast(uint16_t, (__bf16)f);
    int never;
    asm volatile("s_mov_b32 %0, 0" : "=s"(never));
    if (never) asm volatile("");
    return r;
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

#define PULBM_GLB __attribute__((address_space(1)))
#define PULBM_CST __attribute__((address_space(4)))

template <class S> struct Codec;

template <> struct Codec<double> {
    using CT = double;  // compute type
    static constexpr int BYTES = 8;
    __device__ static __forceinline__ double dec(double v, double, double) { return v; }
    __device__ static __forceinline__ double enc(double v, double, double) { return v; }
};

template <> struct Codec<float> {
    using CT = float;
    static constexpr int BYTES = 4;
    __device__ static __forceinline__ float dec(float v, float, float) { return v; }
    __device__ static __forceinline__ float enc(float v, float, float) { return v; }
};

template <> struct Codec<_Float16> {
    using CT = float;
    static constexpr int BYTES = 2;
    __device__ static __forceinline__ float dec(_Float16 v, float inv_scale, float shift)
    {
        return fmaf((float)v, inv_scale, shift);
    }
    __device__ static __forceinline__ _Float16 enc(float v, float scale, float shift)
    {
        return (_Float16)((v - shift) * scale);
    }
};

// BF16 storage: the upper 16 bits of a binary32, held in a uint16_t.
template <> struct Codec<uint16_t> {
    using CT = float;
    static constexpr int BYTES = 2;
    __device__ static __forceinline__ float dec(uint16_t v, float inv_scale, float shift)
    {
        return fmaf(bf16_to_f32(v), inv_scale, shift);
    }
    __device__ static __forceinline__ uint16_t enc(float v, float scale, float shift)
    {
        return f32_to_bf16_rne((v - shift) * scale);
    }
};

}  // namespace pulbm
