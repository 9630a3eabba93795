// Staging of packed weights as MFMA operands, shared by the GEMM kernels (gwq_gemm.hip, gwq_gemm_frag.hip).
#pragma once
#include "gwq_dequant.h"
#include "gwq_internal.h"

namespace gwq {

template <int BITS> struct SlotRegs;
template <> struct SlotRegs<4> { uint32_t w[4]; };
template <> struct SlotRegs<3> { uint32_t w[3], fourth; };    // fourth: the word after the slot's three (slot 3: the tail word)

template <int BITS> __device__ inline void load_slot(SlotRegs<BITS> &r, const uint32_t *group, int slot);
template <> __device__ inline void load_slot<4>(SlotRegs<4> &r, const uint32_t *group, int slot)
{
    const uint4 v = *reinterpret_cast<const uint4 *>(group + 4 * slot);
    r.w[0] = v.x; r.w[1] = v.y; r.w[2] = v.z; r.w[3] = v.w;
}
template <> __device__ inline void load_slot<3>(SlotRegs<3> &r, const uint32_t *group, int slot)
{
    // one 16-byte load at 4-byte alignment; it stays inside the group's 13 words for every slot
    const U128a4 v = *reinterpret_cast<const U128a4 *>(group + 3 * slot);
    r.w[0] = v.x; r.w[1] = v.y; r.w[2] = v.z; r.fourth = v.w;
}

// A 16-bit load that is complete when it returns, invisible to the compiler's bookkeeping of
// outstanding loads: for the rare path inside the staging loop, whose loads would otherwise make
// the compiler wait for every prefetch in flight at each trip of the loop.
__device__ inline uint32_t load_u16_now(const uint16_t *p)
{
    uint32_t v;
    asm volatile("global_load_ushort %0, %1, off\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p) : "memory");
    return v;
}

// A load of 8 bytes at 2-byte alignment (gfx950 global memory takes unaligned addresses).
struct __attribute__((packed, aligned(2))) U64a2 { uint32_t lo, hi; };

// Fragment j (8 codes -> 8 FP16 values s*(q - z)) of a slot.
__device__ inline u32x4 dequant_frag(const SlotRegs<4> &r, int j, uint32_t z, uint32_t s2, const DecodeConsts &d)
{
    const ZeroConsts<4> c(z);
    u32x4 f = decode_word4(r.w[j], c, d);
    f.x = pk_mul(f.x, s2); f.y = pk_mul(f.y, s2); f.z = pk_mul(f.z, s2); f.w = pk_mul(f.w, s2);
    return f;
}
__device__ inline void dequant_all(const SlotRegs<3> &r, uint32_t tail_pair, uint32_t z, uint32_t s2, const DecodeConsts &d,
                                   u32x4 f[4])
{
    decode_slot3(r.w, tail_pair, z, d, f);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[j].x = pk_mul(f[j].x, s2); f[j].y = pk_mul(f[j].y, s2);
        f[j].z = pk_mul(f[j].z, s2); f[j].w = pk_mul(f[j].w, s2);
    }
}

// bfloat16 operands: the eight exact FP16 integers q - z of a fragment times the scale in FP32, rounded once to
// bfloat16 (round to nearest even).
__device__ inline uint32_t scale_pair_bf16(uint32_t h2, float s)
{
    typedef float float2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const half2v h = __builtin_bit_cast(half2v, h2);
    // x * s as a fused multiply-add with -0: one v_fma_mix_f32, which widens its FP16 operand itself
    const float2v p = {__builtin_fmaf((float)h.x, s, -0.0f), __builtin_fmaf((float)h.y, s, -0.0f)};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(p, bf16x2));
}
__device__ inline u32x4 scale_frag_bf16(u32x4 f, float s)
{
    return u32x4{scale_pair_bf16(f.x, s), scale_pair_bf16(f.y, s), scale_pair_bf16(f.z, s), scale_pair_bf16(f.w, s)};
}
// An FP16 bit pattern as the nearest bfloat16's (the stored outliers, for bfloat16 MFMA operands).
__device__ inline uint16_t half_bits_to_bf16_bits(uint32_t h)
{
    return __builtin_bit_cast(uint16_t, (__bf16)(float)__builtin_bit_cast(_Float16, (uint16_t)h));
}

}  // namespace gwq
