// ea_bitops.hpp -- bit-sliced arithmetic and LDS access shared by the engines
// that hold spins as bits (ea_bits.hip: bits are sites; ea_groupbits.hpp: bits
// are walkers).
#pragma once

#include "ea_device.hpp"

namespace ea {

__device__ __forceinline__ uint32_t sel(uint32_t a, uint32_t b, uint32_t m) { return (a & ~m) | (b & m); }
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);  // truth table of the majority
}
// 2 F + (a < b): the comparison's carry goes straight into the add.
__device__ __forceinline__ uint32_t shift_in_less(uint32_t F, uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("v_cmp_lt_u32_e32 vcc, %1, %2\n\tv_addc_co_u32_e32 %0, vcc, %3, %3, vcc"
        : "=v"(r)
        : "v"(a), "v"(b), "v"(F)
        : "vcc");
    return r;
}

// Loads from an LDS byte address.
typedef __attribute__((address_space(3))) const uint32_t lds_u32;
typedef __attribute__((address_space(3))) const uint64_t lds_u64;
__device__ __forceinline__ uint32_t lds_load(uint32_t addr) { return *(lds_u32 *)(size_t)addr; }
__device__ __forceinline__ uint2 lds_load2(uint32_t addr)
{
    const uint64_t v = *(lds_u64 *)(size_t)addr;
    return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
__device__ __forceinline__ uint4 lds_load4(uint32_t addr)
{
    typedef uint32_t u32v4 __attribute__((ext_vector_type(4)));
    const u32v4 v = *(__attribute__((address_space(3))) const u32v4 *)(size_t)addr;
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(size_t)(__attribute__((address_space(3))) const char *)p;
}

// Spin bits of 32 int8 spins (bit b set iff byte b is -1) and back.
__device__ __forceinline__ uint32_t pack4(uint32_t v)
{
    return ((v >> 7) & 1u) | ((v >> 14) & 2u) | ((v >> 21) & 4u) | ((v >> 28) & 8u);
}
__device__ __forceinline__ uint32_t unpack4(uint32_t nib)
{
    return 0x01010101u + ((nib * 0x00204081u) & 0x01010101u) * 0xFEu;  // bytes 0x01 / 0xFF
}

}  // namespace ea
