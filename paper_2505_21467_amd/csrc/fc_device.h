// Device-side helpers shared by the kernel files: storage-type conversion, pieces of tensors at any element, loads into LDS
// and the waits for them, quotients by a launch's constants.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

struct bf16_t {
    uint16_t bits;
};

__device__ __forceinline__ float fc_to_float(float v) { return v; }
__device__ __forceinline__ float fc_to_float(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }

// float -> bfloat16, round to nearest even (the hardware conversion of gfx950); NaN stays NaN.
__device__ __forceinline__ uint16_t fc_bf16_bits(float f)
{
    union { __bf16 h; uint16_t u; } x;
    x.h = (__bf16)f;
    return x.u;
}

// 16- and 8-byte pieces of a caller's tensor that need only be aligned to its elements (views may start anywhere): the
// compiler emits the same single loads and stores for them as for aligned pieces, the hardware takes any address.
struct __attribute__((packed, aligned(2))) fc_any16 {
    uint32_t w[4];
};
struct __attribute__((packed, aligned(2))) fc_any8 {
    uint32_t w[2];
};
template <typename V>
__device__ __forceinline__ V fc_load_any(const void *p)
{
    static_assert(sizeof(V) == 16, "16 bytes");
    return __builtin_bit_cast(V, *(const fc_any16 *)p);
}
template <typename V>
__device__ __forceinline__ void fc_store_any(void *p, V v)
{
    static_assert(sizeof(V) == 16 || sizeof(V) == 8, "16 or 8 bytes");
    if constexpr (sizeof(V) == 16) *(fc_any16 *)p = __builtin_bit_cast(fc_any16, v);
    else *(fc_any8 *)p = __builtin_bit_cast(fc_any8, v);
}

// Direct-to-LDS load: 16 bytes per lane, from a global address of each lane's own to the wave's `l` + 16 lane.
// ONCE: with the non-temporal hint, for bytes that one workgroup reads once and that no cache holds (fc_read_once): they pass
// the memory-side cache by and are the first to leave L2.
template <bool ONCE = false>
__device__ __forceinline__ void fc_load_lds16(const void *g, void *l)
{
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)g,
                                     (void __attribute__((address_space(3))) *)l, 16, 0, ONCE ? 2 : 0);
}
// f(true_type) or f(false_type): a wave-uniform choice of the hint around a group of loads.
template <typename F>
__device__ __forceinline__ void fc_with_hint(bool once, F f)
{
    if (once) f(std::true_type());
    else f(std::false_type());
}

// Wait until at most N of this wave's vector-memory operations are outstanding; LGKM0: and no LDS one.
template <int N, bool LGKM0 = false>
__device__ __forceinline__ void fc_wait_vm()
{
    // gfx9 s_waitcnt immediate: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((LGKM0 ? 0 : 15) << 8) | ((N >> 4) << 14));
}
// Until no LDS operation is outstanding (lgkmcnt(0)).
__device__ __forceinline__ void fc_wait_lds() { fc_wait_vm<63, true>(); }

// x / d, d given as 2^32 / d rounded up (0: d is 1); exact for x d < 2^32.
inline uint32_t fc_reciprocal(int64_t d) { return (uint32_t)((((int64_t)1 << 32) + d - 1) / d); }
__device__ __forceinline__ uint32_t fc_quotient(uint32_t x, uint32_t reciprocal) { return reciprocal ? __umulhi(x, reciprocal) : x; }

// x / d for any x and any d >= 1, without a branch: T. Granlund, P. Montgomery, Division by invariant integers using multiplication
// (1994), figure 4.1.  (As a plain division by an argument it is a chain of 35 instructions.)
struct FcDivisor {
    uint32_t mul, shift1, shift2;
    void set(uint32_t d)
    {
        const uint32_t l = d > 1 ? 32 - (uint32_t)__builtin_clz(d - 1) : 0;  // 2^l is the first power of two from d on
        const uint64_t more = ((uint64_t)1 << l) - d;
        mul = more ? (uint32_t)((more << 32) / d + 1) : 1;
        shift1 = l < 1 ? l : 1;
        shift2 = l - shift1;
    }
    __device__ __forceinline__ uint32_t over(uint32_t x) const
    {
        const uint32_t t = __umulhi(mul, x);
        return (t + ((x - t) >> shift1)) >> shift2;
    }
};

template <typename T>
__device__ __forceinline__ T fc_from_float(float f);
template <>
__device__ __forceinline__ float fc_from_float<float>(float f) { return f; }
template <>
__device__ __forceinline__ bf16_t fc_from_float<bf16_t>(float f)
{
    bf16_t r;
    r.bits = fc_bf16_bits(f);
    return r;
}
