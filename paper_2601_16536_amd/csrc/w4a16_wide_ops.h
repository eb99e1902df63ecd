// Pieces of the kernels that give a wave 64 or more rows of X (w4a16_panel.hip, w4a16_tile_tall.hip): the exact operand
// q - z in the order of k, and compile-time loops.
#pragma once
#include "w4a16_device.h"
#include <type_traits>
#include <utility>

namespace w4a16 {

typedef float float16_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

// FP16: the B operand is (q - z) 2^-9, exact.  Byte e of a packed word holds the codes of k = 2e (bits 0-3) and 2e + 1
// (bits 4-7).  v_perm_b32 puts the first, masked, into the low half and the second, masked, into the high half of a
// register, where they are the FP16 subnormals q 2^-24 and q 2^-20; one packed FMA by (2^15, 2^11) gives (q - z) 2^-9.
struct ExactF16 {
    typedef ActF16 Act;
    typedef uint32_t Zero;  // (-z 2^-9) in both halves
    struct Consts {
        uint32_t lo, hi, mul;
    };
    static __device__ __forceinline__ Consts consts()
    {
        Consts c = {0x0F0F0F0Fu, 0xF0F0F0F0u, 0x68007800u};  // 2^11 | 2^15
        asm volatile("" : "+s"(c.lo), "+s"(c.hi), "+s"(c.mul));
        return c;
    }
    static __device__ __forceinline__ Zero zero(uint32_t z)  // z in bits 0-3
    {
        H2 h, m;
        h.u = (z & 15u) * 0x00010001u;
        m.u = 0xF800F800u;  // -2^15
        h.h = h.h * m.h;
        return h.u;
    }
    static __device__ __forceinline__ float scale(_Float16 s) { return (float)s * 512.0f; }
    // The unpack of one word in kParts parts of about five instructions.
    static constexpr int kParts = 2;
    struct Tmp {
        uint32_t a, b;
    };
    static __device__ __forceinline__ uint32_t pair(const Tmp &t, uint32_t nz, const Consts &c, int e)
    {
        H2 v, m, z;
        // selectors 0-3 pick from the second operand, 4-7 from the first, 0x0c gives zero
        v.u = __builtin_amdgcn_perm(t.b, t.a, 0x0C040C00u + 0x00010001u * (uint32_t)e);
        m.u = c.mul;
        z.u = nz;
        v.h = __builtin_elementwise_fma(v.h, m.h, z.h);
        return v.u;
    }
    static __device__ __forceinline__ void unpack(int part, uint32_t w, Zero nz, const Consts &c, Tmp &t, uint4_t &r)
    {
        if (part == 0) {
            t.a = w & c.lo;
            t.b = w & c.hi;
            r[0] = pair(t, nz, c, 0);
        } else {
            r[1] = pair(t, nz, c, 1);
            r[2] = pair(t, nz, c, 2);
            r[3] = pair(t, nz, c, 3);
        }
    }
    static __device__ __forceinline__ float16_t mfma(uint4_t x, uint4_t b, float16_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, x), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
    }
};

// BF16: the operand is q - z, exact, through FP32: a nibble masked in place is an FP16 subnormal, which the mixed FMA
// reads as it is; the FP32 results are whole numbers below 16, so their upper halves are the bfloat16.
struct ExactBF16 {
    typedef ActBF16 Act;
    typedef float Zero;  // -z
    struct Consts {
        uint32_t lo, hi;
    };
    static __device__ __forceinline__ Consts consts()
    {
        Consts c = {0x000F000Fu, 0x00F000F0u};
        asm volatile("" : "+s"(c.lo), "+s"(c.hi));
        return c;
    }
    static __device__ __forceinline__ Zero zero(uint32_t z) { return -(float)(z & 15u); }
    static __device__ __forceinline__ float scale(_Float16 s) { return (float)s; }
    static constexpr int kParts = 3;
    struct Tmp {
        H2 p[4];
        float d[8];
    };
    static __device__ __forceinline__ void code(Tmp &t, Zero nz, int i)
    {
        const float m = i & 1 ? 1048576.0f : 16777216.0f;
        t.d[i] = __builtin_fmaf((float)t.p[i & 3].h[i >> 2], m, nz);
    }
    static __device__ __forceinline__ void unpack(int part, uint32_t w, Zero nz, const Consts &c, Tmp &t, uint4_t &r)
    {
        if (part == 0) {
            const uint32_t w8 = w >> 8;
            t.p[0].u = w & c.lo;   // codes 0, 4
            t.p[1].u = w & c.hi;   // 1, 5
            t.p[2].u = w8 & c.lo;  // 2, 6
            t.p[3].u = w8 & c.hi;  // 3, 7
            code(t, nz, 0);
        } else if (part == 1) {
#pragma unroll
            for (int i = 1; i < 7; ++i) code(t, nz, i);
        } else {
            code(t, nz, 7);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                r[e] = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, t.d[2 * e + 1]), __builtin_bit_cast(uint32_t, t.d[2 * e]), 0x07060302u);
        }
    }
    static __device__ __forceinline__ float16_t mfma(uint4_t x, uint4_t b, float16_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bfloat8_t, x), __builtin_bit_cast(bfloat8_t, b), c, 0, 0, 0);
    }
};

// f(0), f(1), ... f(N - 1) with the numbers as constants.
template <int... I, typename F>
__device__ __forceinline__ void for_each_constant(std::integer_sequence<int, I...>, const F &f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
// f(0) && f(1) && ... && f(N - 1)
template <int... I, typename F>
__device__ __forceinline__ bool all_constants(std::integer_sequence<int, I...>, const F &f)
{
    return (f(std::integral_constant<int, I>{}) && ...);
}
// f(BEG), ... f(END - 1)
template <int BEG, int END, typename F>
__device__ __forceinline__ void static_range(const F &f)
{
    if constexpr (BEG < END) {
        f(std::integral_constant<int, BEG>{});
        static_range<BEG + 1, END>(f);
    }
}

}  // namespace w4a16
