// Pieces of the kernels whose B operand is q - z itself: the exact operand in the order of k (w4a16_panel.hip, w4a16_tile_tall.hip, w4a16_pair.hip,
// and FP16's in w4a16_tile_wide.hip), the compile-time loops of the first three, and what the stages (128 k) of PANEL and the tall form have in common.
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

// ---- a stage of kStage k: scales and zero points per segment of SEG k, and the slots ----

constexpr int kStage = 128;
constexpr int kSteps = kStage / 16;  // MFMAs 32x32x16 of one result tile

// Eq. 2's constants of a stage for a lane's two columns, from a word of two scales and one of zero points (shifted so that
// the two are in its low byte) per segment.
template <typename Op, int SEGS>
struct StageScales {
    float s[2][SEGS];
    typename Op::Zero z[2][SEGS];
    __device__ __forceinline__ void set(int e, uint32_t scales, uint32_t zeros)
    {
        H2 h;
        h.u = scales;
        s[0][e] = Op::scale(h.h[0]);
        s[1][e] = Op::scale(h.h[1]);
        z[0][e] = Op::zero(zeros);
        z[1][e] = Op::zero(zeros >> 4);
    }
};

// One slot of a stage: an MFMA of tile t = (column half, row block) and what fits beside it.  The tiles take their eight MFMAs one
// after the other.
template <int SLOT, int RT, int SEG>
struct StageSlot {
    static constexpr int kTiles = 2 * RT, kSegs = kStage / SEG, kStepsPerSeg = SEG / 16;
    static constexpr int t = SLOT / kSteps, ct = t / RT, rt = t % RT, ks = SLOT % kSteps;
    static constexpr int seg = ks / kStepsPerSeg, pp = (t * kSegs + seg) & 1;  // segment, and which part sums it adds to
    static constexpr bool kFirst = ks % kStepsPerSeg == 0;                      // of its segment
    // Eq. 2's step of the segment before (the tile before, for one segment per stage), once its last MFMA is through: beside
    // the fourth to sixth MFMA, or the second half of a shorter segment.
    static constexpr bool kOne = kSegs == 1;
    static constexpr int kLate = kOne ? 3 : kStepsPerSeg / 2, kStepSlots = kOne ? 3 : kStepsPerSeg / 2;
    static constexpr int es = ks % kStepsPerSeg - kLate;
    static constexpr bool kStepping = es >= 0 && es < kStepSlots;
    static constexpr int tp = seg ? t : (t + kTiles - 1) % kTiles;
    // this tile's share of the words to be unpacked, in slots that take no step where there is one segment
    static constexpr int w_beg = rt * kSteps / RT, w_end = (rt + 1) * kSteps / RT;
    static constexpr bool kUnpacking = !kOne || !kStepping;
    static constexpr int kUnpackSlots = kOne ? kSteps - kStepSlots : kSteps, kUnpackSlot = kOne && ks > kLate ? ks - kStepSlots : ks;
};

// The slot's vector work.  `word(w)`: the packed word of step w of the half that is unpacked, the second of this stage beside the
// first one's MFMAs, the first of the next stage beside the second one's.
template <typename Op, typename Slot, typename Scales, typename Word, int TILES>
__device__ __forceinline__ void step_and_unpack(float16_t (&tot)[TILES], const float16_t (&part)[2], float &s_prev, const Scales &cur, const Scales &nxt,
                                                const typename Op::Consts &consts, typename Op::Tmp &tmp, uint4_t (&B)[2][kSteps], const Word &word)
{
    if constexpr (Slot::kStepping) {
        static_range<Slot::es * 16 / Slot::kStepSlots, (Slot::es + 1) * 16 / Slot::kStepSlots>([&](auto i_) {
            constexpr int i = decltype(i_)::value;
            tot[Slot::tp][i] = __builtin_fmaf(s_prev, part[Slot::pp ^ 1][i], tot[Slot::tp][i]);
        });
        if constexpr (Slot::es == Slot::kStepSlots - 1) s_prev = cur.s[Slot::ct][Slot::seg];
    }
    if constexpr (Slot::kUnpacking) {
        constexpr int jobs = (Slot::w_end - Slot::w_beg) * Op::kParts, n = Slot::kUnpackSlots, i = Slot::kUnpackSlot;
        static_range<i * jobs / n, (i + 1) * jobs / n>([&](auto jb_) {
            constexpr int jb = decltype(jb_)::value, w = Slot::w_beg + jb / Op::kParts;
            Op::unpack(jb % Op::kParts, word(std::integral_constant<int, w>{}), Slot::ct == 0 ? cur.z[1][w / Slot::kStepsPerSeg] : nxt.z[0][w / Slot::kStepsPerSeg],
                       consts, tmp, B[Slot::ct ^ 1][w]);
        });
    }
}

}  // namespace w4a16
