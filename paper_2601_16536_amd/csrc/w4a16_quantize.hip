// Offline tool, not on the hot path: uniform affine quantization of FP16 weights to the
// INT4 codes, FP16 scales and INT4 zero points the multiply reads (Section 2.1, Eq. 1:
// x_q = round(x / s) + z).  The paper does not say how s and z are found; here, per
// quantisation group of one column, in FP32: lo = min(min w, 0), hi = max(max w, 0),
// s = fp16((hi - lo) / 15) (1 if that is 0), z = clamp(rint(-lo / s), 0, 15),
// q = clamp(rint(w / s) + z, 0, 15), round to nearest even.
#include "w4a16_device.h"
#include "w4a16_internal.h"
#include <type_traits>

namespace w4a16 {
namespace {

constexpr int kCols = 256;      // columns per workgroup: 32 lanes x 8
constexpr int kLaneRows = 16;   // rows (two packed rows) of a thread's eight columns
constexpr int kChunk = 128;     // rows per workgroup and chunk: 8 row lanes
constexpr int kMaxGroups = 4;   // groups of 32 in a chunk

// A workgroup owns 128 rows x 256 columns (whole groups of 32, 64 or 128 rows), or one group of another length, which it
// walks in chunks of 128 rows.  Bound by memory: 2 bytes read and 0.5 written per weight.  A thread loads 16 rows of eight
// columns, 16 bytes each (512 contiguous bytes per half wave), and keeps them in registers between the two walks, so that
// a group up to 128 rows is read once; the form before this one (a thread per column, 2-byte loads, each group read twice,
// a division per weight) took 85 us at K = 4096, N = 11008, this one 24.7 (4.6 TB/s).  Range and parameters meet in LDS.
//
// rint(w / s) without a division per weight: w and s are FP16, so w / s = n + 1/2 exactly, or differs from it by at least
// 2^-14 (the numerator of the difference, over the denominator 2 S with S < 2^11, is a multiple of 2^-2 wherever |w| >= s / 2;
// below that the code is z whatever the quotient).  w r, r = fl(1 / s), is off by at most 2^-19 for quotients below 32, so
// rounding it to a multiple of 2^-16 (by adding 192, whose unit in the last place that is) recovers the exact tie and
// moves nothing else across one.  -> 5 instructions per weight.
__global__ __launch_bounds__(256) void quantize_kernel(const uint16_t *__restrict__ W16, int group, int N, int K, int rows_wg,
                                                      uint32_t *__restrict__ Wp, uint16_t *__restrict__ scales, uint32_t *__restrict__ Zp)
{
    __shared__ uint4_t red[2][8][kCols / 8];                   // lo, hi of a thread's rows, eight columns packed
    __shared__ __attribute__((aligned(16))) float rs[kMaxGroups][kCols], zs[kMaxGroups][kCols];  // 1 / s and z
    const int tid = threadIdx.x, rl = tid >> 5, cl = tid & 31;
    const int nx = (N + kCols - 1) / kCols, by = (int)blockIdx.x / nx, col0 = ((int)blockIdx.x - by * nx) * kCols;
    const int col = col0 + cl * 8;
    const bool live = col < N;  // N is a multiple of 8
    const int row0 = by * rows_wg;
    const int row_end = row0 + rows_wg < K ? row0 + rows_wg : K;  // this workgroup's rows: whole groups
    const int chunks = (row_end - row0 + kChunk - 1) / kChunk;
    const int glen = chunks > 1 ? rows_wg : group;                // several chunks: one group
    const int lanes = glen < kChunk ? glen / kLaneRows : 8;       // row lanes that share a group within a chunk
    const int groups = (row_end - row0 + glen - 1) / glen;        // at most kMaxGroups

    uint4_t d[kLaneRows];
    auto load = [&](int chunk, auto once) {
        const int r = row0 + chunk * kChunk + rl * kLaneRows;
#pragma unroll
        for (int i = 0; i < kLaneRows; ++i) {
            const uint4_t *const p = reinterpret_cast<const uint4_t *>(W16 + (size_t)(r + i) * N + col);
            d[i] = (uint4_t){0u, 0u, 0u, 0u};
            if (live && r + i < row_end) d[i] = decltype(once)::value ? __builtin_nontemporal_load(p) : *p;
        }
    };
    H2 lo[4], hi[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) lo[p].u = hi[p].u = 0u;
    for (int c = 0; c < chunks; ++c) {
        if (chunks == 1) load(c, std::true_type{});  // read once: 24.7 against 28.0 us with ordinary loads
        else load(c, std::false_type{});
#pragma unroll
        for (int i = 0; i < kLaneRows; ++i)
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                H2 v;
                v.u = d[i][p];
                lo[p].h = __builtin_elementwise_min(lo[p].h, v.h);
                hi[p].h = __builtin_elementwise_max(hi[p].h, v.h);
            }
    }
    red[0][rl][cl] = (uint4_t){lo[0].u, lo[1].u, lo[2].u, lo[3].u};
    red[1][rl][cl] = (uint4_t){hi[0].u, hi[1].u, hi[2].u, hi[3].u};
    __syncthreads();
    // a thread per column: the groups' scales and zero points
    const int n = col0 + tid;
    const int grow = row0 / group;  // first group's row of scales
    for (int g = 0; g < groups; ++g) {
        float l = 0.f, h = 0.f;
        for (int e = 0; e < lanes; ++e) {
            const int r = (g * lanes + e) & 7;
            l = fminf(l, (float)reinterpret_cast<const _Float16 *>(&red[0][r][0])[tid]);
            h = fmaxf(h, (float)reinterpret_cast<const _Float16 *>(&red[1][r][0])[tid]);
        }
        _Float16 s16 = (_Float16)((h - l) / 15.0f);
        if (s16 == (_Float16)0.f) s16 = (_Float16)1.f;
        const float s = (float)s16;
        const float z = fminf(fmaxf(rintf(-l / s), 0.f), 15.f);
        rs[g][tid] = 1.0f / s;
        zs[g][tid] = z;
        uint32_t zw = (uint32_t)z << (4 * (tid & 7));
        zw |= __shfl_xor(zw, 1, 64);
        zw |= __shfl_xor(zw, 2, 64);
        zw |= __shfl_xor(zw, 4, 64);
        if (n < N) {  // eight lanes of a zero-point word live or die together
            H2 b;
            b.h = (half2_t){s16, s16};
            scales[(size_t)(grow + g) * N + n] = (uint16_t)(b.u & 0xFFFFu);
            if ((n & 7) == 0) Zp[(size_t)(grow + g) * (N >> 3) + (n >> 3)] = zw;
        }
    }
    __syncthreads();
    const int g = rl / lanes < groups ? rl / lanes : 0;  // (row lanes past the rows store nothing)
    constexpr float kGrid = 192.0f, kInt = 12582912.0f;  // 1.5 2^23: adding it leaves a whole number in the low bits
    float r8[8], z8[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        r8[c] = rs[g][cl * 8 + c];
        z8[c] = (kInt - kGrid) + zs[g][cl * 8 + c];
    }
    for (int c = 0; c < chunks; ++c) {
        if (chunks > 1) load(c, std::false_type{});
        const int r = row0 + c * kChunk + rl * kLaneRows;
#pragma unroll
        for (int w = 0; w < kLaneRows / 8; ++w) {
            uint32_t word[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t acc = 0;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    H2 v;
                    v.u = d[8 * w + i][e >> 1];
                    const float t = __builtin_rintf(__builtin_fmaf((float)v.h[e & 1], r8[e], kGrid));  // 192 is even: ties as without it
                    // a NaN ends as code 0 (the median of it and two numbers is the smaller one)
                    const float q = __builtin_amdgcn_fmed3f(t + z8[e], kInt, kInt + 15.0f);
                    acc = __builtin_amdgcn_alignbit(__builtin_bit_cast(uint32_t, q), acc, 4);  // its low four bits in at the top
                }
                word[e] = acc;
            }
            if (live && r + 8 * w < row_end) {
                uint4_t *const out = reinterpret_cast<uint4_t *>(Wp + (size_t)((r >> 3) + w) * N + col);
                out[0] = (uint4_t){word[0], word[1], word[2], word[3]};
                out[1] = (uint4_t){word[4], word[5], word[6], word[7]};
            }
        }
    }
}

}  // namespace

hipError_t launch_quantize(const uint16_t *W16, int group, int N, int K, uint32_t *Wp, uint16_t *scales, uint32_t *Zp,
                           hipStream_t stream)
{
    const int rows_wg = kChunk % group == 0 ? kChunk : group;
    const long long blocks = (((long long)K + rows_wg - 1) / rows_wg) * ((N + kCols - 1) / kCols);
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(quantize_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, W16, group, N, K, rows_wg, Wp, scales, Zp);
    return hipGetLastError();
}

}  // namespace w4a16
