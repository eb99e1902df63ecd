// Second pass of Split-K (Algorithm 1, Phase 3): C = sum_{i<S} C_i element by
// element in FP32, i ascending, then one round-to-nearest-even cast to FP16 (or
// to bfloat16, for bfloat16 activations).
#include "w4a16_device.h"
#include "w4a16_internal.h"

namespace w4a16 {
namespace {


// One thread owns four consecutive columns of one row (N % 8 == 0 keeps the
// 16-byte loads aligned and inside the row).  What bounds it is latency: a load
// after another takes a microsecond each.  Four in flight whatever S (eight, and
// single ones for the rest, before): the whole multiply of M = 37, K = 10240,
// N = 4608, groups of 64 in seven slices 17.3 -> 16.6 us, of M = 128, K = 18432,
// N = 2048 in eight 23.0 -> 22.6, of M = 100, K = 14336, N = 4096 in four 23.7 -> 23.4.
template <typename Act>
__global__ __launch_bounds__(256) void reduce_kernel(const float *__restrict__ partials, int S, size_t MN,
                                                    uint16_t *__restrict__ Y)
{
    const size_t i4 = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i4 >= MN) return;
    float4_t acc = *reinterpret_cast<const float4_t *>(partials + i4);
    for (int s = 1; s < S; s += 4) {  // up to four loads in flight, added in slice order
        float4_t v[4] = {};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (s + e < S) v[e] = *reinterpret_cast<const float4_t *>(partials + (size_t)(s + e) * MN + i4);
        asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));  // all asked for before the first is added
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (s + e < S) acc += v[e];
    }
    *reinterpret_cast<uint2_t *>(Y + i4) = (uint2_t){Act::pack2(acc[0], acc[1]), Act::pack2(acc[2], acc[3])};
}

// Clears n words of a fixed-point accumulator (a fill kernel, so that a caller may capture it in a HIP graph).
__global__ __launch_bounds__(256) void clear_kernel(unsigned long long *p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

}  // namespace

hipError_t launch_accumulator_clear(unsigned long long *acc, size_t n, hipStream_t stream)
{
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, acc, n);
    return hipGetLastError();
}

hipError_t launch_reduce(const float *partials, int S, int M, int N, uint16_t *Y, bool bf16, hipStream_t stream)
{
    const size_t MN = (size_t)M * N;
    const unsigned blocks = (unsigned)((MN / 4 + 255) / 256);
    if (bf16)
        hipLaunchKernelGGL(reduce_kernel<ActBF16>, dim3(blocks), dim3(256), 0, stream, partials, S, MN, Y);
    else
        hipLaunchKernelGGL(reduce_kernel<ActF16>, dim3(blocks), dim3(256), 0, stream, partials, S, MN, Y);
    return hipGetLastError();
}

}  // namespace w4a16
