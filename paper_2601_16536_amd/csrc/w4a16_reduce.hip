// Second pass of Split-K (Algorithm 1, Phase 3): C = sum_{i<S} C_i element by
// element in FP32, i ascending, then one round-to-nearest-even cast to FP16 (or
// to bfloat16, for bfloat16 activations).
#include "w4a16_device.h"
#include "w4a16_internal.h"
#include <type_traits>

namespace w4a16 {
namespace {


// One thread owns four consecutive columns of one row (N % 8 == 0 keeps the
// 16-byte loads aligned and inside the row).  What bounds it is latency: a load
// after another takes a third of a microsecond each.  Eight in flight, and the
// one to seven that are left over together: this launch for 36 rows of 2048
// columns at 2 / 4 / 7 / 9 / 16 / 17 / 32 slices 2.0 / 2.1 / 2.3 / 2.5 / 3.2 /
// 3.3 / 4.7 us; with the left-over ones singly 1.9 / 2.5 / 3.5 / 2.4 / 4.4 / 3.2 /
// 6.1, in fours, those past the end left out, 2.0 / 2.1 / 2.7 / 2.8 / 3.8 / 3.9 / 6.2.
template <typename Act>
__global__ __launch_bounds__(256) void reduce_kernel(const float *__restrict__ partials, int S, size_t MN,
                                                    uint16_t *__restrict__ Y)
{
    const size_t i4 = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i4 >= MN) return;
    float4_t acc = *reinterpret_cast<const float4_t *>(partials + i4);
    int s = 1;
    auto batch = [&](auto n_) {  // so many loads in flight, added in slice order
        constexpr int n = decltype(n_)::value;
        float4_t v[n];
#pragma unroll
        for (int e = 0; e < n; ++e) v[e] = *reinterpret_cast<const float4_t *>(partials + (size_t)(s + e) * MN + i4);
#pragma unroll
        for (int e = 0; e < n; ++e) acc += v[e];
        s += n;
    };
    while (s + 8 <= S) batch(std::integral_constant<int, 8>());
    switch (S - s) {
    case 1: batch(std::integral_constant<int, 1>()); break;
    case 2: batch(std::integral_constant<int, 2>()); break;
    case 3: batch(std::integral_constant<int, 3>()); break;
    case 4: batch(std::integral_constant<int, 4>()); break;
    case 5: batch(std::integral_constant<int, 5>()); break;
    case 6: batch(std::integral_constant<int, 6>()); break;
    case 7: batch(std::integral_constant<int, 7>()); break;
    default: break;
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
