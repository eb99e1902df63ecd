// W4A16 multiply for few rows of X (the scheduler's choice for M <= 16 where the stripe family does not
// pay): one workgroup per (64-column tile, K slice, block of 16 rows of X), the slice handed out to the
// workgroup's waves in units as they become free.
//
// Operands of the 16x16x32 MFMA in its plain form, as in the tile family (w4a16_tile.hip): a lane's 32-bit
// word (eight k of one column) is its B-operand slice, lane (g, j) holding packed row 4 b + g of block b
// (32 k) and columns 4 j .. 4 j + 3 of the tile (one 16-byte load: a wave-wide load reads 256 contiguous bytes
// of each of four packed rows); the A operand is row j of the workgroup's rows of X, k-group g, from LDS.
// sum_k x_k per row comes from one more MFMA per block, X against a constant operand of ones.
//
// How the slice is shared is the decode kernel's way (w4a16_stripe_dyn.hip): a unit is up to four blocks of one
// quantisation group (the whole group for group = 128) or two or four short groups, a wave draws its next unit from an LDS ticket counter,
// every group's share of it (Eq. 2) is rounded to a multiple of 2^-24, and from there on all sums are exact
// (integer-valued doubles per wave and in LDS, 64-bit integers across workgroups): Algorithm 1's Phase 3 with
// results that do not depend on which wave took which unit.  A wave stages the X of a unit itself, in its own
// LDS (no barrier in the loop).
#include "w4a16_device.h"
#include "w4a16_finish.h"
#include "w4a16_internal.h"
#include <type_traits>

namespace w4a16 {
namespace {

constexpr int kTileCols = 64;
constexpr int kRowsX = 16;
constexpr int kBlockRows = 4;                    // packed rows per block: one MFMA step of 32 k
// LDS entries per packed row, padded: a 16-byte LDS write goes eight lanes at a time (two rows of X x four packed rows)
// over 32 banks; with 18 entries a packed row starts 8 banks after its predecessor and a row of X 4 banks after its own
// (measured: SQ_LDS_BANK_CONFLICT 2.4 times lower than with 17).
constexpr int kRowStride = kRowsX + 2;

// LDS: ticket counter (16 B), the workgroup's sums [column slots][rows][64 lanes] (doubles, Share below), then per wave and ring place one unit of X.
constexpr uint32_t kLdsAcc = 16;
template <int UB>
constexpr uint32_t unit_x_bytes() { return UB * kBlockRows * kRowStride * 16; }

// Which outputs a lane keeps, by MR = rows of X the kernel is compiled for (M rounded up to 1, 2, 4, 8, 16).  The MFMA's result rows
// 4 g + i of lane group g are rows of X again and again where there are fewer than 16 (the A operand repeats them, free), so that
// group g has every output of its column slots and takes on some: all four column slots and rows 4 g .. 4 g + 3 (MR = 16), two slots
// and rows 4 (g mod 2) .. + 3 (8), one slot and rows 0 .. MR - 1 (1, 2, 4).  The unit's last step, which without its memory accesses
// took up to a third of the kernel's loop, is then done for outputs that exist only: 16, 8, 4, 2 or 1 per lane; and a load of X
// takes several blocks.  What bounds the kernel is its vector instructions: with every load out of range (no memory traffic) it takes 80 to 90 %
// of its time, and more waves or units in flight do not help.  us per multiply, sixteen rows' work / the form for M:
// M = 4, K = 4096, N = 11008, BF16 9.4 / 7.95; M = 8, K = 28672, N = 8192 25.55 / 24.7; M = 4, K = 28672, N = 8192 26.0 / 22.5; the same bits.
template <int MR>
struct Share {
    static constexpr int kCols = MR == 16 ? 4 : (MR == 8 ? 2 : 1);  // column slots per lane
    static constexpr int kRows = MR < 4 ? MR : 4;                   // rows per lane
    static constexpr int kSums = 64 * kCols * kRows;
    static constexpr int kRowsStaged = MR < 4 ? 4 : MR;             // rows of X in LDS: what the A operand repeats
    static constexpr int kBlocksPerLoad = 16 / kRowsStaged;         // a wave-wide load of X: 16 rows of one block, 8 of two, 4 of four
    // where the sum of (row r, column q of the tile) lies in LDS: neighbouring lanes on neighbouring banks
    static __device__ __forceinline__ int place(int r, int q)
    {
        const int j = q >> 2;
        if constexpr (MR == 16) return 64 * (4 * (q & 3) + (r & 3)) + 16 * (r >> 2) + j;
        if constexpr (MR == 8) return 64 * (4 * (q & 1) + (r & 3)) + 16 * ((r >> 2) + (q & 2)) + j;
        return 64 * r + 16 * (q & 3) + j;
    }
};

// UB: blocks of 32 k per unit; BPG: those of one group in it (UB unless a unit holds several groups).
// BOUND: the most threads of a workgroup (the registers a wave may use follow from it: 128 at 1024, 256 at 512).
constexpr uint32_t lds_x(int mr) { return kLdsAcc + (uint32_t)(mr * kTileCols * 8); }  // the sums: one per output, whatever the share

template <typename Act, int UB, int BPG, int D, int BOUND, int MR>
__global__ __launch_bounds__(BOUND) void tile_dyn_kernel(const GemmArgs a, const int finish, unsigned long long *__restrict__ sync)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    typedef Share<MR> Sh;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = blockDim.x >> 6;
    const int nthreads = blockDim.x;
    const int g4 = lane >> 4, j = lane & 15;
    // grid: x = K slice (the slices of one tile are neighbours in the launch order, hence on different XCDs),
    // y = column tile, z = block of 16 rows of X
    const int slice = blockIdx.x, tile = blockIdx.y, m0 = blockIdx.z * kRowsX;
    const int col0 = tile * kTileCols + 4 * j;
    const bool ok = col0 < a.N;

    // the workgroup's K slice: groups, blocks, units
    const int gbeg = slice * a.groups_per_split;
    int gend = gbeg + a.groups_per_split;
    if (gend > a.groups) gend = a.groups;
    const int groups = gend - gbeg;
    constexpr int NG = UB / BPG;                     // groups of a unit
    const int upg = NG == 1 ? (a.group >> 5) / UB : 1;            // units per group (of a unit of one group)
    const int units = NG == 1 ? groups * upg : (groups + NG - 1) / NG;
    const int row_base = gbeg * (a.group >> 3);      // first packed row of the slice

    const uint32_t row_w = (uint32_t)a.N * 4u, row_s = (uint32_t)a.N * 2u, row_z = (uint32_t)(a.N >> 3) * 4u;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t *>(a.Wp) + (size_t)row_base * a.N, 0, (uint32_t)groups * (uint32_t)(a.group >> 3) * row_w, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(a.scales) + (size_t)gbeg * a.N, 0, (uint32_t)groups * row_s, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t *>(a.Zp) + (size_t)gbeg * (a.N >> 3), 0, zero_point_bytes(a.Zp, (uint32_t)groups * row_z), kRawBuffer);
    const uint32_t zfill = symmetric_fill(a.Zp);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(a.X), 0, (uint32_t)((size_t)a.M * a.K * 2), kRawBuffer);
    const uint32_t vw = ok ? (uint32_t)(g4 * a.N + col0) * 4u : kOutOfRange;
    const uint32_t vs = ok ? (uint32_t)col0 * 2u : kOutOfRange;
    const uint32_t vz = ok ? (uint32_t)(col0 >> 3) * 4u : kOutOfRange;
    // X: four neighbouring lanes fetch the 64 bytes one block takes of one row of X; load l of a lane is block kBlocksPerLoad l + xb
    constexpr int kLoadsX = (UB + Sh::kBlocksPerLoad - 1) / Sh::kBlocksPerLoad;
    const uint32_t xr = (uint32_t)(lane >> 2) % Sh::kRowsStaged, xb = (uint32_t)(lane >> 2) / Sh::kRowsStaged, xm = (uint32_t)m0 + xr;
    const bool has_x = Sh::kBlocksPerLoad <= UB || xb < UB;
    const uint32_t vx = xm < (uint32_t)a.M && has_x ? (xm * (uint32_t)a.K + ((uint32_t)row_base + kBlockRows * xb + (uint32_t)(lane & 3)) * 8u) * 2u : kOutOfRange;
    const uint32_t xl = (xb * (kBlockRows * kRowStride) + (uint32_t)(lane & 3) * kRowStride + xr) * 16u;  // where it goes in the unit's LDS

    struct Unit {
        uint4_t w[UB], x[kLoadsX];
        uint2_t sc[NG];
        uint32_t zw[NG];
    };
    Unit ring[D];
    int uidx[D];  // unit in ring place p, -1 = none
    auto load_unit = [&](Unit &r, int u) {
        const bool valid = u >= 0;
        const uint32_t uu = valid ? (uint32_t)u : 0u;
        const uint32_t g = NG == 1 ? uu / (uint32_t)upg : uu * NG, b0 = uu * UB;  // first group and first block (of the slice)
        // Groups past the slice's last one: every lane's own offset is out of range (the scalar offset is no part of the slice then, and
        // the range check is not to depend on it).  Their X too: zeros times whatever follows it would not do, that may be an infinity.
#pragma unroll
        for (int l = 0; l < kLoadsX; ++l) {  // X ahead of the weights: loads return in order, and these mostly come from cache
            const uint32_t b = b0 + l * Sh::kBlocksPerLoad, last = (uint32_t)(groups * BPG);
            const bool in = valid && (NG == 1 || b + xb < last);
            r.x[l] = __builtin_amdgcn_raw_buffer_load_b128(rx, in ? vx : kOutOfRange, (NG == 1 || b < last ? b : 0u) * (kBlockRows * 16u), 0);
        }
        uint32_t gin[NG];  // group h of the unit, or 0 where there is none
        bool has[NG];
#pragma unroll
        for (int h = 0; h < NG; ++h) {
            has[h] = valid && (h == 0 || g + h < (uint32_t)groups);
            gin[h] = h == 0 || has[h] ? g + h : 0u;
            r.sc[h] = __builtin_amdgcn_raw_buffer_load_b64(rs, has[h] ? vs : kOutOfRange, gin[h] * row_s, 0);
            r.zw[h] = __builtin_amdgcn_raw_buffer_load_b32(rz, has[h] ? vz : kOutOfRange, gin[h] * row_z, 0) | zfill;
        }
#pragma unroll
        for (int q = 0; q < UB; ++q) {  // read once from DRAM: nontemporal
            const uint32_t b = NG == 1 ? b0 + q : gin[q / BPG] * BPG + q % BPG;
            r.w[q] = __builtin_amdgcn_raw_buffer_load_b128(rw, has[q / BPG] ? vw : kOutOfRange, b * (kBlockRows * row_w), 2);
        }
    };
#pragma unroll
    for (int p = 0; p < D; ++p) {
        const int u = wave + p * waves;
        uidx[p] = u < units ? u : -1;
        load_unit(ring[p], uidx[p]);
    }

    uint32_t *const tickets = reinterpret_cast<uint32_t *>(smem);
    double *const acc = reinterpret_cast<double *>(smem + kLdsAcc);
    if (tid == 0) tickets[0] = (uint32_t)(waves * D);
    for (int e = tid; e < Sh::kSums; e += nthreads) acc[e] = 0.0;
    __syncthreads();

    unsigned char *const myx = smem + lds_x(MR) + (uint32_t)wave * unit_x_bytes<UB>();  // one unit of X, this wave's own
    const uint32_t xa = (uint32_t)((g4 * kRowStride + (MR == 16 ? j : j & (MR == 8 ? 7 : 3))) * 16);  // this lane's A entry of block 0
    const int slot0 = MR == 16 ? 0 : (MR == 8 ? g4 & 2 : g4);                          // the first of this lane's column slots
    const int row0 = MR == 16 ? 4 * g4 : (MR == 8 ? 4 * (g4 & 1) : 0);                 // the first of its rows
    const uint32_t zsh = (uint32_t)((col0 & 4) + slot0) * 4u;                         // its nibbles in its zero-point word

    double tot[Sh::kCols][Sh::kRows];
#pragma unroll
    for (int c = 0; c < Sh::kCols; ++c)
#pragma unroll
        for (int i = 0; i < Sh::kRows; ++i) tot[c][i] = 0.0;
    const Masks masks = make_masks();
    // sum_k x_k over a unit comes from the MFMA too: X against ones (FP16: 16 where the staged x was divided by 16).  (Against
    // ones times 2^-24, subnormals, the sum comes out with fewer bits: an error of 2.3e-4 instead of 2.1e-4.)
    const typename Act::operand_t ones = Act::ones();
    const float4_t zero4 = {0.f, 0.f, 0.f, 0.f};

    auto draw = [&]() -> int {
        uint32_t t = 0;
        if (lane == 0) t = __hip_atomic_fetch_add(tickets, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return (int)__builtin_amdgcn_readfirstlane(t);
    };
    int next = draw();

    auto compute_unit = [&](Unit &r) {
        // only this wave touches its LDS and the LDS operations of one wave complete in order; the fences only
        // keep the compiler from moving them across the staging
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int l = 0; l < kLoadsX; ++l)
            if (has_x) *reinterpret_cast<uint4_t *>(myx + (uint32_t)(l * Sh::kBlocksPerLoad) * (kBlockRows * kRowStride * 16) + xl) = Act::stage_x(r.x[l]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int h = 0; h < NG; ++h) {
            float4_t part[4], xsum;
#pragma unroll
            for (int q = 0; q < BPG; ++q) {
                const int b = h * BPG + q;
                const typename Act::operand_t x = Act::x_operand(*reinterpret_cast<const uint4_t *>(myx + (uint32_t)b * (kBlockRows * kRowStride * 16) + xa));
#pragma unroll
                for (int c = 0; c < 4; ++c) part[c] = Act::mfma(x, Act::unpack(r.w[b][c], masks), q == 0 ? zero4 : part[c]);
                xsum = Act::mfma(x, ones, q == 0 ? zero4 : xsum);
            }
            // the group's share is done: scale and zero point (Eq. 2), then the exact sums
            const unsigned long long scales = (((unsigned long long)r.sc[h][1] << 32) | r.sc[h][0]) >> (16 * slot0);
            const uint32_t zw = r.zw[h] >> zsh;
#pragma unroll
            for (int c = 0; c < Sh::kCols; ++c) {
                H2 s;
                s.u = (uint32_t)(scales >> (16 * c)) & 0xFFFFu;
                const UnitScales u = unit_scales<Act>((float)s.h[0], (zw >> (4 * c)) & 15u);
#pragma unroll
                for (int i = 0; i < Sh::kRows; ++i) {
                    float P = part[c][i];
                    if constexpr (MR == 8) P = g4 & 2 ? part[c + 2][i] : P;
                    if constexpr (MR <= 4) {
                        const float even = g4 & 2 ? part[2][i] : P, odd = g4 & 2 ? part[3][i] : part[1][i];
                        P = g4 & 1 ? odd : even;
                    }
                    add_unit(tot[c][i], u, P, xsum[i]);
                }
            }
            if constexpr (NG > 1) __builtin_amdgcn_sched_barrier(0);  // group after group: mixed, their sums do not fit the registers
        }
    };

    for (;;) {
        bool any = false;
#pragma unroll
        for (int p = 0; p < D; ++p) {
            if (uidx[p] >= 0) {
                any = true;
                compute_unit(ring[p]);
                uidx[p] = next < units ? next : -1;
                load_unit(ring[p], uidx[p]);
                if (next < units) next = draw();
            }
        }
        if (!any) break;
    }

    // ---- Phase 3 inside the workgroup: exact sums in LDS, neighbouring lanes on neighbouring banks.  (As [16][64] the sixteen lanes of a
    // group were 32 bytes apart and the four groups in the same banks; with the conversions to integers per wave 1.7 us from a wave's
    // last unit to the barrier at M = 16, K = 14336, N = 4096, 1.2 now, and 1.0 and 0.3 at M = 1, K = 4096, N = 1024.)
#pragma unroll
    for (int i = 0; i < Sh::kRows; ++i) {
        if (m0 + row0 + i >= a.M) continue;
#pragma unroll
        for (int c = 0; c < Sh::kCols; ++c) add_wave_sum(acc + 64 * (Sh::kRows * c + i) + lane, tot[c][i]);
    }
    __syncthreads();
    // ---- and across workgroups ----
    for (int o = tid; o < MR * kTileCols; o += nthreads) {
        const int r = o / kTileCols, q = o % kTileCols, m = m0 + r, col = tile * kTileCols + q;
        if (m >= a.M || col >= a.N) continue;
        const double t = acc[Sh::place(r, q)];
        const bool nan = t != t;
        const long long fx = nan ? 0ll : (long long)t;
        const size_t out = (size_t)m * a.N + col;
        if (finish == kFinishAccumulator) {
            add_slice<Act>(sync + out, to_fixed(fx), nan, a.split, a.Y + out);
        } else {
            constexpr long long lim = 1ll << 49;
            const float v = nan ? __builtin_nanf("") : (float)((double)(fx < -lim ? -lim : (fx > lim ? lim : fx)) * (1.0 / 16777216.0));
            if (finish == kFinishDirect)
                a.Y[out] = nan ? Act::kNaN : (uint16_t)(Act::pack2(v, 0.f) & 0xFFFFu);
            else
                a.partials[(size_t)slice * a.M * a.N + out] = v;
        }
    }
}

template <typename Act, int UB, int BPG, int D, int BOUND, int MR>
hipError_t launch_mr(const GemmArgs &a, int finish, unsigned long long *sync, int waves, hipStream_t stream)
{
    const size_t lds = lds_x(MR) + (size_t)waves * unit_x_bytes<UB>();
    const int ntiles = (a.N + kTileCols - 1) / kTileCols, row_blocks = (a.M + kRowsX - 1) / kRowsX;
    if (ntiles > 65535 || row_blocks > 65535 || (MR < 16 && a.M > MR)) return hipErrorInvalidValue;
    if (lds > 48 * 1024) {  // beyond the default dynamic-LDS allowance
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&tile_dyn_kernel<Act, UB, BPG, D, BOUND, MR>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((tile_dyn_kernel<Act, UB, BPG, D, BOUND, MR>), dim3(a.split, ntiles, row_blocks), dim3(waves * 64), lds, stream, a, finish, sync);
    return hipGetLastError();
}

template <typename Act, int UB, int BPG, int D>
hipError_t launch_ud(const GemmArgs &a, int finish, unsigned long long *sync, int waves, hipStream_t stream)
{
    // two units in flight need more than 128 registers: up to eight waves per workgroup only (for sweeps: 16 rows only); units of
    // several groups may
    constexpr int BOUND = D == 2 || UB > BPG ? 512 : 1024;
    if (64 * waves > BOUND) return hipErrorInvalidValue;
    if constexpr (D == 2) {
        return launch_mr<Act, UB, BPG, D, BOUND, 16>(a, finish, sync, waves, stream);
    } else {
        if (a.M == 1) return launch_mr<Act, UB, BPG, D, BOUND, 1>(a, finish, sync, waves, stream);
        if (a.M == 2) return launch_mr<Act, UB, BPG, D, BOUND, 2>(a, finish, sync, waves, stream);
        if (a.M <= 4) return launch_mr<Act, UB, BPG, D, BOUND, 4>(a, finish, sync, waves, stream);
        if (a.M <= 8) return launch_mr<Act, UB, BPG, D, BOUND, 8>(a, finish, sync, waves, stream);
        return launch_mr<Act, UB, BPG, D, BOUND, 16>(a, finish, sync, waves, stream);
    }
}

}  // namespace

// `finish` says how the slices meet (w4a16_finish.h); `sync` is the accumulator it may need.  `depth`: units in
// flight per wave (1 or 2).
hipError_t launch_tile_dyn(const GemmArgs &a, int finish, unsigned long long *sync, int waves, int depth, int unit_blocks, hipStream_t stream)
{
    if (a.group % 32 != 0 || waves < 1 || waves > 16) return hipErrorInvalidValue;
    if (!finish_args_ok(a, finish, sync)) return hipErrorInvalidValue;
    const unsigned long long rows = (unsigned long long)a.groups_per_split * (a.group / 8);
    if (rows * a.N * 4ull >= 0x7F000000ull) return hipErrorInvalidValue;  // slice-relative 32-bit buffer offsets
    if ((unsigned long long)a.M * a.K * 2ull >= 0x7F000000ull) return hipErrorInvalidValue;
    // Blocks per unit: the most up to unit_blocks that divide a group, or four of two or four whole groups (in the form with eight
    // waves and one unit in flight).
    const int bpg = a.group / 32;
    int ub = 1;
    if (unit_blocks >= 2 && bpg % 2 == 0) ub = 2;
    if (unit_blocks >= 4 && (bpg % 4 == 0 || (bpg <= 2 && waves <= 8 && depth == 1))) ub = 4;
    auto launch = [&](auto act, auto in_flight) {
        typedef decltype(act) Act;
        constexpr int D = decltype(in_flight)::value;
        if constexpr (D == 1) {
            if (ub == 4 && bpg == 1) return launch_ud<Act, 4, 1, D>(a, finish, sync, waves, stream);
            if (ub == 4 && bpg == 2) return launch_ud<Act, 4, 2, D>(a, finish, sync, waves, stream);
        }
        if (ub == 4) return launch_ud<Act, 4, 4, D>(a, finish, sync, waves, stream);
        if (ub == 2) return launch_ud<Act, 2, 2, D>(a, finish, sync, waves, stream);
        return launch_ud<Act, 1, 1, D>(a, finish, sync, waves, stream);
    };
    if (a.bf16) return depth == 1 ? launch(ActBF16{}, std::integral_constant<int, 1>{}) : hipErrorInvalidValue;  // the scheduler's depth only
    return depth == 2 ? launch(ActF16{}, std::integral_constant<int, 2>{}) : launch(ActF16{}, std::integral_constant<int, 1>{});
}

}  // namespace w4a16
