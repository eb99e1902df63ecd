// W4A16 multiply, TILE family at 64 rows of X per workgroup for BF16 and for groups other than 128 (FP16 with groups of 128
// has w4a16_tile_wide.hip, BF16 with groups of 128 and slices of up to 1024 k the eight-wave w4a16_tile.hip): one workgroup of four waves per (64-column tile, 64 rows of X, K slice), every wave alone on its
// SIMD with a quarter of the slice's K and the whole 64 x 64 result.
//
// What bounds it: a stage (128 k) is 32 MFMAs 32x32x16, 160 vector instructions of unpack (FP16; 272 BF16), 64 of Eq. 2's step
// and about 48 of addressing per wave, 0.77 us measured without the loads; the loads into LDS of X, which every wave
// fetches for itself (64 KiB per workgroup and stage from the L2), and those of the weights bring that to 1.1 and 1.3 us.  So:
//   - the operand is q - z, exact, in the order of k (w4a16_wide_ops.h: 10 vector instructions per word for FP16, 17 for
//     BF16, which the eight-wave form unpacks to 128 + q and pays a fifth MFMA and a second FMA to correct): X needs no
//     reordering and goes straight from global memory into LDS;
//   - X of two stages per wave in LDS (all there is room for), weights of three in registers, asked for in one order, X
//     ahead of the weights; loads return in order, so the waits are counts;
//   - 32x32x16 MFMAs, a tile's eight of a stage as one chain; the order of instructions written down slot by slot, as in
//     w4a16_panel.hip.
// M = 128, K = N = 8192 (256 workgroups): BF16 27.8 us, 34.2 with the eight-wave form; FP16 with groups of 64 27.2, 39.4
// before; M = 110, K = 9856, N = 6704, BF16: 30.7, 45.3 before; M = 37, K = 10240, N = 4608, groups of 64, in three slices:
// 17.1, 18.7 before (16 rows).  One row block (32 rows) of this kind was tried too and is not here: every word is then
// unpacked for 32 rows only (M = 64, K = N = 8192: 20.2 us, the eight- and four-wave forms 22 and 17.7).
// Arithmetic: products x (q - z) exact, sums over a group in FP32 in the MFMA, times s in FP32.
#include "w4a16_finish.h"
#include "w4a16_internal.h"
#include "w4a16_wide_ops.h"

namespace w4a16 {
namespace {

constexpr int kTileCols = 64;
constexpr int kWaves = 4;

// Sizes for RT blocks of 32 rows and SEG k per step of scales.
template <int RT, int SEG>
struct Tall {
    static constexpr int kRows = 32 * RT;
    static constexpr int kSegs = kStage / SEG;
    static constexpr int kBuffers = 2;                  // stages of X per wave in LDS
    static constexpr int kRing = kBuffers + 1;          // stages of weights per wave in registers
    static constexpr int kXLoads = 8 * RT;              // wave-wide loads of a stage's X: four rows of 256 bytes each
    static constexpr int kXBytes = kXLoads * 1024;
    static constexpr int kWLoads = kSteps + 2 * kSegs;  // of its weights, scales and zero points
    static constexpr int kWaveBytes = kBuffers * kXBytes;
    static constexpr int kLds = kWaves * kWaveBytes;
    // operations asked for after the X of the next stage, in the middle of a stage: see the loop
    static constexpr int kWait = (kBuffers - 1) * (kWLoads + kXLoads);
    static constexpr int kWaitFirst = (kRing - 1) * kWLoads + (kBuffers - 1) * kXLoads;
    static_assert(kWait < 64 && kWaitFirst < 64 && kLds <= 160 * 1024, "the wait counter's range, and the LDS of a compute unit");
};

template <typename Op, int RT, int SEG>
__global__ __launch_bounds__(64 * kWaves) void tile_tall_kernel(const GemmArgs a, const int finish, unsigned long long *__restrict__ sync, const Place where)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    typedef Tall<RT, SEG> Sh;
    typedef typename Op::Act Act;
    constexpr int kTiles = 2 * RT;  // 32 x 32 result tiles of a wave: (column half, row block)
    constexpr int kStepsPerSeg = SEG / 16, kSegs = Sh::kSegs, kRing = Sh::kRing;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;

    // workgroup -> (column tile, K slice, row block)
    const int ntiles = (a.N + kTileCols - 1) / kTileCols;
    const int units = ntiles * a.split;
    int unit, rb;
    if (!place_of(where, blockIdx.x, units, &unit, &rb)) return;
    int tile = unit, slice = 0;
    if (a.split > 1) {
        slice = unit / ntiles;
        tile = unit - slice * ntiles;
    }
    const int m0 = rb * Sh::kRows, col0 = tile * kTileCols;

    // The slice's k, and this wave's run of it: whole units of a group, or of a stage where groups are shorter; the first
    // waves one unit more.
    const int run_unit = a.group > kStage ? a.group : kStage;
    const int sbeg = slice * a.groups_per_split * a.group;
    int send = sbeg + a.groups_per_split * a.group;
    if (send > a.K) send = a.K;
    const int run_units = (send - sbeg + run_unit - 1) / run_unit;
    const int per = run_units / kWaves, extra = run_units - per * kWaves;
    const int kbeg = sbeg + (per * wave + (wave < extra ? wave : extra)) * run_unit;
    int kend = kbeg + (per + (wave < extra ? 1 : 0)) * run_unit;
    if (kend > send) kend = send;
    const int klen = kend > kbeg ? kend - kbeg : 0;  // a multiple of 32
    const int stages = (klen + kStage - 1) / kStage;

    float16_t tot[kTiles];
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) tot[t][i] = 0.f;

    unsigned char *const own = smem + wave * Sh::kWaveBytes;
    if (stages > 0) {
        // Every descriptor ends where the wave's run (or the matrix) ends: loads past it return zeros and move nothing.
        const int rows_here = a.M - m0 < Sh::kRows ? a.M - m0 : Sh::kRows;
        const uint32_t row_x = (uint32_t)a.K * 2u, row_w = (uint32_t)a.N * 4u, row_s = (uint32_t)a.N * 2u, row_z = (uint32_t)(a.N >> 3) * 4u;
        const int grp0 = kbeg / a.group;
        const uint32_t ngroups = (uint32_t)(klen / a.group);
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.X) + (size_t)m0 * a.K + kbeg, 0, (uint32_t)rows_here * row_x - (uint32_t)kbeg * 2u, kRawBuffer);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.Wp) + (size_t)(kbeg >> 3) * a.N, 0, (uint32_t)(klen >> 3) * row_w, kRawBuffer);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.scales) + (size_t)grp0 * a.N, 0, ngroups * row_s, kRawBuffer);
        const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.Zp) + (size_t)grp0 * (a.N >> 3), 0, zero_point_bytes(a.Zp, ngroups * row_z), kRawBuffer);
        const uint32_t zfill = symmetric_fill(a.Zp);

        // ---- X: straight from global memory into this wave's LDS; a wave-wide load puts lane l's 16 bytes at base + 16 l ----
        // Four rows of 256 bytes per load; lane l fetches piece (l mod 16) ^ (row mod 8) of row l / 16, so that the MFMA's
        // operand reads (the same piece of consecutive rows) spread over the banks.
        const uint32_t lr = (uint32_t)lane >> 4, lp = (uint32_t)lane & 15u;
        uint32_t xp[2], xg[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            xp[p] = lp ^ (4u * (uint32_t)p + lr);
            xg[p] = (4u * (uint32_t)p + lr) * row_x + xp[p] * 16u;
        }
        int xk = 0;  // k of the run at the next stage to fetch
        uint32_t o0 = 0, o1 = 0;
        auto fetch_x = [&](int buf, int i) {  // load i of Sh::kXLoads; past the run only zeros, for the waits' count
            if (i == 0) {
                o0 = xg[0] + (uint32_t)xk * 2u;
                o1 = xg[1] + (uint32_t)xk * 2u;
                // The run ends inside this stage or before it: by every lane's own offset.  (Where runs are whole stages, a descriptor of no bytes from there on saves
                // three vector instructions a stage and loses: K = 512, N = 115728, M = 46, BF16, groups of 256, 46.6 us so and 50.1 with it, K = N = 8192, M = 128 27.9
                // and 28.1; in w4a16_panel.hip it gains 0.7 %.)
                if (klen - xk < kStage) {
                    if (xk + (int)xp[0] * 8 >= klen) o0 = kOutOfRange;
                    if (xk + (int)xp[1] * 8 >= klen) o1 = kOutOfRange;
                }
                xk = klen - xk < kStage ? klen : xk + kStage;
            }
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(own + buf * Sh::kXBytes + i * 1024), 16, (i & 1 ? o1 : o0) + (uint32_t)(i >> 1) * 8u * row_x, 0, 0, 0);
        };
        const uint32_t xa0 = (uint32_t)l32 * 256u, x7 = (uint32_t)l32 & 7u;
        auto read_a = [&](int buf, int rt, int ks) {
            const uint32_t piece = (uint32_t)(2 * ks + half) ^ x7;
            return *reinterpret_cast<const uint4_t *>(own + buf * Sh::kXBytes + rt * 8192 + xa0 + piece * 16u);
        };

        // ---- weights, scales, zero points: registers, kRing stages; the lane's columns are 2 l32 and 2 l32 + 1 of the tile ----
        const int col = col0 + 2 * l32;
        // (The offsets of columns past N begin at 2^31.  A slice of few long groups may be one wave's run, up to 2 GiB of weights: then they pass 2^32 and
        // come back as offsets into the run.  The descriptor bounds them, and what they read belongs to columns that are not stored.)
        uint32_t vw = col < a.N ? (uint32_t)half * row_w + (uint32_t)col * 4u : kOutOfRange;
        uint32_t vs = col < a.N ? (uint32_t)col * 2u : kOutOfRange;
        uint32_t vz = col < a.N ? (uint32_t)(col >> 3) * 4u : kOutOfRange;
        const uint32_t zsh = (uint32_t)(col & 7) * 4u;
        uint2_t wq[kRing][kSteps];
        uint32_t sq[kRing][kSegs], zq[kRing][kSegs];
        int srem = 0;  // k into the group at the next stage (groups longer than a stage)
        auto load_w = [&](int place, int i) {  // load i of Sh::kWLoads
            if (i < 2 * kSegs) {
                const uint32_t e = (uint32_t)i >> 1;
                if (i & 1) zq[place][e] = __builtin_amdgcn_raw_buffer_load_b32(rz, vz + e * row_z, 0, 0);
                else sq[place][e] = __builtin_amdgcn_raw_buffer_load_b32(rs, vs + e * row_s, 0, 0);
                if (i == 2 * kSegs - 1) {
                    uint32_t ds = kSegs * row_s, dz = kSegs * row_z;
                    if (SEG == kStage) {  // the group may be several stages long
                        srem += kStage;
                        if (srem < a.group) ds = dz = 0u;
                        else srem = 0;
                    }
                    vs += ds;
                    vz += dz;
                }
            } else {
                const int ks = i - 2 * kSegs;
                wq[place][ks] = __builtin_amdgcn_raw_buffer_load_b64(rw, vw + (uint32_t)ks * 2u * row_w, 0, 2);  // nontemporal
                if (ks == kSteps - 1) vw += 16u * row_w;
            }
        };

        typedef StageScales<Op, kSegs> Scales;
        auto scales_of = [&](int place, Scales &g) {
#pragma unroll
            for (int e = 0; e < kSegs; ++e) g.set(e, sq[place][e], (zq[place][e] | zfill) >> zsh);
        };

        const typename Op::Consts consts = Op::consts();
        float16_t part[2];
#pragma unroll
        for (int i = 0; i < 16; ++i) part[0][i] = part[1][i] = 0.f;
        const float16_t zero16 = part[0];
        uint4_t A[RT][kSteps], B[2][kSteps];
        typename Op::Tmp tmp;

        // the stages before the loop, each one's weights ahead of its X: they come from further away
        static_range<0, kRing>([&](auto s_) {
            constexpr int s = decltype(s_)::value;
            static_range<0, Sh::kWLoads>([&](auto i) { load_w(s, i); });
            asm volatile("" ::: "memory");
            if constexpr (s < Sh::kBuffers) static_range<0, Sh::kXLoads>([&](auto i) { fetch_x(s, i); });
            asm volatile("" ::: "memory");
        });
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(Sh::kWaitFirst) : "memory");
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ks = 0; ks < kSteps; ++ks) A[rt][ks] = read_a(0, rt, ks);
        Scales cur, nxt;
        scales_of(0, cur);
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks)
#pragma unroll
            for (int p = 0; p < Op::kParts; ++p) Op::unpack(p, wq[0][ks][0], cur.z[0][ks / kStepsPerSeg], consts, tmp, B[0][ks]);

        int buf = 0;
        float s_prev = 0.f;
        // One stage from ring place R.  One slot per MFMA; the compiler may not move anything from slot to slot.
        auto do_stage = [&](auto place) {
            constexpr int R = decltype(place)::value, RN = (R + 1) % kRing;
            const int nbuf = buf + 1 == Sh::kBuffers ? 0 : buf + 1;
            for_each_constant(std::make_integer_sequence<int, kTiles * kSteps>{}, [&](auto slot_) {
                constexpr int slot = decltype(slot_)::value;
                typedef StageSlot<slot, RT, SEG> Slot;
                constexpr int ct = Slot::ct, rt = Slot::rt, ks = Slot::ks;
                if constexpr (slot == RT * kSteps) {
                    // The next stage's X has landed when at most the operations asked for after it are on their way: X of
                    // kBuffers - 1 stages, weights of as many.
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(Sh::kWait) : "memory");
                }
                part[Slot::pp] = Op::mfma(A[rt][ks], B[ct][ks], Slot::kFirst ? zero16 : part[Slot::pp]);
                if constexpr (ct == 1) A[rt][ks] = read_a(nbuf, rt, ks);
                step_and_unpack<Op, Slot>(tot, part, s_prev, cur, nxt, consts, tmp, B, [&](auto w) {
                    if constexpr (ct == 0) return wq[R][w][1];
                    else return wq[RN][w][0];
                });
                if constexpr (slot == RT * kSteps - 1) scales_of(RN, nxt);
                // X of the stage kBuffers on, into the buffer whose stage is all in registers, beside the first half's MFMAs;
                // the weights kRing on, into the registers the first half has emptied, beside the first ones of the second.
                if constexpr (slot == 1) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // in registers: it has arrived
                if constexpr (ct == 0 && slot >= 1) {
                    constexpr int n = RT * kSteps - 1, i = slot - 1;
                    static_range<i * Sh::kXLoads / n, (i + 1) * Sh::kXLoads / n>([&](auto q) { fetch_x(buf, q); });
                }
                if constexpr (ct == 1 && rt == 0) {
                    static_range<ks * Sh::kWLoads / kSteps, (ks + 1) * Sh::kWLoads / kSteps>([&](auto q) { load_w(R, q); });
                }
                if constexpr (slot == kTiles * kSteps - 1) asm volatile("" ::: "memory");  // the loads of a stage stay in it
                __builtin_amdgcn_sched_barrier(0);
            });
            cur = nxt;
            buf = nbuf;
        };
        // (every way round the loop passes all ring places, so that the compiler knows which loads are on their way at each)
        int left = stages;
        auto more = [&](auto place) {
            do_stage(place);
            return --left > 0;
        };
        while (all_constants(std::make_integer_sequence<int, kRing>{}, more)) {
        }
        // the fetches past the run's end write into this wave's LDS too: they must have landed before the final sums
        // reuse the space
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        constexpr int kLast = (kTiles * kSegs - 1) & 1;
#pragma unroll
        for (int i = 0; i < 16; ++i) tot[kTiles - 1][i] = __builtin_fmaf(s_prev, part[kLast][i], tot[kTiles - 1][i]);
    }

    // Phase 3 inside the workgroup: the waves exchange their sums in the layout the registers have.  The 16 RT pieces of a
    // lane (row block, element: two neighbouring columns) are dealt out to the four waves, 4 RT neighbouring ones each; a
    // wave writes the pieces it does not own into its own staging space (nobody else ever touched it, and its loads have
    // landed: no barrier before), and after one barrier adds up its pieces, in the order of the waves whoever the owner
    // is.  Lane (half, l32), element i: row 8 (i / 4) + 4 half + i mod 4 of its row block.
    typedef float float2_v __attribute__((ext_vector_type(2)));
    float2_v *const space = reinterpret_cast<float2_v *>(own);
    const bool accumulate = finish == kFinishAccumulator;
#pragma unroll
    for (int u = 0; u < 16 * RT; ++u)
        if (accumulate || u / (4 * RT) != wave) space[u * 64 + lane] = (float2_v){tot[u >> 4][u & 15], tot[RT + (u >> 4)][u & 15]};
    __syncthreads();
    if (accumulate) {
        // one atomic add per output: consecutive lanes on consecutive outputs (w4a16_finish.h); a wave's share of the
        // pieces is 8 RT rows of 64 columns
        const int col = col0 + lane;
        unsigned long long total[8 * RT];  // all on their way before the first is looked at
#pragma unroll
        for (int i = 0; i < 8 * RT; ++i) {
            const int r = 8 * RT * wave + i, u = r >> 1, m = m0 + 32 * (u >> 4) + 8 * ((u & 15) >> 2) + 4 * (r & 1) + (u & 3);
            total[i] = 0ull;
            if (m >= a.M || col >= a.N) continue;
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) v += reinterpret_cast<const float *>(smem + w * Sh::kWaveBytes)[u * 128 + (r & 1) * 64 + lane];
            const bool nan = v != v;
            total[i] = add_slice_value(sync + (size_t)m * a.N + col, to_fixed(nan ? 0.f : v), nan);
        }
#pragma unroll
        for (int i = 0; i < 8 * RT; ++i) {
            const int r = 8 * RT * wave + i, u = r >> 1, m = m0 + 32 * (u >> 4) + 8 * ((u & 15) >> 2) + 4 * (r & 1) + (u & 3);
            const size_t out = (size_t)m * a.N + col;
            if (m < a.M && col < a.N) finish_slice<Act>(sync + out, total[i], a.split, a.Y + out);
        }
        return;
    }
    const int col = col0 + 2 * l32;
#pragma unroll
    for (int u = 0; u < 16 * RT; ++u) {
        if (u / (4 * RT) != wave) continue;  // uniform
        float2_v v = {0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w == wave) v += (float2_v){tot[u >> 4][u & 15], tot[RT + (u >> 4)][u & 15]};
            else v += reinterpret_cast<const float2_v *>(smem + w * Sh::kWaveBytes)[u * 64 + lane];
        }
        const int m = m0 + 32 * (u >> 4) + 8 * ((u & 15) >> 2) + 4 * half + (u & 3);
        if (m >= a.M || col >= a.N) continue;  // N is a multiple of 8: the two columns are inside together
        const size_t out = (size_t)m * a.N + col;
        if (finish == kFinishDirect)
            *reinterpret_cast<uint32_t *>(a.Y + out) = Act::pack2(v[0], v[1]);
        else
            store_partial(a.partials + (size_t)slice * a.M * a.N + out, v[0], v[1]);
    }
}

template <typename Op, int RT, int SEG>
hipError_t launch(const GemmArgs &a, int finish, unsigned long long *sync, hipStream_t stream)
{
    typedef Tall<RT, SEG> Sh;
    const int ntiles = (a.N + kTileCols - 1) / kTileCols;
    const int row_blocks = (a.M + Sh::kRows - 1) / Sh::kRows;
    long long grid;
    const Place where = place((long long)ntiles * a.split, row_blocks, &grid);
    if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&tile_tall_kernel<Op, RT, SEG>), hipFuncAttributeMaxDynamicSharedMemorySize, Sh::kLds);  // beyond the default dynamic-LDS allowance
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((tile_tall_kernel<Op, RT, SEG>), dim3((unsigned)grid), dim3(64 * kWaves), Sh::kLds, stream, a, finish, sync, where);
    return hipGetLastError();
}

template <typename Op, int RT>
hipError_t launch_seg(const GemmArgs &a, int finish, unsigned long long *sync, hipStream_t stream)
{
    if (a.group % 128 == 0) return launch<Op, RT, 128>(a, finish, sync, stream);
    return a.group == 64 ? launch<Op, RT, 64>(a, finish, sync, stream) : launch<Op, RT, 32>(a, finish, sync, stream);
}

}  // namespace

hipError_t launch_tile_tall(const GemmArgs &a, int finish, unsigned long long *sync, hipStream_t stream)
{
    if (!panel_takes(a.group) || !finish_args_ok(a, finish, sync)) return hipErrorInvalidValue;
    const unsigned long long rows = (unsigned long long)a.groups_per_split * (a.group / 8);
    if (rows * a.N * 4ull >= 0x7F000000ull) return hipErrorInvalidValue;  // slice-relative 32-bit buffer offsets
    if ((unsigned long long)a.M * a.K * 2ull >= 0x7F000000ull) return hipErrorInvalidValue;
    return a.bf16 ? launch_seg<ExactBF16, 2>(a, finish, sync, stream) : launch_seg<ExactF16, 2>(a, finish, sync, stream);
}

}  // namespace w4a16
