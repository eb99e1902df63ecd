// W4A16 multiply, PAIR form of the TILE family (the scheduler's choice for many shapes of 17 to some hundred rows, see use_pair):
// one workgroup of eight waves per (128 columns, 32 RT rows of X, K slice), RT = 1 or 2.  Two waves share a quarter of the
// slice's K, each with half of the columns, so that a wave has 32 RT x 64 of the result and every SIMD has two waves.
//
// What bounds such a multiply is instruction issue.  Unpack and Eq. 2's step are 7 vector instructions per MFMA 32x32x16 at 64 rows (10 with
// BF16), and beside them come the reads, fetches, waits and scalar instructions.  A wave alone on its SIMD (w4a16_panel.hip,
// w4a16_tile_tall.hip) issues one after the other: 66 cycles per MFMA measured at 64 rows.  Of two waves one takes the slots
// that the other leaves: in a probe an MFMA and 8 vector instructions take 54 cycles of a lone wave and 45 of two.  So:
//   - 256 registers per wave: 64 totals, 64 part sums, operands of two steps; X and weights in LDS;
//   - the step of 16 k is the unit of the order: its four MFMAs, beside them the reads and the unpack of the next step;
//   - X is shared by two waves and read for 128 columns, half the traffic from the L2 of a 64-column tile.  A compute unit takes a load in
//     16 cycles whatever its width (measured; an LDS load of 4 bytes a lane 32): hence 16 bytes a lane for X and weights both;
//   - the loads are spread over the slots between two barriers: all of them behind the barrier, waves that ask for more than the 64
//     bytes a cycle that a compute unit takes in wait in line, 1700 cycles per 128 k;
//   - 16-byte pieces of X sit rotated by half the row number: a read of sixteen rows falls into all 64 banks.
// Per 128 k of both waves of a SIMD 4100 cycles (64 MFMAs), 3000 without the loads.  Cold, us, against the plan before: M = 100, K = 14336, N = 4096 26.5 -> 22.9;
// M = 256, K = N = 8192 42.5 -> 37.3; M = 44, K = 27904, N = 2080 26.0 -> 18.9; M = 183, K = 3456, N = 8392 26.7 -> 19.6; M = 128 and 64, K = N = 8192 no faster.
// Arithmetic: products x (q - z) exact, sums over a group in FP32 in the MFMA, times s in FP32: as in w4a16_panel.hip.
#include "w4a16_finish.h"
#include "w4a16_internal.h"
#include "w4a16_wide_ops.h"

namespace w4a16 {
namespace {

constexpr int kWaveCols = 64;
constexpr int kColWaves = 2, kKWaves = 4;
constexpr int kWaves = kColWaves * kKWaves;
constexpr int kChunk = 64;                    // k that a wave works on between two barriers
constexpr int kChunkSteps = kChunk / 16;
constexpr int kXRing = 3, kWRing = 4;         // chunks of X and of weights in LDS

// Sizes for RT blocks of 32 rows and SEG k per step of scales.
template <int RT, int SEG>
struct Pair {
    static constexpr int kRows = 32 * RT;
    static constexpr int kSegs = SEG < kChunk ? kChunk / SEG : 1;     // steps of scales in a chunk
    static constexpr int kXBytes = kRows * kChunk * 2;                // X of a chunk, for the two waves that share it
    static constexpr int kXLoads = kXBytes / 1024 / kColWaves;        // wave-wide loads of it per wave
    static constexpr int kWBytes = kChunk / 8 * kWaveCols * 4;        // a wave's packed weights of a chunk
    static constexpr int kWLoads = kWBytes / 1024;
    static constexpr int kXAll = kKWaves * kXRing * kXBytes;
    static constexpr int kSumBytes = 16 * RT * 64 * 8;                // a wave's sums
    static constexpr int kNeed = kXAll + kWaves * kWRing * kWBytes;
    static constexpr int kLds = kNeed > kWaves * kSumBytes ? kNeed : kWaves * kSumBytes;
    static_assert(kLds <= 160 * 1024, "the LDS of a compute unit");
    // loads of scales and zero points for chunk c: a segment of 128 k begins with an even chunk
    static constexpr int scale_loads(int c) { return SEG > kChunk ? (c & 1 ? 0 : 2) : 2 * kSegs; }
};

template <typename Op, int RT, int SEG>
__global__ __launch_bounds__(64 * kWaves, 2) void pair_kernel(const GemmArgs a, const int finish, const int row_blocks)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    typedef Pair<RT, SEG> Sh;
    typedef typename Op::Act Act;
    constexpr int kTiles = 2 * RT, kSegs = Sh::kSegs;  // 32 x 32 result tiles of a wave: (column half, row block)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cw = wave % kColWaves, kw = wave / kColWaves;
    const int l32 = lane & 31, half = lane >> 5;

    // workgroup -> (column tile, K slice, row block)
    const int ntiles = (a.N + kPairCols - 1) / kPairCols;
    const int units = ntiles * a.split;
    int unit, rb;
    if (!place_in_eighths(blockIdx.x, gridDim.x, units, row_blocks, &unit, &rb)) return;
    const int slice = unit / ntiles, tile = unit - slice * ntiles;
    const int m0 = rb * Sh::kRows, col = tile * kPairCols + cw * kWaveCols + 2 * l32;

    // The slice's k, and the run of it that this wave and its partner work on: whole units of two chunks, the first
    // runs one unit more.  Every wave goes as many times round the loop as the longest run has chunks.
    constexpr int kUnit = 2 * kChunk;
    const int sbeg = slice * a.groups_per_split * a.group;
    const int send = a.K - sbeg < a.groups_per_split * a.group ? a.K : sbeg + a.groups_per_split * a.group;
    const int run_units = (send - sbeg + kUnit - 1) / kUnit;
    const int per = run_units / kKWaves, extra = run_units - per * kKWaves;
    const int kbeg = sbeg + (per * kw + (kw < extra ? kw : extra)) * kUnit;
    int kend = kbeg + (per + (kw < extra ? 1 : 0)) * kUnit;
    if (kend > send) kend = send;
    const int klen = kend > kbeg ? kend - kbeg : 0;  // a multiple of 32
    const int chunks = (per + (extra ? 1 : 0)) * (kUnit / kChunk);

    // Every descriptor ends where the run (or the matrix) ends: loads past it return zeros and move nothing.
    const int rows_here = a.M - m0 < Sh::kRows ? a.M - m0 : Sh::kRows;
    const uint32_t row_x = (uint32_t)a.K * 2u, row_w = (uint32_t)a.N * 4u, row_s = (uint32_t)a.N * 2u, row_z = (uint32_t)(a.N >> 3) * 4u;
    const int grp0 = kbeg / a.group;
    const uint32_t ngroups = klen ? (uint32_t)((kend - 1) / a.group - grp0 + 1) : 0u;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.X) + (size_t)m0 * a.K + (klen ? kbeg : 0), 0, klen ? (uint32_t)rows_here * row_x - (uint32_t)kbeg * 2u : 0u, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.Wp) + (klen ? (size_t)(kbeg >> 3) * a.N : 0), 0, (uint32_t)(klen >> 3) * row_w, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.scales) + (klen ? (size_t)grp0 * a.N : 0), 0, ngroups * row_s, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.Zp) + (klen && a.Zp ? (size_t)grp0 * (a.N >> 3) : 0), 0, zero_point_bytes(a.Zp, ngroups * row_z), kRawBuffer);
    const uint32_t zfill = symmetric_fill(a.Zp);

    // ---- X: straight from global memory into LDS; a wave-wide load puts lane l's 16 bytes at base + 16 l ----
    // Eight rows of 128 bytes per load; lane l fetches piece (l mod 8) ^ (row / 2 mod 8) of row l / 8, so that the MFMA's operand
    // reads (the same piece of sixteen consecutive rows, 256 bytes of banks to two rows) fall into different banks.
    uint32_t xpiece[2], vx[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {  // by the parity of the load: row / 2 mod 8 = 4 p + lane / 16
        xpiece[p] = ((uint32_t)lane & 7u) ^ (4u * (uint32_t)p + ((uint32_t)lane >> 4));
        vx[p] = (uint32_t)(cw * Sh::kXLoads * 8 + (lane >> 3)) * row_x + xpiece[p] * 16u;
    }
    int xleft = klen;  // k of the run from the next chunk to fetch on
    uint32_t ox[2] = {0, 0};
    unsigned char *const lds_x = smem + kw * kXRing * Sh::kXBytes;
    unsigned char *const lds_w = smem + Sh::kXAll + wave * kWRing * Sh::kWBytes;
    uint32_t xto = 0, wto = 0;  // ring places of the next fetch, in bytes
    auto fetch_x = [&](int i) {  // load i of Sh::kXLoads; past the run only zeros, for the waits' count
        if (i == 0) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                ox[p] = vx[p];
                if (xleft < kChunk && (int)xpiece[p] * 8 >= xleft) ox[p] = kOutOfRange;  // the run ends inside this chunk or before it
                vx[p] += kChunk * 2u;
            }
            xleft = xleft < kChunk ? 0 : xleft - kChunk;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(lds_x + xto + (cw * Sh::kXLoads + i) * 1024), 16, ox[i & 1] + (uint32_t)i * 8u * row_x, 0, 0, 0);
        if (i == Sh::kXLoads - 1) xto = xto == (kXRing - 1) * Sh::kXBytes ? 0u : xto + Sh::kXBytes;
    };
    // ---- weights, likewise: four packed rows of the wave's 64 columns per load (not nontemporal as in the other forms: M = 100, K = 14336,
    // N = 4096 24.7 us so and 23.7 without, M = 50, groups of 64 20.1 and 19.5; at four row blocks and more within 1 %) ----
    const uint32_t wcol = (uint32_t)(tile * kPairCols + cw * kWaveCols) + 4u * ((uint32_t)lane & 15u);
    uint32_t vw = wcol < (uint32_t)a.N ? ((uint32_t)lane >> 4) * row_w + wcol * 4u : kOutOfRange;
    auto fetch_w = [&](int i) {  // load i of Sh::kWLoads
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr_t)(lds_w + wto + i * 1024), 16, vw + (uint32_t)i * 4u * row_w, 0, 0, 0);
        if (i == Sh::kWLoads - 1) {
            if (vw != kOutOfRange) vw += 8u * row_w;
            wto = wto == (kWRing - 1) * Sh::kWBytes ? 0u : wto + Sh::kWBytes;
        }
    };
    // ---- reads from LDS ----
    uint32_t xat[kChunkSteps];
#pragma unroll
    for (int ks = 0; ks < kChunkSteps; ++ks) xat[ks] = (uint32_t)l32 * 128u + (((uint32_t)(2 * ks + half) ^ (((uint32_t)l32 >> 1) & 7u)) * 16u);
    auto read_a = [&](uint32_t from, int rt, int ks) { return *reinterpret_cast<const uint4_t *>(lds_x + from + xat[ks] + rt * 4096); };
    const uint32_t wat = (uint32_t)half * 256u + (uint32_t)l32 * 8u;
    auto read_w = [&](uint32_t from, int ks) { return *reinterpret_cast<const uint2_t *>(lds_w + from + wat + ks * 512); };

    // ---- scales and zero points: registers, two chunks; the lane's columns are 2 l32 and 2 l32 + 1 of the wave's 64 ----
    uint32_t vs = col < a.N ? (uint32_t)col * 2u : kOutOfRange;
    uint32_t vz = col < a.N ? (uint32_t)(col >> 3) * 4u : kOutOfRange;
    const uint32_t zsh = (uint32_t)(col & 7) * 4u;
    uint32_t sq[2][kSegs], zq[2][kSegs];
    int srem = kbeg - grp0 * a.group;  // k into the group at the next segment (groups longer than one)
    auto load_s = [&](auto place_, auto i_) {  // load i of Sh::scale_loads
        constexpr int place = decltype(place_)::value, i = decltype(i_)::value, e = i >> 1;
        if constexpr (i & 1) zq[place][e] = __builtin_amdgcn_raw_buffer_load_b32(rz, vz + (uint32_t)e * row_z, 0, 0);
        else sq[place][e] = __builtin_amdgcn_raw_buffer_load_b32(rs, vs + (uint32_t)e * row_s, 0, 0);
        if constexpr (i == Sh::scale_loads(place) - 1) {
            uint32_t ds = kSegs * row_s, dz = kSegs * row_z;
            if constexpr (SEG > kChunk) {  // the group may be several segments long
                srem += SEG;
                if (srem < a.group) ds = dz = 0u;
                else srem = 0;
            }
            if (vs != kOutOfRange) {
                vs += ds;
                vz += dz;
            }
        }
    };

    const typename Op::Consts consts = Op::consts();
    float16_t tot[kTiles], part[kTiles];
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) tot[t][i] = part[t][i] = 0.f;
    float16_t zero16;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero16[i] = 0.f;
    uint4_t A[2][RT], B[2][2];  // by the parity of the step
    typename Op::Tmp tmp;
    float s[2][kSegs], s_prev[2] = {0.f, 0.f};
    typename Op::Zero z[2][kSegs];
    auto set_scales = [&](auto place_) {
        constexpr int place = decltype(place_)::value;
#pragma unroll
        for (int e = 0; e < kSegs; ++e) {
            H2 h;
            h.u = sq[place][e];
            const uint32_t zw = (zq[place][e] | zfill) >> zsh;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                s[c][e] = Op::scale(h.h[c]);
                z[c][e] = Op::zero(zw >> (4 * c));
            }
            // converted here: put off until they are used, they would share their registers with the next ones, whose loads would be
            // waited for as soon as they are asked for
            asm volatile("" : "+v"(s[0][e]), "+v"(s[1][e]));
        }
    };

    typedef std::integral_constant<int, 0> Even;
    typedef std::integral_constant<int, 1> Odd;
    auto fence = [] { asm volatile("" ::: "memory"); };
    // What is asked for between the barrier in chunk h and the one in chunk h + 1, R: the parity of h: X and scales of chunk h + 3,
    // weights of h + 4.  Spread over the slots between the two: a compute unit takes in 64 bytes per cycle, and waves that ask
    // for more at once wait for it (all of it behind the barrier: 1700 cycles per 128 k).
    constexpr int kSlots = kChunkSteps * kTiles;
    auto fetch_batch = [&](auto place, auto pos_) {
        constexpr int R = decltype(place)::value, pos = decltype(pos_)::value;
        constexpr int nx = Sh::kXLoads, ns = nx + (SEG > kChunk && R == 0 ? 0 : Sh::scale_loads(0)), n = ns + Sh::kWLoads;
        static_range<pos * n / kSlots, (pos + 1) * n / kSlots>([&](auto i_) {
            constexpr int i = decltype(i_)::value;
            if constexpr (i < nx) fetch_x(i);
            else if constexpr (i < ns) load_s(std::integral_constant<int, R ^ 1>{}, std::integral_constant<int, i - nx>{});
            else fetch_w(i - ns);
            fence();
        });
    };
    auto all_w = [&] { static_range<0, Sh::kWLoads>([&](auto i) { fetch_w(i); }); };
    auto all_x = [&] { static_range<0, Sh::kXLoads>([&](auto i) { fetch_x(i); }); };
    constexpr int kBatch = Sh::kXLoads + Sh::scale_loads(0) + Sh::kWLoads;  // of an odd chunk
    // before the loop: what is asked for ahead of the last step of chunk -1
    all_x(); fence();
    static_range<0, Sh::scale_loads(0)>([&](auto i) { load_s(Even(), i); });
    fence(); all_w(); fence(); all_w(); all_x(); fence();
    static_range<0, Sh::scale_loads(1)>([&](auto i) { load_s(Odd(), i); });
    fence(); all_w(); fence();
    static_range<0, kTiles>([&](auto pos) { fetch_batch(Odd(), pos); });
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(Sh::scale_loads(1) + 2 * Sh::kWLoads + Sh::kXLoads + kTiles * kBatch / kSlots) : "memory");
    __builtin_amdgcn_s_barrier();
    fence();
    uint32_t xfrom = 0, wfrom = 0;  // ring places of the chunk in use
    uint2_t w[2];  // words, by the parity of the step
    w[0] = read_w(wfrom, 0);
    w[1] = read_w(wfrom, 1);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) A[0][rt] = read_a(xfrom, rt, 0);
    set_scales(Even());
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int p = 0; p < Op::kParts; ++p) Op::unpack(p, w[0][ct], z[ct][0], consts, tmp, B[0][ct]);

    // One chunk, R: its parity.  One slot per MFMA; the compiler may not move anything from slot to slot.  A step's operands are
    // read and unpacked beside the MFMAs of the step before, its words read one step earlier still.
    auto do_chunk = [&](auto place) {
        constexpr int R = decltype(place)::value;
        const uint32_t xnext = xfrom == (kXRing - 1) * Sh::kXBytes ? 0u : xfrom + Sh::kXBytes, wnext = wfrom == (kWRing - 1) * Sh::kWBytes ? 0u : wfrom + Sh::kWBytes;
        for_each_constant(std::make_integer_sequence<int, kChunkSteps * kTiles>{}, [&](auto slot_) {
            constexpr int slot = decltype(slot_)::value, ks = slot / kTiles, t = slot % kTiles, ct = t / RT, rt = t % RT;
            constexpr bool kLastStep = ks == kChunkSteps - 1;
            constexpr int kn = kLastStep ? 0 : ks + 1;  // the step after this one: in this chunk, or the first of the next
            constexpr bool kFirst = SEG > kChunk ? (R == 0 && ks == 0) : ks % (SEG / 16) == 0;  // of its segment
            if constexpr (kFirst) {  // Eq. 2's step of the segment before
#pragma unroll
                for (int i = 0; i < 16; ++i) tot[t][i] = __builtin_fmaf(s_prev[ct], part[t][i], tot[t][i]);
            }
            part[t] = Op::mfma(A[ks & 1][rt], B[ks & 1][ct], kFirst ? zero16 : part[t]);
            if constexpr (kFirst && t == kTiles - 1) {
                constexpr int e = SEG < kChunk ? ks / (SEG / 16) : 0;
                s_prev[0] = s[0][e];
                s_prev[1] = s[1][e];
            }
            constexpr int parts = 2 * Op::kParts;
            if constexpr (t < RT) A[(ks & 1) ^ 1][t] = read_a(kLastStep ? xnext : xfrom, t, kn);
            static_range<t * parts / kTiles, (t + 1) * parts / kTiles>([&](auto p_) {
                constexpr int p = decltype(p_)::value, c = p / Op::kParts;
                Op::unpack(p % Op::kParts, w[kn & 1][c], z[c][SEG < kChunk ? kn / (SEG / 16) : 0], consts, tmp, B[(ks & 1) ^ 1][c]);
            });
            fetch_batch(std::integral_constant<int, kLastStep ? R : R ^ 1>{}, std::integral_constant<int, (slot + kTiles) % kSlots>{});
            if constexpr (ks == kChunkSteps - 2 && t == kTiles - 1) {
                // The next chunk's weights (asked for three chunks ago) and X (two) have landed when at most what was asked for after
                // that X is on its way.  Behind the barrier X has for every wave, and no wave reads this chunk's X any more (the
                // operands of its last step are in registers).
                constexpr int kLater = Sh::scale_loads(0) + Sh::scale_loads(1) + 2 * Sh::kWLoads + Sh::kXLoads;
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kLater) : "memory");
                __builtin_amdgcn_s_barrier();
                fence();
                if constexpr (SEG <= kChunk || R == 1) set_scales(std::integral_constant<int, R ^ 1>{});
            }
            if constexpr (t == (ks == kChunkSteps - 2 ? kTiles - 1 : 0)) w[ks & 1] = read_w(ks < kChunkSteps - 2 ? wfrom : wnext, (ks + 2) % kChunkSteps);
            __builtin_amdgcn_sched_barrier(0);
        });
        xfrom = xnext;
        wfrom = wnext;
    };
    for (int left = chunks; left > 0; left -= 2) {
        do_chunk(Even());
        do_chunk(Odd());
    }
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) tot[t][i] = __builtin_fmaf(s_prev[t / RT], part[t][i], tot[t][i]);

    // Phase 3 inside the workgroup: the four waves of a column half exchange their sums in the layout the registers have.
    // The 16 RT pieces of a lane (row block, element: two neighbouring columns) are dealt out to them, 4 RT neighbouring ones
    // each; a wave writes the pieces it does not own into LDS, and after a barrier adds up its own, in the order of
    // the waves whoever the owner is.  Lane (half, l32), element i: row 8 (i / 4) + 4 half + i mod 4 of its row block.
    // The fetches past the run's end write into LDS too: all have to have landed before it is used for the sums.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    typedef float float2_v __attribute__((ext_vector_type(2)));
    float2_v *const space = reinterpret_cast<float2_v *>(smem + wave * Sh::kSumBytes);
#pragma unroll
    for (int u = 0; u < 16 * RT; ++u)
        if (u / (4 * RT) != kw) space[u * 64 + lane] = (float2_v){tot[u >> 4][u & 15], tot[RT + (u >> 4)][u & 15]};
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16 * RT; ++u) {
        if (u / (4 * RT) != kw) continue;  // uniform
        float2_v v = {0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kKWaves; ++w) {
            if (w == kw) v += (float2_v){tot[u >> 4][u & 15], tot[RT + (u >> 4)][u & 15]};
            else v += reinterpret_cast<const float2_v *>(smem + (w * kColWaves + cw) * Sh::kSumBytes)[u * 64 + lane];
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
hipError_t launch(const GemmArgs &a, int finish, hipStream_t stream)
{
    typedef Pair<RT, SEG> Sh;
    const int ntiles = (a.N + kPairCols - 1) / kPairCols;
    const int row_blocks = (a.M + Sh::kRows - 1) / Sh::kRows;
    const long long grid = eighths_grid((long long)ntiles * a.split, row_blocks);
    if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&pair_kernel<Op, RT, SEG>), hipFuncAttributeMaxDynamicSharedMemorySize, Sh::kLds);  // beyond the default dynamic-LDS allowance
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((pair_kernel<Op, RT, SEG>), dim3((unsigned)grid), dim3(64 * kWaves), Sh::kLds, stream, a, finish, row_blocks);
    return hipGetLastError();
}

template <typename Op, int RT>
hipError_t launch_seg(const GemmArgs &a, int finish, hipStream_t stream)
{
    if (a.group % 128 == 0) return launch<Op, RT, 128>(a, finish, stream);
    return a.group == 64 ? launch<Op, RT, 64>(a, finish, stream) : launch<Op, RT, 32>(a, finish, stream);
}

template <typename Op>
hipError_t launch_rows(const GemmArgs &a, int finish, int rows_x, hipStream_t stream)
{
    return rows_x == 32 ? launch_seg<Op, 1>(a, finish, stream) : launch_seg<Op, 2>(a, finish, stream);
}

}  // namespace

hipError_t launch_pair(const GemmArgs &a, int finish, int rows_x, hipStream_t stream)
{
    if (!panel_takes(a.group) || (rows_x != 32 && rows_x != 64) || finish == kFinishAccumulator || !finish_args_ok(a, finish, nullptr)) return hipErrorInvalidValue;
    const unsigned long long rows = (unsigned long long)a.groups_per_split * (a.group / 8);
    if (rows * a.N * 4ull >= 0x7F000000ull) return hipErrorInvalidValue;  // slice-relative 32-bit buffer offsets
    if ((unsigned long long)a.M * a.K * 2ull >= 0x7F000000ull) return hipErrorInvalidValue;
    return a.bf16 ? launch_rows<ExactBF16>(a, finish, rows_x, stream) : launch_rows<ExactF16>(a, finish, rows_x, stream);
}

}  // namespace w4a16
