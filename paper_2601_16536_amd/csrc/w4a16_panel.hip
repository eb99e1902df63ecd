// W4A16 multiply for prompts, and from 17 rows on for batches over a long K or many columns: one workgroup of four
// waves per (32 RT rows of X, 256 columns, K slice), every wave alone on its SIMD with 32 RT x 64 of the result; RT = 4, and
// 1 to 4 in the last row block.
//
// What bounds a multiply of many rows is the matrix pipe, then the power limit (the clock falls from 2.4 to about 1.7 GHz
// under it); what the 64 x 64 form (w4a16_tile_wide.hip) spent its time on was the vector instructions around each MFMA, a
// word's unpack being used for 64 rows only, and X, which every wave fetched for itself.  Here:
//   - a word is unpacked once for 128 rows: 10 vector instructions (17 for BF16) for 4 MFMAs 32x32x16; Eq. 2's step costs 2
//     per MFMA more.  A wave can issue 5 beside an MFMA's 32 cycles for nothing (measured: 35.5 cycles; 6: 40);
//   - the operand is q - z, exact, in the order of k, so that X can go from global memory straight into LDS; it is unpacked by
//     the wave that uses it, from its own 64 columns: the weights cross no barrier and no wave repeats another's work;
//   - the four waves share X: a stage (128 k) of all rows in LDS, read into registers once (128 of the 256 accumulation
//     registers) and used for both halves of the wave's columns;
//   - one tile of 32 x 32 at a time runs through the stage's eight MFMAs (a chain on one accumulator runs at the full rate:
//     measured, 32 cycles each), so two sets of 16 part sums are enough beside the 128 totals: while one tile's chain runs, the
//     tile before it takes its step tot += s part;
//   - the order of instructions is written down slot by slot, one MFMA each.  Left to the compiler's scheduler the same
//     loop took 243 us where this one takes 224 (M = 2048, K = N = 8192).
// M = 2048, K = N = 8192: 224-232 us = 1.2 PFLOP/s (FP16; BF16 229-243), 656 us before; ten launches one after another under
// the trace, where the power limit sets in: 231 rising to 266 (BF16 271 to 278, the first two 334 and 319).  The vendor's FP16 GEMM on dense weights takes 235-265.  M = 777, K = 4096, N = 11008: 76 us (BF16, cold weights).
// Arithmetic: products x (q - z) are exact in FP32, sums over a group in FP32 in the MFMA, times s in FP32: as in
// w4a16_tile_wide.hip.
#include "w4a16_device.h"
#include "w4a16_internal.h"
#include "w4a16_wide_ops.h"

namespace w4a16 {
namespace {

constexpr int kWaves = 4;
constexpr int kMainRt = kPanelRows / 32;
constexpr int kWaveCols = 64;
constexpr int kCols = kWaves * kWaveCols;
static_assert(kCols == kPanelCols, "the planner's tile");
constexpr int kBuffers = 3;       // stages in LDS: the one in use and two on their way
constexpr int kXcds = 8;
constexpr int kRowGroup = 8;      // row blocks that neighbouring workgroups of an XCD cover before the next column tile

// Sizes for RT blocks of 32 rows and SEG k per step of scales.
template <int RT, int SEG>
struct Panel {
    static constexpr int kRows = 32 * RT;
    static constexpr int kSegs = kStage / SEG;
    static constexpr int kXBytes = kRows * kStage * 2;          // X of a stage
    static constexpr int kXLoads = kXBytes / 1024 / kWaves;     // wave-wide loads of it per wave
    static constexpr int kWBytes = kStage / 8 * kWaveCols * 4;  // a wave's packed weights of a stage
    static constexpr int kWLoads = kWBytes / 1024;
    static constexpr int kSLoads = (kSegs + 1) / 2;             // 32 lanes per scale row of 64 columns
    static constexpr int kSBytes = kSLoads * 256;
    static constexpr int kZBytes = 256;
    static constexpr int kPerStage = kXLoads + kWLoads + kSLoads + 1;
    static constexpr int kStageBytes = kXBytes + kWaves * (kWBytes + kSBytes + kZBytes);
    static constexpr int kLds = kBuffers * kStageBytes;
    static_assert(kLds <= 160 * 1024 && 2 * kPerStage < 64 && (kBuffers + 1) * kStage / 8 <= 64, "LDS of a compute unit, the wait counter's range, and rows of weights asked for ahead");
};

// One workgroup's part: rows m0 .. m0 + 32 RT - 1, 256 columns from tile_col0 on, k from kbeg to kend.  The result goes to
// Y, or as FP32 to `partial` ([rows of the tile or piece][256]).
template <typename Op, int RT, int SEG>
__device__ __forceinline__ void panel(const GemmArgs &a, unsigned char *const smem, const int m0, const int tile_col0, const int kbeg, const int kend, float *const partial)
{
    typedef Panel<RT, SEG> Sh;
    typedef typename Op::Act Act;
    constexpr int kTiles = 2 * RT;               // 32 x 32 result tiles of a wave: (column half, row block)
    constexpr int kStepsPerSeg = SEG / 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int col0 = tile_col0 + wave * kWaveCols;

    const int klen = kend - kbeg;  // a multiple of 32
    const int stages = (klen + kStage - 1) / kStage;

    // Every descriptor ends where the slice (or the matrix) ends: loads past it return zeros and move nothing.
    const int rows_here = a.M - m0 < Sh::kRows ? a.M - m0 : Sh::kRows;
    const uint32_t row_x = (uint32_t)a.K * 2u, row_w = (uint32_t)a.N * 4u, row_s = (uint32_t)a.N * 2u, row_z = (uint32_t)(a.N >> 3) * 4u;
    const int grp0 = kbeg / a.group;
    const uint32_t ngroups = (uint32_t)(klen / a.group);
    __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.X) + (size_t)m0 * a.K + kbeg, 0, (uint32_t)rows_here * row_x - (uint32_t)kbeg * 2u, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.Wp) + (size_t)(kbeg >> 3) * a.N, 0, (uint32_t)(klen >> 3) * row_w, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.scales) + (size_t)grp0 * a.N, 0, ngroups * row_s, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.Zp) + (size_t)grp0 * (a.N >> 3), 0, zero_point_bytes(a.Zp, ngroups * row_z), kRawBuffer);
    const uint32_t zfill = symmetric_fill(a.Zp);

    // ---- addresses of the fetches into LDS: a wave-wide load puts lane l's bytes at base + 16 l (or 4 l) ----
    // X: four rows of 256 bytes per load; lane l fetches 16-byte piece (l mod 16) ^ (row mod 8) of row l / 16, so that the
    // MFMA's operand reads (the same piece of consecutive rows) spread over the banks.
    const uint32_t lr = (uint32_t)lane >> 4, lp = (uint32_t)lane & 15u;
    const uint32_t xrow = (uint32_t)(wave * Sh::kXLoads * 4) + lr;  // row of this wave's first load
    uint32_t xp[2], xg[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        // row mod 8 of load q: 4 ((wave kXLoads + q) mod 2) + lr, and kXLoads is even
        xp[p] = lp ^ (4u * (uint32_t)p + lr);
        xg[p] = (xrow + 4u * (uint32_t)p) * row_x + xp[p] * 16u;
    }
    const uint32_t wcol = (uint32_t)col0 + 4u * lp;
    // Four packed rows per load.  The offsets run on past the slice's end, for the stages asked for ahead: those of columns that exist stay below 2^32 (64 rows of
    // 2^22 columns are 1 GiB) and return zeros.  Those of columns past N begin at 2^31; with 2 GiB of weights they pass 2^32 and come back as offsets into the
    // matrix: the descriptor bounds them, and what they read belongs to columns that are not stored.
    uint32_t vw = wcol < (uint32_t)a.N ? lr * row_w + wcol * 4u : kOutOfRange;
    const uint32_t scol = (uint32_t)col0 + 2u * (uint32_t)l32;
    const uint32_t zcol = (uint32_t)col0 + 8u * ((uint32_t)lane & 7u), zseg = (uint32_t)lane >> 3;
    uint32_t vs = scol < (uint32_t)a.N ? scol * 2u + (uint32_t)half * row_s : kOutOfRange;
    uint32_t vz = zcol < (uint32_t)a.N && zseg < (uint32_t)Sh::kSegs ? zseg * row_z + (zcol >> 3) * 4u : kOutOfRange;
    if (Sh::kSegs == 1 && half) vs = kOutOfRange;

    unsigned char *const lds_w = smem + kBuffers * Sh::kXBytes + wave * kBuffers * Sh::kWBytes;
    unsigned char *const lds_s = smem + kBuffers * (Sh::kXBytes + kWaves * Sh::kWBytes) + wave * kBuffers * (Sh::kSBytes + Sh::kZBytes);

    // Stage `st` of the slice into LDS buffer `buf`, in Sh::kPerStage loads: number i of them.  Past the last stage only
    // zeros arrive, for the waits' count.  Nothing orders these loads but the waits: the compiler may move them between
    // the fences around two barriers, where nobody reads the buffer they fill.
    uint32_t o0 = xg[0], o1 = xg[1];
    int fetched = 0;  // stages asked for
    int srem = 0;     // k into the group at the next stage (groups longer than a stage)
    auto fetch = [&](int buf, int i) {
        if (i < Sh::kXLoads) {
            if (i == 0) {
                const int left = klen - fetched * kStage;  // k from this stage's start to the slice's end
                o0 = xg[0] + (uint32_t)fetched * 256u;
                o1 = xg[1] + (uint32_t)fetched * 256u;
                if constexpr (SEG == kStage) {  // slices are whole stages: past the last one nothing is to be fetched
                    if (left <= 0) rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.X), 0, 0u, kRawBuffer);
                } else if (left < kStage) {  // the slice ends inside this stage: X beyond it must read as zero, also where it is another row's
                    if ((int)xp[0] * 8 >= left) o0 = kOutOfRange;
                    if ((int)xp[1] * 8 >= left) o1 = kOutOfRange;
                }
            }
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(smem + buf * Sh::kXBytes + (wave * Sh::kXLoads + i) * 1024), 16, (i & 1 ? o1 : o0) + (uint32_t)(i >> 1) * 8u * row_x, 0, 0, 0);
        } else if (i < Sh::kXLoads + Sh::kWLoads) {
            const int q = i - Sh::kXLoads;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr_t)(lds_w + buf * Sh::kWBytes + q * 1024), 16, vw + (uint32_t)q * 4u * row_w, 0, 0, 0);
            if (q == Sh::kWLoads - 1) vw += 16u * row_w;
        } else if (i < Sh::kPerStage - 1) {
            const int q = i - Sh::kXLoads - Sh::kWLoads;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(lds_s + buf * (Sh::kSBytes + Sh::kZBytes) + q * 256), 4, vs + (uint32_t)q * 2u * row_s, 0, 0, 0);
        } else {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rz, (lds_ptr_t)(lds_s + buf * (Sh::kSBytes + Sh::kZBytes) + Sh::kSBytes), 4, vz, 0, 0, 0);
            uint32_t ds = Sh::kSegs * row_s, dz = Sh::kSegs * row_z;
            if (SEG == kStage) {  // the group may be several stages long
                srem += kStage;
                if (srem < a.group) ds = dz = 0u;
                else srem = 0;
            }
            vs += ds;
            vz += dz;
            ++fetched;
        }
    };

    // ---- addresses of the reads from LDS ----
    const uint32_t xa0 = (uint32_t)l32 * 256u, x7 = (uint32_t)l32 & 7u;
    const uint32_t zsh = (uint32_t)((2 * l32) & 7) * 4u;  // the lane's two columns are 2 l32 and 2 l32 + 1 of the wave's 64
    auto read_a = [&](int buf, int rt, int ks) {
        const uint32_t piece = (uint32_t)(2 * ks + half) ^ x7;
        return *reinterpret_cast<const uint4_t *>(smem + buf * Sh::kXBytes + rt * 8192 + xa0 + piece * 16u);
    };
    auto read_w = [&](int buf, int ct, int ks) {
        return *reinterpret_cast<const uint32_t *>(lds_w + buf * Sh::kWBytes + (2 * ks + half) * 256 + (2 * l32 + ct) * 4);
    };

    const typename Op::Consts consts = Op::consts();
    float16_t tot[kTiles], part[2];
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) tot[t][i] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) part[0][i] = part[1][i] = 0.f;
    const float16_t zero16 = part[0];
    uint4_t A[RT][kSteps], B[2][kSteps];

    typedef StageScales<Op, Sh::kSegs> Scales;
    uint32_t sraw[Sh::kSegs], zraw[Sh::kSegs];
    auto read_scales_raw = [&](int buf) {
        const unsigned char *const bs = lds_s + buf * (Sh::kSBytes + Sh::kZBytes);
#pragma unroll
        for (int e = 0; e < Sh::kSegs; ++e) {
            sraw[e] = *reinterpret_cast<const uint32_t *>(bs + e * 128 + l32 * 4);
            zraw[e] = *reinterpret_cast<const uint32_t *>(bs + Sh::kSBytes + e * 32 + (l32 >> 2) * 4);
        }
    };
    auto convert_scales = [&](Scales &g) {
#pragma unroll
        for (int e = 0; e < Sh::kSegs; ++e) g.set(e, sraw[e], (zraw[e] | zfill) >> zsh);
    };

#pragma unroll
    for (int b = 0; b < kBuffers; ++b) {
#pragma unroll
        for (int i = 0; i < Sh::kPerStage; ++i) fetch(b, i);
        asm volatile("" ::: "memory");
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * Sh::kPerStage) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    Scales cur, nxt;
    read_scales_raw(0);
    convert_scales(cur);
    typename Op::Tmp tmp;
    uint32_t wv[2][kSteps];  // by the parity of the tile that unpacks them
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks) A[rt][ks] = read_a(0, rt, ks);
#pragma unroll
    for (int ks = 0; ks < kSteps; ++ks) {
        const uint32_t w = read_w(0, 0, ks);
#pragma unroll
        for (int p = 0; p < Op::kParts; ++p) Op::unpack(p, w, cur.z[0][ks / kStepsPerSeg], consts, tmp, B[0][ks]);
    }
#pragma unroll
    for (int ks = 0; ks < kSteps / RT; ++ks) wv[0][ks] = read_w(0, 1, ks);

    int buf = 0;
    float s_prev = 0.f;
    for (int st = 0; st < stages; ++st) {
        const int nbuf = buf + 1 == kBuffers ? 0 : buf + 1;
        // One slot per MFMA.  The compiler may not move anything from slot to slot: each holds what fits beside one MFMA.
        for_each_constant(std::make_integer_sequence<int, kTiles * kSteps>{}, [&](auto slot_) {
            constexpr int slot = decltype(slot_)::value;
            typedef StageSlot<slot, RT, SEG> Slot;
            constexpr int t = Slot::t, ct = Slot::ct, rt = Slot::rt, ks = Slot::ks, w_end = Slot::w_end;
            part[Slot::pp] = Op::mfma(A[rt][ks], B[ct][ks], Slot::kFirst ? zero16 : part[Slot::pp]);
            if constexpr (ct == 1) A[rt][ks] = read_a(nbuf, rt, ks);
            step_and_unpack<Op, Slot>(tot, part, s_prev, cur, nxt, consts, tmp, B, [&](auto w) { return wv[t & 1][w]; });
            // the words of the next tile's share
            if constexpr (ks == 2) {
                if constexpr (rt + 1 < RT) static_range<w_end, (rt + 2) * kSteps / RT>([&](auto w) { wv[(t & 1) ^ 1][w] = read_w(ct == 0 ? buf : nbuf, ct ^ 1, w); });
                else static_range<0, kSteps / RT>([&](auto w) { wv[(t & 1) ^ 1][w] = read_w(nbuf, ct, w); });
            }
            if constexpr (slot == 1) {
                // The next stage has landed when at most the stage after it is on its way; behind the barrier it has for
                // every wave, and no wave reads X of this stage (all in registers) any more: its buffer is refilled.
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(Sh::kPerStage) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if constexpr (ct == 0 && rt == RT - 1 && ks == (RT == 1 ? 2 : 0)) read_scales_raw(nbuf);  // behind the barrier
            if constexpr (ct == 0 && rt == RT - 1 && ks == 7) convert_scales(nxt);
            // The refill: X beside the first half's MFMAs, the rest (whose buffers this wave has just read for the last time)
            // beside the second's, which also fetch A.
            constexpr int pos = rt * kSteps + ks - (ct == 0 ? 2 : 0), slots = RT * kSteps - (ct == 0 ? 2 : 0);
            constexpr int f0 = ct == 0 ? 0 : Sh::kXLoads, fn = ct == 0 ? Sh::kXLoads : Sh::kPerStage - Sh::kXLoads;
            if constexpr (pos >= 0) static_range<f0 + pos * fn / slots, f0 + (pos + 1) * fn / slots>([&](auto i) { fetch(buf, i); });
            __builtin_amdgcn_sched_barrier(0);
        });
        cur = nxt;
        buf = nbuf;
    }
    // the fetches past the slice's end write into LDS too: they must have landed before the workgroup's LDS is given away
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    constexpr int kLast = (kTiles * Sh::kSegs - 1) & 1;
#pragma unroll
    for (int i = 0; i < 16; ++i) tot[kTiles - 1][i] = __builtin_fmaf(s_prev, part[kLast][i], tot[kTiles - 1][i]);

    // lane (half, l32), element i of row tile rt: row 32 rt + 8 (i / 4) + 4 half + i mod 4, columns 2 l32 and 2 l32 + 1
    const int col = col0 + 2 * l32;
    if (col >= a.N) return;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int m = m0 + 32 * rt + 8 * (i >> 2) + 4 * half + (i & 3);
            if (m >= a.M) continue;
            const float v0 = tot[rt][i], v1 = tot[RT + rt][i];
            if (partial)
                store_partial(partial + (m - m0) * kCols + (col - tile_col0), v0, v1);
            else
                *reinterpret_cast<uint32_t *>(a.Y + (size_t)m * a.N + col) = Act::pack2(v0, v1);
        }
}

// Tiles are numbered blocks of 128 rows first, then the last block of 32 LAST rows (the shorter ones fill the compute
// units that are left over); within the blocks of 128 rows, kRowGroup row blocks x all column tiles after one another,
// row blocks fastest, so that neighbours share their weights and a few of them X.  The first `direct` tiles are done
// whole.  The others are cut: those of 128 rows into `pieces` of 32 LAST rows (1: not), and each piece into a.split slices of K
// of `slice_k` (1: none), which the second launch adds up.  Pieces of rows cost more unpack, slices their partials and the
// launch: M = 1000, K = N = 4096, groups of 64 (128 tiles): 47.3 us in 2 slices, 43.1 in 256 pieces; M = 777, K = 4096, N = 11008, BF16 (2 tiles
// of 128 rows and 43 of 32 past the first round): 84 in 5 slices, 76 in 51 pieces of 32 rows and 5 slices.
struct TileOf {
    int m0, col0;
    bool last;
};
struct Cut {
    int direct, large;  // whole tiles; tiles of 128 rows among the cut ones
    int count;          // pieces
    int pieces;         // of a tile of 128 rows
};
__device__ __forceinline__ TileOf tile_of(int id, int main_blocks, int ntiles)
{
    const int main_total = main_blocks * ntiles;
    if (id >= main_total) return {main_blocks * 32 * kMainRt, (id - main_total) * kCols, true};
    const int band = id / (kRowGroup * ntiles);
    const int band_rows = main_blocks - band * kRowGroup < kRowGroup ? main_blocks - band * kRowGroup : kRowGroup;
    const int in_band = id - band * kRowGroup * ntiles;
    const int tile = in_band / band_rows;
    return {(band * kRowGroup + in_band - tile * band_rows) * 32 * kMainRt, tile * kCols, false};
}

__device__ __forceinline__ TileOf piece_of(const Cut &c, int id, int main_blocks, int ntiles)
{
    const int whole = c.large * c.pieces;
    if (id >= whole) return tile_of(c.direct + c.large + id - whole, main_blocks, ntiles);
    const int tile = id / c.pieces;
    TileOf t = tile_of(c.direct + tile, main_blocks, ntiles);
    t.m0 += (id - tile * c.pieces) * (kPanelRows / c.pieces);
    t.last = c.pieces > 1;
    return t;
}

template <typename Op, int LAST, int SEG>
__global__ __launch_bounds__(64 * kWaves) void panel_kernel(const GemmArgs a, const int main_blocks, const Cut c, const int slice_k)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int ntiles = (a.N + kCols - 1) / kCols;
    // Workgroup b runs on XCD b mod 8: an XCD takes a contiguous range of the whole tiles, then of the (piece, slice) pairs.
    const int direct_per_xcd = (c.direct + kXcds - 1) / kXcds;
    const int xcd = (int)(blockIdx.x % kXcds);
    int local = (int)(blockIdx.x / kXcds), kbeg = 0, kend = a.K;
    float *partial = nullptr;
    TileOf t;
    if (local < direct_per_xcd) {
        const int id = xcd * direct_per_xcd + local;
        if (id >= c.direct) return;
        t = tile_of(id, main_blocks, ntiles);
    } else {
        local -= direct_per_xcd;
        const int pairs = c.count * a.split, per_xcd = (pairs + kXcds - 1) / kXcds;
        const int pair = xcd * per_xcd + local;
        if (local >= per_xcd || pair >= pairs) return;
        const int slice = pair / c.count, id = pair - slice * c.count;
        t = piece_of(c, id, main_blocks, ntiles);
        kbeg = slice * slice_k;
        kend = a.K - kbeg < slice_k ? a.K : kbeg + slice_k;
        if (a.split > 1) partial = a.partials + ((size_t)id * a.split + slice) * (kPanelPartial / c.pieces);
    }
    if constexpr (LAST != kMainRt) {
        if (t.last) {
            panel<Op, LAST, SEG>(a, smem, t.m0, t.col0, kbeg, kend, partial);
            return;
        }
    }
    panel<Op, kMainRt, SEG>(a, smem, t.m0, t.col0, kbeg, kend, partial);
}

// The second launch: Y of the cut tiles, slices added in ascending order.  A workgroup takes four rows of a piece.
template <typename Act>
__global__ __launch_bounds__(256) void panel_reduce_kernel(const GemmArgs a, const int main_blocks, const Cut cut)
{
    const int ntiles = (a.N + kCols - 1) / kCols, parts = kPanelRows / 4 / cut.pieces, idx = (int)blockIdx.x / parts;
    const TileOf t = piece_of(cut, idx, main_blocks, ntiles);
    const int r = ((int)blockIdx.x - idx * parts) * 4 + (int)(threadIdx.x >> 6), c = (int)(threadIdx.x & 63u) * 4;
    if (t.m0 + r >= a.M || t.col0 + c >= a.N) return;
    const size_t stride = kPanelPartial / cut.pieces;
    const float *p = a.partials + (size_t)idx * a.split * stride + r * kCols + c;
    float4_t acc = *reinterpret_cast<const float4_t *>(p);
    int s = 1;
    for (; s + 4 <= a.split; s += 4) {  // four loads in flight, added in slice order
        float4_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const float4_t *>(p + (size_t)(s + e) * stride);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc += v[e];
    }
    for (; s < a.split; ++s) acc += *reinterpret_cast<const float4_t *>(p + (size_t)s * stride);
    *reinterpret_cast<uint2_t *>(a.Y + (size_t)(t.m0 + r) * a.N + t.col0 + c) = (uint2_t){Act::pack2(acc[0], acc[1]), Act::pack2(acc[2], acc[3])};
}

template <typename Op, int LAST, int SEG>
hipError_t launch(const GemmArgs &a, const PanelPlan &p, hipStream_t stream)
{
    const int main_blocks = p.tiles_m - (p.last_rows < kPanelRows ? 1 : 0);
    const Cut cut = {p.tiles_m * p.tiles_n - p.split_tiles, p.split_tiles - p.split_small(), p.cut(), p.pieces};
    const long long grid = (((long long)cut.direct + kXcds - 1) / kXcds + ((long long)cut.count * p.split + kXcds - 1) / kXcds) * kXcds;
    const int lds = main_blocks ? Panel<kMainRt, SEG>::kLds : Panel<LAST, SEG>::kLds;
    const void *const kernel = reinterpret_cast<const void *>(&panel_kernel<Op, LAST, SEG>);
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, Panel<kMainRt, SEG>::kLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((panel_kernel<Op, LAST, SEG>), dim3((unsigned)grid), dim3(64 * kWaves), lds, stream, a, main_blocks, cut, p.slice_k);
    if (p.split > 1) hipLaunchKernelGGL((panel_reduce_kernel<typename Op::Act>), dim3((unsigned)(cut.count * (kPanelRows / 4 / p.pieces))), dim3(256), 0, stream, a, main_blocks, cut);
    return hipGetLastError();
}

template <typename Op, int LAST>
hipError_t launch_seg(const GemmArgs &a, const PanelPlan &p, hipStream_t stream)
{
    if (a.group % 128 == 0) return launch<Op, LAST, 128>(a, p, stream);
    return a.group == 64 ? launch<Op, LAST, 64>(a, p, stream) : launch<Op, LAST, 32>(a, p, stream);
}

template <typename Op>
hipError_t launch_op(const GemmArgs &a, const PanelPlan &p, hipStream_t stream)
{
    switch (p.pieces > 1 ? kPanelRows / p.pieces : p.last_rows) {
    case 32: return launch_seg<Op, 1>(a, p, stream);
    case 64: return launch_seg<Op, 2>(a, p, stream);
    case 96: return launch_seg<Op, 3>(a, p, stream);
    default: return launch_seg<Op, 4>(a, p, stream);
    }
}

}  // namespace

hipError_t launch_panel(const GemmArgs &a, const PanelPlan &p, hipStream_t stream)
{
    if (!panel_takes(a.group) || p.tiles_m != (a.M + kPanelRows - 1) / kPanelRows || p.tiles_n != (a.N + kPanelCols - 1) / kPanelCols) return hipErrorInvalidValue;
    if (p.last_rows != (a.M - (p.tiles_m - 1) * kPanelRows + 31) / 32 * 32) return hipErrorInvalidValue;  // (so every piece of 32 rows begins inside the matrix)
    if (p.split_tiles < 0 || p.split_tiles > p.tiles_m * p.tiles_n || a.split != p.split) return hipErrorInvalidValue;
    // pieces of the rows that the last row block's tiles have, if there are any
    if ((p.pieces != 1 && p.pieces != 2 && p.pieces != 4) || (p.pieces > 1 && p.last_rows < kPanelRows && p.last_rows != kPanelRows / p.pieces)) return hipErrorInvalidValue;
    // slices cover K, none is empty, each begins at a group and at a whole stage of scales
    if (p.split < 1 || (p.split > 1 && (!a.partials || !p.split_tiles || p.slice_k % a.group || (a.group < kStage && p.slice_k % kStage))) ||
        (long long)p.slice_k * (p.split - 1) >= a.K || (long long)p.slice_k * p.split < a.K) return hipErrorInvalidValue;
    if (a.K / 8 * (unsigned long long)a.N * 4ull >= 0x7F000000ull || (unsigned long long)a.M * a.K * 2ull >= 0x7F000000ull) return hipErrorInvalidValue;  // 32-bit buffer offsets
    return a.bf16 ? launch_op<ExactBF16>(a, p, stream) : launch_op<ExactF16>(a, p, stream);
}

}  // namespace w4a16
