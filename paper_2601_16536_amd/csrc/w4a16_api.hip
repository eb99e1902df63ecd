// C-ABI layer of the W4A16 GEMM library: argument checks, the Split-K
// scheduler (Algorithm 1 takes the split factor S and the block sizes as
// inputs and gives no rule for them; the rule lives here), workspace
// management and dispatch to the kernel launchers.
#include "../../include/w4a16.h"
#include "w4a16_internal.h"

#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <string.h>
#include <vector>

namespace {

using namespace w4a16;

constexpr int kMaxDevices = 64;

// Split buffers for callers that cannot allocate (w4a16_gemm_noalloc): one array per GPU the library is loaded on,
// held until the process ends.  Host code never uses the array's name as an address: each device's copy is
// looked up once with hipGetSymbolAddress.
constexpr size_t kScratchBytes = W4A16_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

struct DeviceState {
    int cus = 0;             // compute units (0 = not read yet)
    void *ws = nullptr;      // library-owned workspace (fp32 partials of the two-pass plans)
    size_t ws_bytes = 0;
    void *acc = nullptr;     // library-owned fixed-point accumulator: all zero between calls
    size_t acc_bytes = 0;
    bool acc_dirty = false;  // a launch that used it failed: cleared again before the next use
    std::vector<void *> retired;  // outgrown buffers: work already enqueued (or captured in a graph) may still use them
    void *user_ws = nullptr;      // w4a16_set_workspace: the caller's split buffers for this device
    size_t user_ws_bytes = 0;
    void *scratch_ptr = nullptr;  // this device's copy of `scratch`
};

std::mutex g_mutex;
DeviceState g_dev[kMaxDevices];
thread_local char t_hip_error[256] = "";

void note_hip_error(hipError_t e)
{
    const char *s = hipGetErrorString(e);
    strncpy(t_hip_error, s ? s : "unknown HIP error", sizeof(t_hip_error) - 1);
    t_hip_error[sizeof(t_hip_error) - 1] = 0;
}

// ---- tuning knobs (for sweeps and tests only) ----------------------------------
//
// Process-wide; each starts from the environment variable of the same name in capitals with the prefix
// W4A16_ (read once, when the library first needs it) and can be changed with w4a16_tune.  0 = the
// scheduler's own choice.
struct Tuning {
    int stripe_finish = 0;  // 1: slices always meet in the accumulator, 2: always in the workspace + second pass
    int stripe_waves = 0;   // waves per STRIPE workgroup
    int stripe_dyn = 0;     // M <= 4: 0/1 = units handed out by ticket (the default), 2 = equal contiguous runs per wave
    int stripe_unit = 0;    // packed rows per unit of the ticket form (2 or 4)
    int stripe_depth = 0;   // units in flight per wave of the ticket form (1, 2; 9 = one, its successor requested ahead of use)
    int stripe_dot2 = 0;    // 1: v_dot2_f32_f16 on the vector ALU instead of the MFMA (measurement only)
    int tile_rows = 0;      // rows of X per TILE workgroup (16, 32, 64)
    int tile_dyn = 0;       // 16 rows of X per workgroup: 1 = units always handed out by ticket, 2 = never (equal runs per wave)
    int tile_depth = 0;     // units in flight per wave of the ticket form (1, 2)
    int tile_waves = 0;     // waves per TILE workgroup (4..8)
    int tile_unit = 0;      // 16 rows of X per workgroup, by ticket: blocks of 32 k per unit (1, 2, 4; 4: of several groups where these are short)
    int tile_wide = 0;      // TILE at 32 or 64 rows of X per workgroup: 2 = the eight-wave form instead of the four-wave one
    int panel = 0;          // M > 16: 1 = always the four-wave 256-column form, 2 = never
    int panel_split = 0;    // its split of the tiles past the last whole round of compute units (1 = none)
    int panel_pieces = 0;   // and the pieces of rows that it cuts them into (1, 2, 4)
    int pair = 0;           // M > 16: 1 = always the eight-wave 128-column form, 2 = never
    int pair_split = 0;     // its split of K
    int log = 0;            // 1: every call prints its plan on stderr
};

struct Knob {
    const char *name;
    int Tuning::*field;
};
const Knob kKnobs[] = {
    {"stripe_finish", &Tuning::stripe_finish}, {"stripe_waves", &Tuning::stripe_waves}, {"stripe_dyn", &Tuning::stripe_dyn},
    {"stripe_unit", &Tuning::stripe_unit},     {"stripe_depth", &Tuning::stripe_depth}, {"stripe_dot2", &Tuning::stripe_dot2},
    {"tile_rows", &Tuning::tile_rows},         {"tile_dyn", &Tuning::tile_dyn},         {"tile_depth", &Tuning::tile_depth},
    {"tile_waves", &Tuning::tile_waves},       {"tile_wide", &Tuning::tile_wide},         {"tile_unit", &Tuning::tile_unit},
    {"panel", &Tuning::panel},                 {"panel_split", &Tuning::panel_split},     {"panel_pieces", &Tuning::panel_pieces},
    {"pair", &Tuning::pair},                   {"pair_split", &Tuning::pair_split},
    {"log", &Tuning::log},
};

Tuning &tuning()
{
    static Tuning t = [] {
        Tuning v;
        for (const Knob &k : kKnobs) {
            char env[64] = "W4A16_";
            size_t n = strlen(env);
            for (const char *c = k.name; *c && n + 1 < sizeof env; ++c) env[n++] = (char)(*c >= 'a' && *c <= 'z' ? *c - 32 : *c);
            env[n] = 0;
            if (const char *e = getenv(env)) v.*(k.field) = atoi(e);
        }
        return v;
    }();
    return t;
}

// Current device index, or -1 when no GPU is usable (planning still works then,
// with the MI355X's 256 compute units assumed).
int current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return -1;
    }
    return (dev >= 0 && dev < kMaxDevices) ? dev : -1;
}

int compute_units(int dev)
{
    if (dev < 0) return 256;
    std::lock_guard<std::mutex> lock(g_mutex);
    if (g_dev[dev].cus == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
            (void)hipGetLastError();
            cus = 256;
        }
        g_dev[dev].cus = cus;
    }
    return g_dev[dev].cus;
}

int check_shape(int group, int M, int N, int K)
{
    if (M < 1 || N < 8 || K < 8) return W4A16_ERR_SHAPE;
    if (N % 8 != 0 || K % 8 != 0) return W4A16_ERR_SHAPE;
    if (M > 16 * 65535 || N > (1 << 22) || (long long)K > (1LL << 30)) return W4A16_ERR_SHAPE;
    if (group < 32 || group % 32 != 0 || K % group != 0) return W4A16_ERR_GROUP;
    return W4A16_OK;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// The kernels address X, and a K slice of the weights, with 32-bit byte offsets.
bool fits_32bit_offsets(int M, int N, int K, int group, int gps)
{
    return (unsigned long long)M * K * 2ull < 0x7F000000ull && (unsigned long long)gps * (group / 8) * N * 4ull < 0x7F000000ull;
}

// ---- the Split-K scheduler ---------------------------------------------------
//
// Algorithm 1 takes the split factor S and the block sizes as inputs.  Here the
// scheduler (kernel = AUTO, split = 0) chooses them from the shape alone:
//
// STRIPE (M = 1 from 4 MB of packed weights on, M = 2 ... 4 on large matrices where tile_beats_stripe does not
//   hold): 256-column stripes x S slices of K with S = compute units / stripes, rounded down: one workgroup per compute unit whose waves share the slice.
// TILE (everything else): 64-column tiles x 16, 32 or 64 rows of X per workgroup (as many rows as still
//   leave a workgroup per compute unit at S = 1), eight or four waves; up to 16 rows they share the slice by ticket, in a form for
//   1, 2, 4, 8 or 16 rows; S = compute units / workgroups, rounded down (a workgroup too many would run as a second round).
//
// PANEL (a form of TILE, M > 16): tiles of 128 rows x 256 columns for prompts, and for batches whose 64-column tiles would
//   run in several rounds or over a long K (use_panel).
// PAIR (a form of TILE, M > 16): tiles of 32 or 64 rows x 128 columns, where its model has it clearly cheaper than these two (use_pair).
//
// WAVE_SPLIT (M <= 4) is kept as a forced plan (w4a16_gemm_ex), the data-parallel form for comparisons:
//   one workgroup of sixteen waves per column tile of 32 or 64 columns; the sixteen waves are sixteen K
//   slices whose partial results meet in LDS.  A split across workgroups is added only when the column
//   tiles cover at most a quarter of the compute units and the slices stay long.
//
// How the K slices of different workgroups of a STRIPE or TILE plan meet: in the 64-bit fixed-point accumulator (one
// returning atomic add per output and slice; measured: the GPU retires about 150 of them per nanosecond)
// while that is cheaper than a second launch (about 3.3 us, measured), else in the FP32 workspace and the
// second pass.  Measured crossover: between 0.5 M and 1 M adds.  The other families always take the second pass.
// At 64 rows of X per workgroup (`rows`; BF16, and groups other than 128) the adds come in a burst of 4096 from every workgroup at once, and
// the crossover is lower (M = 37, K = 10240, N = 4608, S = 3, 511 K adds: 23.8 us in the accumulator; M = 64, 885 K adds, second pass: 18.1;
// BF16, groups of 128, M = 114, K = 1280, N = 1520, S = 3, 520 K adds: 15.8 and 9.9).
bool slices_meet_in_accumulator(int M, int N, int S, int rows)
{
    if (S > 63) return false;  // the accumulator counts arrivals in six bits
    if (tuning().stripe_finish == 1) return true;
    if (tuning().stripe_finish == 2) return false;
    return (long long)S * M * N <= (rows == 64 ? 160 : 640) * 1024;
}

int finish_of(int kernel, int M, int N, int S, int rows)
{
    if (S == 1) return kFinishDirect;
    if (kernel != W4A16_KERNEL_STRIPE && kernel != W4A16_KERNEL_TILE) return kFinishSecondPass;
    return slices_meet_in_accumulator(M, N, S, rows) ? kFinishAccumulator : kFinishSecondPass;
}

// The rows that decide it for a TILE plan.  kFrugal's plans, and FP16 with groups of 128 (w4a16_tile_wide.hip), keep the higher crossover.
int burst_rows(int tile_m, int group, bool bf16, bool frugal) { return frugal || (group == 128 && !bf16) ? 0 : tile_m; }

// Workspace of a plan: nothing, the accumulator [M, N], or the FP32 partials [S, M, N].
size_t workspace_of(int kernel, int M, int N, int S, int rows)
{
    switch (finish_of(kernel, M, N, S, rows)) {
    case kFinishDirect: return 0;
    case kFinishAccumulator: return (size_t)M * N * sizeof(unsigned long long);
    default: return (size_t)S * M * N * sizeof(float);
    }
}

bool stripe_by_ticket(int M) { return M <= 4 && tuning().stripe_dyn != 2; }
// TILE with one block of 16 rows of X: the ticket form (measured 1 to 6 % faster than equal runs per wave at M <= 16;
// with several row blocks, which re-read the weights from the L2, 3 % slower).
bool tile_by_ticket(int M, int rows_x) { return rows_x == 16 && (tuning().tile_dyn == 1 || (M <= 16 && tuning().tile_dyn != 2)); }

// Column tiles and row blocks are grid dimensions of the ticket form (w4a16_tile_dyn.hip).
bool ticket_grid_fits(int M, int N) { return ((long long)N + 63) / 64 <= 65535 && ((long long)M + 15) / 16 <= 65535; }

// TILE with four waves per workgroup: at 32 and 64 rows of X, FP16 with groups of 128 (w4a16_tile_wide.hip), and at 64 rows
// BF16 and the other lengths of group (w4a16_tile_tall.hip; at 32 rows these run the eight-wave form).  Both take FP16 with
// groups of 128 at 64 rows: M = 128, N = 8192, K = 512 / 2048 / 8192: 6.3 / 9.7 / 25.5 us (wide), 7.0 / 10.3 / 26.5 (tall).
bool tile_four(int rows_x, int group, bool bf16)
{
    return ((rows_x == 64 && panel_takes(group)) || (rows_x == 32 && group == 128 && !bf16)) && tuning().tile_wide != 2;
}

// Up to 1024 k per slice a wave of the tall form has no more stages than it keeps in flight, and the BF16 eight-wave kernel for
// groups of 128 is as fast or faster: 64 rows, BF16, K = 1024: M = 48, N = 16384 / 48640: 8.6 / 22.6 us against 8.9 / 23.2; M = 128,
// N = 8192: 8.7 against 8.8; K = 1536, M = 48, N = 16384: 11.0 against 10.4.  Groups of other lengths have a slower eight-wave kernel.
bool short_slices(int group, bool bf16, int gps) { return bf16 && group == 128 && gps <= 8; }

// Blocks of 32 k per unit of the ticket form.  With groups of 64 and 32 a unit may be one group (2 or 1 KiB of weights in flight per wave)
// or several: four blocks (4 KiB).  Several need more registers, so that a second workgroup may not fit the compute unit (more workgroups
// than units: 1.0 to 1.2 times the time at 1 and 2 rows, up to 1.6 at 16), and they are fewer: a short slice has too few for its waves to share
// evenly, the more so the more rows a unit's last step has.  From 1020 drawn shapes (K = 512 ... 32768, N = 512 ... 40000, 1 to 16 rows, both formats) timed both ways, the slices from
// which several are faster; time over that with one group, at k per slice: groups of 32, up to 4 rows 0.94 at 1056, 0.78 at 2048, 0.66 at 8064; 5 to 8 rows 1.05
// at 1344, 0.95 at 1728, 0.81 at 4160; 9 to 16 rows 1.15 at 1472, 1.04 at 2272, 0.97 at 3488, 0.91 at 8576; groups of 64, 1 and 2 rows 1.05 at 1472, 0.95 at 1792, 0.85 at 5184;
// 3 and 4 rows 1.03 at 1664, 0.95 at 2304, 0.90 at 5504; 5 to 8 rows 1.08 at 1600, 1.03 at 2688, 0.96 at 4160; 9 to 16 rows 1.07 at 5248, 1.00 at 9344, 0.97 at 15360.
// It takes several for 304 of them: 15 % faster in the mean, the slowest 2 % slower.
int ticket_unit_blocks(int M, int group, int gps, int workgroups, int cus)
{
    if (tuning().tile_unit) return tuning().tile_unit;
    if (group > 64) return 4;
    const int from = group == 32 ? (M <= 4 ? 1024 : (M <= 8 ? 1600 : 3072)) : (M <= 2 ? 1728 : (M <= 4 ? 2048 : (M <= 8 ? 2816 : 14336)));
    return workgroups <= cus && gps * group >= from ? 4 : group / 32;
}

// Whether TILE's plan at 2 to 4 rows is the faster one where STRIPE is a candidate: from 1560 (shape, rows, format, group) timed both ways (K = 256 ...
// 40000, N = 1024 ... 200000, 20 to 400 MB of weights).  What decides is how evenly either family's plan loads the compute units: `use`
// is the tiles' work over that of all units for the rounds the plan takes, at its longest slice.  TILE, whose forms for few rows do less per
// unit, wins where it uses at least 0.92 of what STRIPE does: 13 % in the mean in one round of workgroups, and at 3 and 4 rows in two (us, TILE / STRIPE:
// M = 4, K = N = 8192 9.1 / 11.0; K = 28672, N = 8192 22.4 / 26.0; K = 13568, N = 31840 37.7 / 42.2).  In more rounds, at 2 rows in two, and where slices beyond 12288 k leave
// a tenth of the units idle, it is up to 16 % slower where they use the same (M = 2, K = 15360, N = 24576 41.5 / 35.8; M = 4, K = 33280, N = 14336 47.9 / 44.8),
// and wins where STRIPE leaves more of them idle (M = 3, K = 9216, N = 36512, 143 stripes 32.8 / 46.6): from 1.1.  Where N is no multiple of 32 rows of W do not begin on 128 bytes, and a tile's 256 bytes of one lie in three lines
// (M = 2, K = 31360, N = 8408 37.5 / 26.2): from 1.3, at 3 and 4 rows, up to three rounds.  And only with units of four blocks: groups of 128 k and
// multiples, of 64 (several to a unit) and, at 3 and 4 rows in one round, of 32; with others the unit is one or two blocks (M = 4, K = 15168, N = 13968,
// groups of 96 44.7 / 24.4).  473 of the 1560 go to TILE: 14 % faster than STRIPE in the mean, the worst 2 % slower.
bool tile_beats_stripe(int M, int N, int K, int group, int cus)
{
    if (!ticket_grid_fits(M, N)) return false;
    const int G = K / group;
    auto use = [&](long long tiles, long long *rounds, int *k) {  // S as make_plan has it
        int S = (int)(cus / tiles);
        S = S < 1 ? 1 : (S > G ? G : S);
        const int gps = (G + S - 1) / S;
        *k = gps * group;
        *rounds = (tiles * ((G + gps - 1) / gps) + cus - 1) / cus;
        return (double)tiles * G / ((double)*rounds * cus * gps);
    };
    long long rounds, stripe_rounds;
    int k, stripe_k;
    const double tile = use(((long long)N + 63) / 64, &rounds, &k), stripe = use(((long long)N + 255) / 256, &stripe_rounds, &stripe_k);
    const bool aligned = N % 32 == 0;
    if (group == 32) return aligned && M > 2 && rounds == 1 && tile >= 0.92 * stripe;
    if (group != 64 && group % 128 != 0) return false;
    if (!aligned) return M > 2 && rounds <= 3 && tile >= 1.3 * stripe;
    const bool one = (rounds == 1 || (rounds == 2 && M > 2)) && (k <= 12288 || tile >= 0.9);
    return tile >= (one ? 0.92 : 1.1) * stripe;
}

// LDS a STRIPE workgroup needs for a slice of gps groups, and the most it may use.
size_t stripe_lds(int M, int group, int gps, int waves)
{
    return stripe_by_ticket(M) ? stripe_dyn_lds_bytes(M, group, gps) : stripe_lds_bytes(M, group, gps, waves);
}
size_t stripe_lds_max(int M) { return (size_t)(stripe_by_ticket(M) ? stripe_dyn_lds_limit() : stripe_lds_limit()); }

// Estimated time (us) of a TILE plan for M > 16: `rows` of X per workgroup, K in S slices.  A model of three terms with
// constants measured on K = N = 8192 and on the paper's Fig. 2 shapes at M = 32 and 64 (it orders the 30 plans measured
// there as the clock does): a fixed 3 us; rounds of workgroups x blocks of 32 k per wave x the time of a block
// (four-wave form: 0.24 us at 32 rows, 0.37 at 64; eight-wave form: 0.37, 0.56, 0.94 at 16, 32, 64 rows); and how the
// slices meet (accumulator: 1 us, and beyond 200 K adds 1 us per 60 K; second pass: 3.3 us and the partials at 3 TB/s).
// (The four-wave form's blocks, 5 to 9 % shorter since its unpack in ten instructions, and the second pass, since partials are written through, have the older
// costs here and in panel_cost; only pair_cost is fitted to the kernels as they are.)
// `frugal`: the costs by which kFrugal's plans are chosen, the same for both formats.
double tile_plan_cost(int M, int N, int K, int group, int rows, int S, int cus, bool bf16, bool frugal)
{
    const int G = K / group;
    const int gps = (G + S - 1) / S;
    S = (G + gps - 1) / gps;
    const bool four = tile_four(rows, group, bf16 && !frugal) && (rows == 32 || group == 128 || !frugal);
    const int waves = four ? 4 : 8;
    const double per_block = four ? (rows == 64 ? (group == 32 ? 0.45 : 0.37) : 0.24) : (rows == 64 ? 0.94 : (rows == 32 ? 0.56 : 0.37));
    const long long tiles = (N + 63) / 64, wgs = tiles * ((M + rows - 1) / rows) * S;
    const long long rounds = (wgs + cus - 1) / cus;
    const long long blocks = ((long long)gps * (group / 32) + waves - 1) / waves;
    double finish = 0.0;
    if (S > 1) {
        const double adds = (double)S * M * N;
        finish = slices_meet_in_accumulator(M, N, S, burst_rows(rows, group, bf16, frugal)) ? 1.0 + (adds > 2e5 ? (adds - 2e5) / 6e4 : 0.0) : 3.3 + 2.0 * adds * 4.0 / 3e6;
    }
    return 3.0 + (double)rounds * (double)blocks * per_block + finish;
}

// The next S whose slices are shorter: every S up to it is the same plan.  (With many groups and few columns most are: K = 28672,
// N = 64, groups of 32 had 768 plans to cost, 20 us, longer than the multiply.)
int next_split(int G, int s)
{
    const int gps = (G + s - 1) / s;
    return gps > 1 ? (G + gps - 2) / (gps - 1) : G + 1;
}

// Rows of X per workgroup and S (`split` 0: up to one workgroup per compute unit) that the model finds cheapest.
struct TileChoice {
    int rows, S;
    double cost;
};
TileChoice cheapest_tiles(int M, int N, int K, int group, int split, int cus, bool bf16, bool frugal)
{
    TileChoice best = {16, 1, 1e30};
    const int G = K / group;
    for (int r = 16; r <= 64; r *= 2) {
        if (r > 16 && r / 2 >= M) break;  // more than half of the block's rows would be empty
        const long long w1 = (long long)((N + 63) / 64) * ((M + r - 1) / r);
        const int smax = split ? split : ((int)(cus / w1) < 1 ? 1 : ((int)(cus / w1) > G ? G : (int)(cus / w1)));
        for (int s = split ? split : 1; s <= smax; s = next_split(G, s)) {
            const double c = tile_plan_cost(M, N, K, group, r, s, cus, bf16, frugal);
            if (c < best.cost) best = {r, s, c};
        }
    }
    return best;
}

// The choice for one format.  BF16 has costs of its own with groups of 128 (at 32 rows the eight-wave form), which are good for
// about a tenth: FP16's choice stays where it is no more than that dearer.  On 250 drawn shapes of 17 to 600 rows where the two
// differ, against FP16's choice: 13 % faster in the mean (M = 272, K = 3200, N = 5400: 39.0 -> 26.7 us), the slowest 2 % slower; whatever
// is cheapest by BF16's costs: 11 % in the mean, but 7 of 200 shapes 2 to 17 % slower.
TileChoice choose_tiles(int M, int N, int K, int group, int split, int cus, bool bf16, bool frugal)
{
    TileChoice c = cheapest_tiles(M, N, K, group, split, cus, false, frugal);
    if (!bf16 || frugal || group != 128) return c;
    const TileChoice own = cheapest_tiles(M, N, K, group, split, cus, true, false);
    c.cost = tile_plan_cost(M, N, K, group, c.rows, c.S, cus, true, false);
    return own.cost < 0.9 * c.cost ? own : c;
}

// PANEL form (w4a16_panel.hip), for the scheduler's own plans beyond 16 rows: tiles of 128 x 256, the last row block of
// 32, 64, 96 or 128 rows, one tile per compute unit at a time.  The tiles past the last whole round of compute units may be
// cut to fill the units once more: those of 128 rows into pieces of 64 or 32 rows, and all of them into S slices of K, whose FP32
// partials (at most one tile per unit, 32 MB) are summed by a second launch.  Pieces of rows need no partials, or with slices
// half or a quarter of them, but a word is unpacked once for each.  Costs (us), fitted to 26 (shape, format, group) measured with and without the split (M = 129 ... 2048,
// K = 2048 ... 28672, N = 1024 ... 28672): a stage of 128 k 1.3 at 128 rows, 0.8, 0.6, 0.47 of that at 96, 64, 32 rows
// (the unpack is the same work at any number of rows), a quarter and a half more with groups of 64 and 32 (more of Eq. 2's
// steps), a tenth more for BF16; 3 per tile for its first loads and its stores; the second launch 5 and the partials at 3.5 TB/s.  A piece of 64 or 32 rows
// takes 0.73 and 0.66 (BF16 0.77 and 0.7) of a stage: fitted to 12 shapes with every cut forced (M = 384, K = N = 5120: 60 tiles in 4 slices 33.9 us, 120 pieces
// in 2 slices 33.6, 240 pieces of 32 rows 39.8; M = 1000, K = N = 4096, groups of 64: 47.3 in 2 slices, 43.1 in 256 pieces).  Pieces have to be 4 %
// cheaper than slices alone.  Of 70 drawn shapes (M = 100 ... 2048) whose plan they change, against the plan before: 0.895 of its time
// in the geometric mean (M = 567, K = 8192, N = 6720 88 -> 68; M = 777, K = 4096, N = 11008, BF16 84 -> 76; the best 0.56, the worst 1.04).
double panel_cost(int M, int N, int K, int group, bool bf16, int cus, bool may_split, PanelPlan *p)
{
    static const double kRel[5] = {0.0, 0.47, 0.6, 0.8, 1.0}, kPieceRel[2][3] = {{0.0, 0.66, 0.73}, {0.0, 0.7, 0.77}};
    const double stage = 1.3 * (group == 32 ? 1.5 : (group == 64 ? 1.25 : 1.0)) * (bf16 ? 1.1 : 1.0);
    const double kStageUs[5] = {0.0, stage * kRel[1], stage * kRel[2], stage * kRel[3], stage};
    const double fixed = 3.0;
    p->tiles_m = (M + kPanelRows - 1) / kPanelRows;
    p->tiles_n = (N + kPanelCols - 1) / kPanelCols;
    p->last_rows = (M - (p->tiles_m - 1) * kPanelRows + 31) / 32 * 32;
    p->split_tiles = 0;
    p->pieces = 1;
    p->split = 1;
    p->slice_k = K;
    const int unit = group < 128 ? 128 : group;  // slices begin at a group and at a whole stage
    const int units = (K + unit - 1) / unit, last_rt = p->last_rows / 32;
    const long long tiles = (long long)p->tiles_m * p->tiles_n, small = last_rt < 4 ? p->tiles_n : 0, large = tiles - small;
    // time of the first `n` tiles, the large ones first
    auto whole = [&](long long n, int k) {
        const double stages = (k + 127) / 128, c4 = stages * kStageUs[4] + fixed, cl = stages * kStageUs[last_rt] + fixed;
        const long long n4 = n < large ? n : large, nl = n - n4;
        double t = (double)(n4 / cus) * c4;
        const long long busy = n4 % cus, idle = cus - busy;
        if (busy == 0) return t + (double)((nl + cus - 1) / cus) * cl;
        const long long fit = idle * (c4 >= 2.0 * cl ? (long long)(c4 / cl) : 1);
        if (nl <= fit) {
            const double s = (double)((nl + idle - 1) / idle) * cl;
            return t + (s > c4 ? s : c4);
        }
        return t + c4 + (double)((nl - fit + cus - 1) / cus) * cl;
    };
    double best = whole(tiles, K);
    const long long rest = tiles % cus, done = tiles - rest;
    if (rest) {
        const double before = whole(done, K);
        const int small_rest = (int)(rest < small ? rest : small), large_rest = (int)rest - small_rest;
        const int want_split = tuning().panel_split, want_pieces = tuning().panel_pieces;
        bool found = want_split <= 1 && want_pieces == 0;  // (a cut that was asked for is taken whatever it costs)
        for (int pieces = 1; pieces <= 4; pieces *= 2) {
            if (pieces > 1 && (large_rest == 0 || (small && p->last_rows != kPanelRows / pieces))) continue;
            if (want_pieces && pieces != want_pieces) continue;
            const int cut = large_rest * pieces + small_rest, rt = large_rest ? 4 / pieces : last_rt;
            const int smax = (int)(cus / cut) < units ? (int)(cus / cut) : units;
            for (int s = pieces > 1 ? 1 : 2; s <= smax && s <= 16; ++s) {
                if ((s > 1 && (!may_split || want_split == 1)) || (want_split > 1 && s != want_split)) continue;
                const int k = (units + s - 1) / s * unit;
                if ((long long)k * (s - 1) >= K) continue;  // an empty slice
                const double c = before + (double)((k + 127) / 128) * (pieces > 1 ? stage * kPieceRel[bf16][rt] : kStageUs[rt]) + fixed +
                                 (s > 1 ? 5.0 + (double)cut * s * kPanelPartial * 4.0 / 3.5e6 * (rt / 4.0) : 0.0);
                if (c < (pieces > 1 && p->pieces == 1 && found ? 0.96 : 1.0) * best || !found) {
                    found = true;
                    best = c;
                    p->split_tiles = (int)rest;
                    p->pieces = pieces;
                    p->split = s;
                    p->slice_k = s > 1 ? k : K;
                }
            }
        }
    }
    return 3.0 + best;
}

bool use_panel(int M, int N, int K, int group, bool bf16, int cus, bool may_split, PanelPlan *p, double *p_cost)
{
    if (tuning().panel == 2 || !panel_takes(group) || !fits_32bit_offsets(M, N, K, group, K / group)) return false;
    if ((long long)((M + kPanelRows - 1) / kPanelRows) * ((N + kPanelCols - 1) / kPanelCols) > (1 << 24)) return false;  // a launch's blocks
    if (tuning().panel == 1 && M > 16) {
        *p_cost = panel_cost(M, N, K, group, bf16, cus, may_split, p);
        return true;
    }
    if (M <= 16) return false;
    // Against the cheapest plan of 64-column tiles.  Beyond 128 rows each of their rounds after the first costs about 3.5 us
    // more than the model says (measured: M = 512 ... 2048, two to nine rounds).  Up to 128 rows PANEL wins where 64-column
    // tiles need several rounds or K is long (K = 28672, N = 8184, M = 32 / 64: 41.7 / 52.6 against 29.9 / 40.3 us; K = 18432, N = 7168,
    // M = 64: 32.5 against 28.7; K = 8192, N = 8184, M = 32 / 64: 16.4 / 19.3 against 15.9 / 20.2; K = 4096: 10.4 / 11.5 against 14.8 / 20.3);
    // there it has to be 7 % cheaper, as the two models are together good for about that: of 160 FP16 shapes (M = 17, 32, 48, 64,
    // K = 4096 ... 28672, N = 1024 ... 8184, groups of 128) it is taken for 31 and faster on
    // every one, as on 150 drawn ones of 17 to 64 rows and below 8192 columns (22 % in the mean).
    const double cost = *p_cost = panel_cost(M, N, K, group, bf16, cus, may_split, p), factor = M <= 128 ? 0.93 : (p->pieces > 1 ? 0.93 : 1.0);
    const int G = K / group;
    for (int r = 64; r >= 16; r /= 2) {
        const long long wgs = (long long)((N + 63) / 64) * ((M + r - 1) / r);
        int smax = (int)(cus / wgs);
        smax = smax < 1 ? 1 : (smax > G ? G : smax);
        for (int s = 1; s <= smax; s = next_split(G, s)) {
            const double c = tile_plan_cost(M, N, K, group, r, s, cus, bf16, false) + (M > 128 ? 3.5 * (double)((wgs * s - 1) / cus) : 0.0);
            if (cost >= factor * c) return false;
        }
    }
    return true;
}

// PAIR form (w4a16_pair.hip), for the scheduler's own plans beyond 16 rows: tiles of 32 or 64 rows x 128 columns, K in S slices, at
// most as many workgroups as compute units where there are several.  Costs (us), fitted to 230 timings of 110 drawn shapes (M = 17 ... 700,
// K = 2048 ... 28672, N = 1024 ... 28672), 6 % off in the mean: a round 5.8 (launch, first loads, the sums) and 1.3 to 2.7 per stage of 128 k of
// a quarter of the slice; slices 1.4 and the partials at 1.9 TB/s.  32 rows, BF16, groups of 64: 1.5 is a tenth too little beyond 8192 k (19 shapes 7 to 15 % above;
// M = 1027, K = 17984, N = 3952 was 9 % slower in PAIR than in PANEL).
double pair_cost(int M, int N, int K, int group, bool bf16, int cus, int rows, int S)
{
    static const double kStageUs[2][2][3] = {{{1.3, 1.45, 1.77}, {1.6, 1.5, 2.03}}, {{1.75, 2.06, 2.42}, {1.99, 2.22, 2.7}}};  // rows, format, group
    const int G = K / group, gps = (G + S - 1) / S;
    S = (G + gps - 1) / gps;
    const long long wgs = (long long)((N + kPairCols - 1) / kPairCols) * ((M + rows - 1) / rows) * S, rounds = (wgs + cus - 1) / cus;
    const long long stages = ((long long)gps * group + 511) / 512;
    double stage = kStageUs[rows == 64][bf16][group == 32 ? 2 : (group == 64 ? 1 : 0)];
    if (rows == 32 && bf16 && group == 64 && gps * group > 8192) stage = 1.64;
    return 0.3 + (double)rounds * (5.8 + (double)stages * stage) +
           (S > 1 ? 1.4 + (double)S * M * N * 4.0 / 1.9e6 : 0.0);
}

// Whether the PAIR form's cheapest plan is cheaper than PANEL's (`panel`, of cost `cost`) where that is the plan so far, or than the 64-column tiles':
// by 4 % (PANEL's by 7, up to 128 rows by 13), as the models are good for about that.  Groups of 32 and 64 at up to 32 rows are dearer in 64-column tiles than
// their model has it.  By more where the gain is not there:
//   - FP16 with groups of 128, whose 64-column tiles are the fast ones, gives up an unsplit plan for slices, or one of 16 rows, for a clear gain only (11 shapes with 16
//     rows at 0.90 to 0.96: 3 to 9 % faster than PAIR; K = 1536, M = 141, N = 3576: 7.8 us, PAIR 8.4);
//   - BF16 unsplit against PANEL in slices, beyond 128 rows and 6144 k: 205 shapes at 0.89 to 0.93 are 2.4 % faster in PANEL in the mean, by up to 12 % (M = 155,
//     K = 27200, N = 5624, groups of 64: 88.5 us, PAIR 98.3).  Not so shorter K (61: PAIR 1 % faster), PAIR in slices (236: the same) and groups of 32 (47: PAIR 8 % faster).
// Of 5707 shapes drawn afterwards (17 to 2048 rows) that the models' error alone would send to PAIR, 57 change by these two and pair_cost's long slices, to 0.96 of their
// time; beyond 1.02 of the time before PAIR were 17, and are 4.  Of 306 drawn shapes (17 to 700 rows, every format and group) 75 go to PAIR: 0.850 of their time before in the
// geometric mean, 0.56 (M = 387, K = 2304, N = 2704, groups of 32) to 1.06 (M = 117, K = 16128, N = 1864, groups of 32).
bool use_pair(int M, int N, int K, int group, bool bf16, int cus, const PanelPlan *panel, double cost, TileChoice *c)
{
    const int G = K / group, want = tuning().pair, want_rows = tuning().tile_rows, want_split = tuning().pair_split;
    if (want == 2 || !panel_takes(group)) return false;
    const Tuning &knobs = tuning();
    if (want != 1 && (want_rows || knobs.tile_wide || knobs.panel || knobs.panel_split || knobs.panel_pieces)) return false;  // 64-column tiles, or PANEL, are asked for
    c->cost = 1e30;
    for (int rows = 32; rows <= 64; rows += 32) {
        if (want == 1 && want_rows && rows != want_rows) continue;
        if (rows == 64 && M <= 32 && !(want == 1 && want_rows == 64 && 128ll * K < 0x7F000000)) continue;  // (asked for: X's offsets of all 64 rows)
        const long long w1 = (long long)((N + kPairCols - 1) / kPairCols) * ((M + rows - 1) / rows);
        if (w1 > (1 << 24)) continue;
        int smax = (int)(cus / w1);
        smax = smax < 1 ? 1 : (smax > G ? G : smax);
        for (int s = 1; s <= smax; s = next_split(G, s)) {
            const int S = want_split ? (want_split < G ? want_split : G) : s, gps = (G + S - 1) / S;
            if (!fits_32bit_offsets(M, N, K, group, gps)) continue;
            const double us = pair_cost(M, N, K, group, bf16, cus, rows, S);
            if (us < c->cost) *c = {rows, (G + gps - 1) / gps, us};
        }
    }
    if (c->cost >= 1e30) return false;
    if (want == 1) return true;
    if (panel) {
        const bool dear = bf16 && panel->split > 1 && group >= 64 && c->S == 1 && K > 6144;
        return c->cost < (M <= 128 ? 0.87 : (dear ? 0.89 : 0.93)) * cost;
    }
    const TileChoice tiles = choose_tiles(M, N, K, group, 0, cus, bf16, false);
    const long long wgs = (long long)((N + 63) / 64) * ((M + tiles.rows - 1) / tiles.rows) * tiles.S;
    double factor = group < 128 && tiles.rows <= 32 ? 1.05 : 0.96;
    if (!bf16 && group == 128 && tiles.S == 1 && (c->S > 1 || tiles.rows == 16)) factor = 0.84;
    return c->cost < factor * (tiles.cost + (M > 128 ? 3.5 * (double)((wgs - 1) / cus) : 0.0));
}

// How much workspace a plan may ask for.  kBest: whatever pays.  kUnsplit: a plan of the PANEL form splits no tiles, and none is of the PAIR form.
// kFrugal: 64-column tiles only, split so that the slices of up to 640 K adds meet in the accumulator: many of these plans
// need nothing, the others 8 bytes per output where kBest may take the FP32 partials of all slices.  kBare: 64-column tiles
// and S = 1, no workspace at all.  The last three differ from kBest for the scheduler's own plans beyond 16 rows only.
enum Thrift { kBest, kUnsplit, kFrugal, kBare };

// `panel` (may be null) gets the plan's details where it is one of the PANEL form (tile_n = kPanelCols).
int make_plan(int M, int N, int K, int group, int kernel, int split, int cus, w4a16_plan *p, PanelPlan *panel = nullptr, bool bf16 = false, Thrift thrift = kBest)
{
    const bool frugal = thrift == kFrugal;
    const int G = K / group;
    const bool automatic = kernel == W4A16_KERNEL_AUTO && split == 0;
    if (kernel == W4A16_KERNEL_AUTO) {
        // STRIPE: M = 1 from 4 MB of packed weights on, and at 2 to 4 rows, from 20 and 32 MB on, where TILE is not faster.  Below
        // these sizes it is TILE, many of whose plans there need no workspace: they are not to change for ones that share an accumulator.
        const double packed = 0.5 * (double)K * (double)N;
        bool stripe = (M == 1 && packed >= 4e6) || (M == 2 && packed >= 20e6) || (M <= 4 && packed >= 32e6);
        if (stripe && M >= 2 && tile_beats_stripe(M, N, K, group, cus)) {
            // The scheduler's own plan, or one asked for again by its S.  With another S it is STRIPE, whose workgroups TILE has four of.
            w4a16_plan own;
            stripe = split != 0 && !(make_plan(M, N, K, group, W4A16_KERNEL_TILE, 0, cus, &own, nullptr, bf16) == W4A16_OK && own.split == split);
        }
        kernel = stripe ? W4A16_KERNEL_STRIPE : W4A16_KERNEL_TILE;
    }
    if (kernel != W4A16_KERNEL_WAVE_SPLIT && kernel != W4A16_KERNEL_STRIPE && kernel != W4A16_KERNEL_TILE)
        return W4A16_ERR_UNSUPPORTED;
    if (kernel == W4A16_KERNEL_WAVE_SPLIT && M > 4) return W4A16_ERR_UNSUPPORTED;
    if (kernel == W4A16_KERNEL_STRIPE && M > 16) return W4A16_ERR_UNSUPPORTED;
    // bfloat16 activations: the forms the scheduler chooses from (STRIPE by ticket for M <= 4, TILE)
    if (bf16 && (kernel == W4A16_KERNEL_WAVE_SPLIT || (kernel == W4A16_KERNEL_STRIPE && !stripe_by_ticket(M)))) return W4A16_ERR_UNSUPPORTED;
    if (split < 0 || split > G) return W4A16_ERR_UNSUPPORTED;
    p->kernel = kernel;
    if (automatic && thrift == kBare && M > 16) split = 1;
    long long tiles;
    int S = split;
    if (kernel == W4A16_KERNEL_STRIPE) {
        p->tile_n = 256;
        p->tile_m = M <= 4 ? 4 : 16;
        tiles = (N + 255) / 256;
        if (tiles > 65535) return W4A16_ERR_UNSUPPORTED;  // a grid dimension
        const int wmin = stripe_min_waves(M), wmax = stripe_max_waves(M);
        if (S == 0) S = (int)(cus / tiles);  // at most one workgroup per compute unit (measured, N = 14336: 280 workgroups 11.4 us, 224 8.9 us)
        if (S < 1) S = 1;
        if (S > G) S = G;
        int gps = (G + S - 1) / S;
        // the slice's X rows (and, handed out by ticket, its scales) must fit the workgroup's LDS and its weights a
        // 31-bit buffer: shorten the slice if not
        while (gps > 1 && (stripe_lds(M, group, gps, wmin) > stripe_lds_max(M) || !fits_32bit_offsets(1, N, 8, group, gps)))
            gps = (gps + 1) / 2;
        S = (G + gps - 1) / gps;
        if (stripe_lds(M, group, gps, wmin) > stripe_lds_max(M)) return W4A16_ERR_UNSUPPORTED;
        if (S > 65535) return W4A16_ERR_UNSUPPORTED;  // a grid dimension of the many-row form
        // Waves: at least four blocks of 16 k each, eight at most.  The ticket form (M <= 4) has eight however short its slice, where its workgroups
        // are alone on their compute units: they stage the slice together and their sums meet cheaply (M = 1, us, two or four waves for a slice of
        // one or two groups / eight: K = 2048, N = 4096 5.5 / 4.4; K = N = 4096 5.3 / 4.9; K = 6144, N = 1536 5.1 / 4.6; ten or twelve: within 3 % where the
        // slice is long, slower where it is short).  Several workgroups of few waves share a unit better (K = 128, N = 199992, two / eight 5.9 / 7.1;
        // M = 4, K = 256, N = 164072, four / eight 9.3 / 10.4), but for two of one or two waves each (M = 4, K = 128, N = 90888 7.7 / 6.2).
        const long long nblocks = (long long)gps * (group / 16), wgs = tiles * S;
        const bool eight = stripe_by_ticket(M) && (wgs <= cus || (wgs <= 2 * cus && nblocks <= 8));
        int waves = eight ? 8 : (int)(nblocks / 4);
        const int wbest = stripe_by_ticket(M) ? 8 : (wmax > 12 ? 12 : wmax);
        waves = waves < wmin ? wmin : (waves > wbest ? wbest : waves);
        if (tuning().stripe_waves >= wmin && tuning().stripe_waves <= wmax) waves = tuning().stripe_waves;
        while (waves > wmin && stripe_lds(M, group, gps, waves) > stripe_lds_max(M)) --waves;
        p->waves_k = waves;
        p->threads = waves * 64;
        p->split = S;
        p->groups_per_split = gps;
        p->workgroups = (int)(tiles * S);
        p->workspace_bytes = workspace_of(kernel, M, N, S, 0);
        return fits_32bit_offsets(M, N, K, group, gps) ? W4A16_OK : W4A16_ERR_UNSUPPORTED;
    }
    PanelPlan pp;
    double cost = 0.0;
    const bool by_panel = automatic && thrift < kFrugal && use_panel(M, N, K, group, bf16, cus, thrift == kBest, &pp, &cost);
    TileChoice pair;
    if (automatic && thrift == kBest && M > 16 && use_pair(M, N, K, group, bf16, cus, by_panel ? &pp : nullptr, cost, &pair)) {
        p->kernel = W4A16_KERNEL_TILE;
        p->tile_n = kPairCols;
        p->tile_m = pair.rows;
        p->waves_k = 4;
        p->threads = 512;
        p->split = pair.S;
        p->groups_per_split = (G + pair.S - 1) / pair.S;
        p->workgroups = (N + kPairCols - 1) / kPairCols * ((M + pair.rows - 1) / pair.rows) * pair.S;
        p->workspace_bytes = pair.S > 1 ? (size_t)pair.S * M * N * sizeof(float) : 0;
        return W4A16_OK;
    }
    if (by_panel) {
        p->kernel = W4A16_KERNEL_TILE;
        p->tile_n = kPanelCols;
        p->tile_m = kPanelRows;
        p->waves_k = 1;
        p->threads = 256;
        p->split = pp.split;
        p->groups_per_split = pp.slice_k / group;
        p->workgroups = pp.tiles_m * pp.tiles_n - pp.split_tiles + pp.cut() * pp.split;
        p->workspace_bytes = pp.split > 1 ? (size_t)pp.cut() * pp.split * (kPanelPartial / pp.pieces) * sizeof(float) : 0;
        if (panel) *panel = pp;
        return W4A16_OK;
    }
    if (kernel == W4A16_KERNEL_TILE) {
        p->tile_n = 64;
        p->waves_k = 8;
        p->threads = 512;
        tiles = (N + 63) / 64;
        // Rows of X per workgroup: as many (16, 32 or 64: each loaded weight word feeds that many MFMA rows)
        // as still leave one workgroup per compute unit without splitting K across workgroups (a split costs
        // the FP32 partials and the second pass).
        int rows_x = 64;
        while (rows_x > 16 && (rows_x / 2 >= M || tiles * ((M + rows_x - 1) / rows_x) < cus)) rows_x /= 2;
        const int tr = tuning().tile_rows;
        if (tr == 16 || tr == 32 || tr == 64) {
            rows_x = tr;
        } else if (M > 16 && group % 32 == 0) {
            // M > 16, the scheduler's own S: the rule above is a poor one where it puts a few workgroups more than
            // compute units into a second round, or gives up large row blocks that a split of K would have filled
            // (measured, N = 7168, K = 18432, M = 64: 49.7 us at 16 rows against 33.0 at 64 rows, S = 2): the
            // cheapest of (rows, S) by the model, S up to one workgroup per compute unit (a forced S: the rows for it)
            const TileChoice c = choose_tiles(M, N, K, group, split, cus, bf16, frugal);
            rows_x = c.rows;
            S = c.S;
        }
        if (tile_by_ticket(M, rows_x) && !ticket_grid_fits(M, N)) return W4A16_ERR_UNSUPPORTED;
        p->tile_m = rows_x;
        const int tw = tuning().tile_waves;
        if (tw >= 4 && tw <= (tile_by_ticket(M, rows_x) ? 16 : 8)) { p->waves_k = tw; p->threads = 64 * tw; }
        const long long wgs = tiles * ((M + rows_x - 1) / rows_x);
        if (S == 0) S = (int)(cus / wgs);  // never more workgroups than compute units: the extra ones would run as a second round
        if (S < 1) S = 1;
        if (S > G) S = G;
        int gps = (G + S - 1) / S;
        while (gps > 1 && !fits_32bit_offsets(1, N, 8, group, gps)) gps = (gps + 1) / 2;
        S = (G + gps - 1) / gps;
        if (tile_four(rows_x, group, bf16) && !short_slices(group, bf16, gps)) { p->waves_k = 4; p->threads = 256; }
        p->split = S;
        p->groups_per_split = gps;
        p->workgroups = (int)(wgs * S);
        p->workspace_bytes = workspace_of(kernel, M, N, S, burst_rows(p->tile_m, group, bf16, frugal));
        if (((long long)tiles * S + 7) / 8 * 8 * ((M + rows_x - 1) / rows_x) > 0x7FFFFFFFLL) return W4A16_ERR_UNSUPPORTED;
        return fits_32bit_offsets(M, N, K, group, gps) ? W4A16_OK : W4A16_ERR_UNSUPPORTED;
    }
    {  // WAVE_SPLIT
        p->tile_n = (N + 63) / 64 >= cus ? 64 : 32;
        p->tile_m = 4;
        p->waves_k = 16;
        p->threads = 1024;
        tiles = (N + p->tile_n - 1) / p->tile_n;
        if (tiles > 65535) return W4A16_ERR_UNSUPPORTED;  // a grid dimension
        if (S == 0) {
            // One launch unless the tiles cover at most a quarter of the compute units AND each
            // workgroup would still stream at least 128 KiB per slice (below that the second
            // pass costs more than the idle units).
            S = 1;
            const long long per_wg = (long long)K * p->tile_n / 2;
            if (4 * tiles <= cus) {
                S = (int)(cus / tiles);
                if (S > per_wg / (128 * 1024)) S = (int)(per_wg / (128 * 1024));
            }
        }
    }
    if (S < 1) S = 1;
    if (S > G) S = G;
    int gps = (G + S - 1) / S;
    // slices keep 32-bit buffer offsets: raise S until a slice is below ~2 GiB
    while (gps > 1 && !fits_32bit_offsets(1, N, 8, group, gps)) gps = (gps + 1) / 2;
    S = (G + gps - 1) / gps;  // no empty slice
    p->split = S;
    p->groups_per_split = gps;
    p->workgroups = (int)(tiles * S);
    p->workspace_bytes = workspace_of(kernel, M, N, S, 0);
    return fits_32bit_offsets(M, N, K, group, gps) ? W4A16_OK : W4A16_ERR_UNSUPPORTED;
}

// ---- split buffers --------------------------------------------------------------

// True when `stream` is being captured into a graph: nothing may be allocated or synchronised then.
bool capturing(hipStream_t stream)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

// Grows one of the library-owned buffers.  The old buffer is not freed: work enqueued earlier, or recorded in a
// graph, may still use it; it goes to the retired list until w4a16_shutdown.  Never called during stream capture.
int grow(DeviceState &d, void **buf, size_t *have, size_t bytes, size_t floor_bytes, bool zeroed)
{
    size_t want = bytes + bytes / 4;
    if (want < floor_bytes) want = floor_bytes;
    void *ptr = nullptr;
    hipError_t e = hipMalloc(&ptr, want);
    if (e != hipSuccess) { note_hip_error(e); (void)hipGetLastError(); return W4A16_ERR_WORKSPACE; }
    if (zeroed) {
        // cleared before any stream can see it: the copy engine's memset, then a wait for the device
        e = hipMemset(ptr, 0, want);
        if (e == hipSuccess) e = hipDeviceSynchronize();
        if (e != hipSuccess) { note_hip_error(e); (void)hipFree(ptr); return W4A16_ERR_HIP; }
    }
    if (*buf) d.retired.push_back(*buf);
    *buf = ptr;
    *have = want;
    return W4A16_OK;
}

enum Source { kFromLibrary, kFromCall, kFromScratch };

struct Buffers {
    unsigned long long *sync = nullptr;  // the accumulator: zero before the launch, left zero by it
    float *partials = nullptr;
    bool library_acc = false;
};

int find_buffers(int dev, const w4a16_plan &plan, int finish, int M, int N, hipStream_t st, Source src, void *call_ws,
                 size_t call_ws_bytes, Buffers *out)
{
    if (finish == kFinishDirect) return W4A16_OK;
    void *given = nullptr;
    size_t given_bytes = 0;
    if (src == kFromCall) {
        given = call_ws;
        given_bytes = call_ws_bytes;
    } else if (src == kFromScratch) {
        std::lock_guard<std::mutex> lock(g_mutex);
        DeviceState &d = g_dev[dev];
        if (!d.scratch_ptr) {  // once per device, with that device current
            void *ptr = nullptr;
            hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !ptr) { note_hip_error(e); (void)hipGetLastError(); return W4A16_ERR_HIP; }
            d.scratch_ptr = ptr;
        }
        given = d.scratch_ptr;
        given_bytes = kScratchBytes;
    } else {
        std::lock_guard<std::mutex> lock(g_mutex);
        if (g_dev[dev].user_ws) {
            given = g_dev[dev].user_ws;
            given_bytes = g_dev[dev].user_ws_bytes;
        }
    }
    if (given) {
        if (given_bytes < plan.workspace_bytes) return W4A16_ERR_WORKSPACE;
        if (finish == kFinishAccumulator) {  // contents unknown: cleared by a small launch first
            out->sync = static_cast<unsigned long long *>(given);
            hipError_t e = launch_accumulator_clear(out->sync, (size_t)M * N, st);
            if (e != hipSuccess) { note_hip_error(e); return W4A16_ERR_HIP; }
        } else {
            out->partials = static_cast<float *>(given);
        }
        return W4A16_OK;
    }
    // library-owned, grown on demand
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState &d = g_dev[dev];
    if (finish == kFinishAccumulator) {
        if (d.acc_bytes < plan.workspace_bytes) {
            if (capturing(st)) return W4A16_ERR_WORKSPACE;
            int rc = grow(d, &d.acc, &d.acc_bytes, plan.workspace_bytes, 1u << 20, true);
            if (rc) return rc;
            d.acc_dirty = false;
        }
        out->sync = static_cast<unsigned long long *>(d.acc);
        out->library_acc = true;
        if (d.acc_dirty) {
            hipError_t e = launch_accumulator_clear(out->sync, d.acc_bytes / 8, st);
            if (e != hipSuccess) { note_hip_error(e); return W4A16_ERR_HIP; }
            d.acc_dirty = false;
        }
    } else {
        if (d.ws_bytes < plan.workspace_bytes) {
            if (capturing(st)) return W4A16_ERR_WORKSPACE;
            int rc = grow(d, &d.ws, &d.ws_bytes, plan.workspace_bytes, 0, false);
            if (rc) return rc;
        }
        out->partials = static_cast<float *>(d.ws);
    }
    return W4A16_OK;
}

void log_plan(const char *entry, int M, int N, int K, int group, const w4a16_plan &p, int finish, int unit_blocks)
{
    static const char *const kFinish[] = {"direct", "accumulator", "second pass"};
    char unit[24] = "";
    if (unit_blocks) snprintf(unit, sizeof unit, " unit=%d", unit_blocks);
    fprintf(stderr, "w4a16: %s M=%d N=%d K=%d group=%d -> kernel=%d S=%d groups/slice=%d tile=%dx%d waves=%d workgroups=%d finish=%s workspace=%zu%s\n",
            entry, M, N, K, group, p.kernel, p.split, p.groups_per_split, p.tile_m, p.tile_n, p.waves_k, p.workgroups,
            kFinish[finish], p.workspace_bytes, unit);
}

int run(const char *entry, const void *X, const uint32_t *Wp, const void *scales, const uint32_t *zeros, int group, int M, int N,
        int K, void *Y, void *stream, int kernel, int split, Source src, void *call_ws, size_t call_ws_bytes, bool bf16 = false)
{
    t_hip_error[0] = 0;
    if (!X || !Wp || !scales || !Y) return W4A16_ERR_NULL;  // zeros may be null: symmetric quantisation
    if (src == kFromCall && !call_ws) return W4A16_ERR_NULL;
    int rc = check_shape(group, M, N, K);
    if (rc) return rc;
    if (!aligned16(X) || !aligned16(Wp) || !aligned16(scales) || !aligned16(zeros) || !aligned16(Y)) return W4A16_ERR_ALIGN;
    if (src == kFromCall && (reinterpret_cast<uintptr_t>(call_ws) & 255u)) return W4A16_ERR_ALIGN;

    const int dev = current_device();
    if (dev < 0) { note_hip_error(hipErrorNoDevice); return W4A16_ERR_HIP; }
    const int cus = compute_units(dev);
    w4a16_plan plan;
    PanelPlan panel;
    bool by_panel = false, by_pair = false;
    int finish = kFinishDirect;
    Buffers b;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // A split is worth a workspace where the call brings one; where it is not to be had, the plans that need less.  Buffers
    // that calls share (the library's, a registered workspace, the fixed array) are for shapes only whose frugal plan needs
    // them too: calls that need none may overlap on several streams.
    // Where the library's own buffers are too small and cannot grow (under a capture), the scheduler's plans end with one that
    // needs none; a caller whose own memory is too small for kFrugal is told so.
    bool only_free = false, bare = false;
    if (src == kFromLibrary && M > 16 && kernel == W4A16_KERNEL_AUTO && split == 0) {
        std::lock_guard<std::mutex> lock(g_mutex);
        bare = !g_dev[dev].user_ws;
    }
    if (src != kFromCall && M > 16) {
        w4a16_plan frugal;
        only_free = make_plan(M, N, K, group, kernel, split, cus, &frugal, nullptr, bf16, kFrugal) == W4A16_OK && frugal.workspace_bytes == 0;
    }
    for (Thrift thrift : {kBest, kUnsplit, kFrugal, kBare}) {
        if (thrift == kBare && !bare) break;
        rc = make_plan(M, N, K, group, kernel, split, cus, &plan, &panel, bf16, thrift);
        if (rc) return rc;
        if (only_free && plan.workspace_bytes != 0) continue;  // (never kFrugal's)
        by_panel = plan.kernel == W4A16_KERNEL_TILE && plan.tile_n == kPanelCols;
        by_pair = plan.kernel == W4A16_KERNEL_TILE && plan.tile_n == kPairCols;
        finish = by_panel || by_pair ? (plan.split > 1 ? kFinishSecondPass : kFinishDirect)
                          : finish_of(plan.kernel, M, N, plan.split, burst_rows(plan.tile_m, group, bf16, thrift == kFrugal));
        t_hip_error[0] = 0;
        rc = find_buffers(dev, plan, finish, M, N, st, src, call_ws, call_ws_bytes, &b);
        if (rc != W4A16_ERR_WORKSPACE) break;
    }
    if (rc) return rc;
    const bool tile_ticket = plan.kernel == W4A16_KERNEL_TILE && !by_panel && !by_pair && tile_by_ticket(M, plan.tile_m);
    const int unit_blocks = tile_ticket ? ticket_unit_blocks(M, group, plan.groups_per_split, plan.workgroups, cus) : 0;
    if (tuning().log) log_plan(entry, M, N, K, group, plan, finish, unit_blocks);

    GemmArgs a;
    a.X = static_cast<const uint16_t *>(X);
    a.Wp = Wp;
    a.scales = static_cast<const uint16_t *>(scales);
    a.Zp = zeros;
    a.Y = static_cast<uint16_t *>(Y);
    a.partials = b.partials;
    a.group = group; a.M = M; a.N = N; a.K = K;
    a.split = plan.split;
    a.groups_per_split = plan.groups_per_split;
    a.groups = K / group;
    a.bf16 = bf16 ? 1 : 0;

    hipError_t e;
    if (plan.kernel == W4A16_KERNEL_STRIPE && stripe_by_ticket(M)) {
        // measured on K = 4096 ... 28672 at M = 1, 2, 4: units of four packed rows, one in flight per wave, eight waves
        // (deeper rings, smaller or larger units, a successor requested ahead of use: all slower by 2 to 10 %)
        const int tu = tuning().stripe_unit, td = tuning().stripe_depth;
        const int unit = tu == 2 ? 2 : (tu == 8 && group % 64 == 0 ? 8 : 4), depth = td == 2 ? 2 : (td == 9 ? 0 : 1);
        if (bf16)
            e = launch_stripe_dyn(a, finish, b.sync, plan.waves_k, 4, 1, false, st);
        else
            e = launch_stripe_dyn(a, finish, b.sync, plan.waves_k, unit, depth, tuning().stripe_dot2 == 1, st);
    } else if (plan.kernel == W4A16_KERNEL_STRIPE) {
        e = launch_stripe(a, finish, b.sync, plan.waves_k, st);
    } else if (by_panel) {
        e = launch_panel(a, panel, st);
    } else if (by_pair) {
        e = launch_pair(a, finish, plan.tile_m, st);
    } else if (tile_ticket) {
        e = launch_tile_dyn(a, finish, b.sync, plan.waves_k, tuning().tile_depth == 2 && !bf16 && plan.waves_k <= 8 ? 2 : 1, unit_blocks, st);
    } else if (plan.kernel == W4A16_KERNEL_TILE && tile_four(plan.tile_m, group, bf16) && !short_slices(group, bf16, plan.groups_per_split)) {
        if (plan.tile_m == 64 && (bf16 || group != 128)) e = launch_tile_tall(a, finish, b.sync, st);
        else e = launch_tile_wide(a, finish, b.sync, plan.tile_m, st);
    } else if (plan.kernel == W4A16_KERNEL_TILE) {
        e = launch_tile(a, finish, b.sync, plan.tile_m, plan.waves_k, st);
    } else {
        e = launch_wave_split(a, plan.tile_n, st);
    }
    if (e == hipSuccess && finish == kFinishSecondPass && !by_panel) e = launch_reduce(a.partials, plan.split, M, N, a.Y, bf16, st);
    if (e != hipSuccess) {
        note_hip_error(e);
        if (b.library_acc) {  // what the failed launch left in the accumulator is unknown
            std::lock_guard<std::mutex> lock(g_mutex);
            g_dev[dev].acc_dirty = true;
        }
        return W4A16_ERR_HIP;
    }
    return W4A16_OK;
}

}  // namespace

extern "C" {

int w4a16_gemm(const void *X, const uint32_t *Wpacked, const void *scales, const uint32_t *zeros, int group, int M,
               int N, int K, void *Y, void *stream)
{
    return run("gemm", X, Wpacked, scales, zeros, group, M, N, K, Y, stream, W4A16_KERNEL_AUTO, 0, kFromLibrary, nullptr, 0);
}

int w4a16_gemm_ex(const void *X, const uint32_t *Wpacked, const void *scales, const uint32_t *zeros, int group, int M,
                  int N, int K, void *Y, void *stream, int kernel, int split)
{
    return run("gemm_ex", X, Wpacked, scales, zeros, group, M, N, K, Y, stream, kernel, split, kFromLibrary, nullptr, 0);
}

int w4a16_gemm_ws(const void *X, const uint32_t *Wpacked, const void *scales, const uint32_t *zeros, int group, int M,
                  int N, int K, void *Y, void *stream, int kernel, int split, void *workspace, size_t workspace_bytes)
{
    return run("gemm_ws", X, Wpacked, scales, zeros, group, M, N, K, Y, stream, kernel, split, kFromCall, workspace, workspace_bytes);
}

int w4a16_gemm_noalloc(const void *X, const uint32_t *Wpacked, const void *scales, const uint32_t *zeros, int group, int M,
                       int N, int K, void *Y, void *stream, int kernel, int split)
{
    return run("gemm_noalloc", X, Wpacked, scales, zeros, group, M, N, K, Y, stream, kernel, split, kFromScratch, nullptr, 0);
}

int w4a16_gemm_bf16(const void *X, const uint32_t *Wpacked, const void *scales, const uint32_t *zeros, int group, int M,
                    int N, int K, void *Y, void *stream, int kernel, int split)
{
    return run("gemm_bf16", X, Wpacked, scales, zeros, group, M, N, K, Y, stream, kernel, split, kFromLibrary, nullptr, 0, true);
}

size_t w4a16_scratch_bytes(int M, int N, int K, int group, int bf16)
{
    w4a16_plan p;
    if (M <= 16 || check_shape(group, M, N, K)) return 0;
    const int dev = current_device();
    if (dev >= 0) {  // a registered workspace is what the caller wants used, and nothing beside it
        std::lock_guard<std::mutex> lock(g_mutex);
        if (g_dev[dev].user_ws) return 0;
    }
    if (make_plan(M, N, K, group, W4A16_KERNEL_AUTO, 0, compute_units(dev), &p, nullptr, bf16 != 0)) return 0;
    const bool partials_only = p.kernel == W4A16_KERNEL_TILE && (p.tile_n == kPanelCols || p.tile_n == kPairCols);  // whatever is split there takes the second pass
    if (!partials_only && finish_of(p.kernel, M, N, p.split, burst_rows(p.tile_m, group, bf16 != 0, false)) != kFinishSecondPass) return 0;
    return p.workspace_bytes;
}

int w4a16_gemm_scratch(const void *X, const uint32_t *Wpacked, const void *scales, const uint32_t *zeros, int group, int M,
                       int N, int K, void *Y, void *stream, int bf16, void *scratch, size_t scratch_bytes)
{
    return run("gemm_scratch", X, Wpacked, scales, zeros, group, M, N, K, Y, stream, W4A16_KERNEL_AUTO, 0, kFromCall, scratch, scratch_bytes, bf16 != 0);
}

int w4a16_set_workspace(void *workspace, size_t workspace_bytes)
{
    if (workspace && (reinterpret_cast<uintptr_t>(workspace) & 255u)) return W4A16_ERR_ALIGN;
    if (workspace && workspace_bytes < 256) return W4A16_ERR_WORKSPACE;
    const int dev = current_device();
    if (dev < 0) { note_hip_error(hipErrorNoDevice); return W4A16_ERR_HIP; }
    std::lock_guard<std::mutex> lock(g_mutex);
    g_dev[dev].user_ws = workspace;
    g_dev[dev].user_ws_bytes = workspace ? workspace_bytes : 0;
    return W4A16_OK;
}

size_t w4a16_workspace_bytes(int M, int N, int K, int group)
{
    w4a16_plan p;
    if (check_shape(group, M, N, K)) return 0;
    if (make_plan(M, N, K, group, W4A16_KERNEL_AUTO, 0, compute_units(current_device()), &p)) return 0;
    return p.workspace_bytes ? p.workspace_bytes : 256;
}

int w4a16_query_plan(int M, int N, int K, int group, int kernel, int split, w4a16_plan *out)
{
    if (!out) return W4A16_ERR_NULL;
    int rc = check_shape(group, M, N, K);
    if (rc) return rc;
    return make_plan(M, N, K, group, kernel, split, compute_units(current_device()), out);
}

int w4a16_query_plan_bf16(int M, int N, int K, int group, int kernel, int split, w4a16_plan *out)
{
    if (!out) return W4A16_ERR_NULL;
    int rc = check_shape(group, M, N, K);
    if (rc) return rc;
    return make_plan(M, N, K, group, kernel, split, compute_units(current_device()), out, nullptr, true);
}

int w4a16_tune(const char *knob, int value)
{
    if (!knob) return W4A16_ERR_NULL;
    for (const Knob &k : kKnobs)
        if (strcmp(knob, k.name) == 0) {
            tuning().*(k.field) = value;
            return W4A16_OK;
        }
    return W4A16_ERR_UNSUPPORTED;
}

int w4a16_reduce(const float *partials, int S, int M, int N, void *Y, void *stream)
{
    t_hip_error[0] = 0;
    if (!partials || !Y) return W4A16_ERR_NULL;
    if (S < 1 || M < 1 || N < 8 || N % 8 != 0) return W4A16_ERR_SHAPE;
    if (!aligned16(partials) || !aligned16(Y)) return W4A16_ERR_ALIGN;
    hipError_t e = launch_reduce(partials, S, M, N, static_cast<uint16_t *>(Y), false, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) { note_hip_error(e); return W4A16_ERR_HIP; }
    return W4A16_OK;
}

int w4a16_dequant(const uint32_t *Wpacked, const void *scales, const uint32_t *zeros, int group, int N, int K,
                  void *W16, void *stream)
{
    t_hip_error[0] = 0;
    if (!Wpacked || !scales || !W16) return W4A16_ERR_NULL;  // zeros may be null: symmetric quantisation
    int rc = check_shape(group, 1, N, K);
    if (rc) return rc;
    if (!aligned16(Wpacked) || !aligned16(scales) || !aligned16(zeros) || !aligned16(W16)) return W4A16_ERR_ALIGN;
    hipError_t e = launch_dequant(Wpacked, static_cast<const uint16_t *>(scales), zeros, group, N, K,
                                  static_cast<uint16_t *>(W16), static_cast<hipStream_t>(stream));
    if (e != hipSuccess) { note_hip_error(e); return W4A16_ERR_HIP; }
    return W4A16_OK;
}

int w4a16_stream_probe(const void *a, size_t a_bytes, const void *b, size_t b_bytes, const void *c, size_t c_bytes, void *sink,
                       void *stream)
{
    t_hip_error[0] = 0;
    if (!sink || (!a && !b && !c)) return W4A16_ERR_NULL;
    if (!aligned16(a) || !aligned16(b) || !aligned16(c) || (reinterpret_cast<uintptr_t>(sink) & 3u)) return W4A16_ERR_ALIGN;
    const int dev = current_device();
    if (dev < 0) { note_hip_error(hipErrorNoDevice); return W4A16_ERR_HIP; }
    hipError_t e = launch_stream_probe(a, a ? a_bytes : 0, b, b ? b_bytes : 0, c, c ? c_bytes : 0, static_cast<uint32_t *>(sink),
                                       compute_units(dev), static_cast<hipStream_t>(stream));
    if (e != hipSuccess) { note_hip_error(e); return W4A16_ERR_HIP; }
    return W4A16_OK;
}

int w4a16_quantize(const void *W16, int group, int N, int K, uint32_t *Wpacked, void *scales, uint32_t *zeros,
                   void *stream)
{
    t_hip_error[0] = 0;
    if (!W16 || !Wpacked || !scales || !zeros) return W4A16_ERR_NULL;
    int rc = check_shape(group, 1, N, K);
    if (rc) return rc;
    if (!aligned16(W16) || !aligned16(Wpacked) || !aligned16(scales) || !aligned16(zeros)) return W4A16_ERR_ALIGN;
    hipError_t e = launch_quantize(static_cast<const uint16_t *>(W16), group, N, K, Wpacked, static_cast<uint16_t *>(scales),
                                   zeros, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) { note_hip_error(e); return W4A16_ERR_HIP; }
    return W4A16_OK;
}

const char *w4a16_status_string(int status)
{
    switch (status) {
    case W4A16_OK: return "ok";
    case W4A16_ERR_NULL: return "null pointer";
    case W4A16_ERR_SHAPE: return "bad shape (need M >= 1, N % 8 == 0, K % 8 == 0)";
    case W4A16_ERR_GROUP: return "bad group (need group % 32 == 0 and K % group == 0)";
    case W4A16_ERR_ALIGN: return "pointer not aligned (16 bytes for data, 256 for a workspace)";
    case W4A16_ERR_WORKSPACE: return "workspace too small, or it would have to be allocated while the stream is being captured, or allocation failed";
    case W4A16_ERR_HIP: return "HIP runtime error";
    case W4A16_ERR_UNSUPPORTED: return "forced kernel or split not valid for this shape, or the shape is beyond the kernels' 32-bit offsets";
    default: return "unknown status";
    }
}

const char *w4a16_last_hip_error(void) { return t_hip_error; }

void w4a16_shutdown(void)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    for (int d = 0; d < kMaxDevices; ++d) {
        DeviceState &s = g_dev[d];
        if (!s.ws && !s.acc && s.retired.empty()) continue;
        int prev = -1;
        if (hipGetDevice(&prev) == hipSuccess && hipSetDevice(d) == hipSuccess) {
            if (s.ws) (void)hipFree(s.ws);
            if (s.acc) (void)hipFree(s.acc);
            for (void *p : s.retired) (void)hipFree(p);
            (void)hipSetDevice(prev);
        }
        s.ws = nullptr;
        s.ws_bytes = 0;
        s.acc = nullptr;
        s.acc_bytes = 0;
        s.acc_dirty = false;
        s.retired.clear();
    }
}

}  // extern "C"
