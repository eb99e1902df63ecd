// Which workgroup works on what, where several row blocks of X share the weights of a column tile and K slice.
#pragma once

namespace w4a16 {

// Workgroup -> (unit, row block): a unit is a column tile and K slice, whose row blocks read the same weights.  Workgroup b runs on
// XCD b mod 8.  The row blocks of a unit are to be on one XCD, next to each other: they start together, and the second reader finds the
// weights in that XCD's L2.  Two ways to deal them out:
//   - whole units, neighbouring ones to an XCD (64-column tiles, wherever this fills no XCD for a round more than an even share would);
//   - an eighth of the (unit, row block) pairs to an XCD, in order, so that the units at its ends are on two: 50 column tiles of 5 row blocks
//     are 250 workgroups, but in whole units 35 on two of the XCDs, a second round on their 32 compute units (M = 300, K = 4096,
//     N = 3200, BF16: 29.3 us in whole units, 16.6 in eighths; M = 190, K = 8192, N = 5376 48.8 and 25.9; M = 48, K = 4096, N = 5376 (16 rows)
//     14.0 and 9.8).
// Where the rounds are the same, eighths lose: M = 104, K = 6912, N = 1888, groups of 256 (16 rows, 30 units of 7 row blocks) 13.8 us in whole units, 14.7 in
// eighths; of 4372 such drawn shapes at 16 and 32 rows of X per workgroup 335 were 2 to 7 % slower in eighths than with whole units dealt out one by
// one, and one is with neighbouring ones.  PAIR (w4a16_pair.hip) is in eighths throughout: with whole units within 1 % of that (3500 shapes).  One row block:
// units in launch order.
constexpr unsigned kPlaceXcds = 8, kPlaceUnits = 32;  // XCDs, and the compute units of each

inline long long eighths_grid(long long units, int row_blocks) { return (units * row_blocks + kPlaceXcds - 1) / kPlaceXcds * kPlaceXcds; }

// In eighths of the grid.  False: nothing to do (the grid is rounded up to whole rounds of XCDs).
__host__ __device__ inline bool place_in_eighths(unsigned block, unsigned blocks, int units, int row_blocks, int *unit, int *rb)
{
    *unit = (int)block;
    *rb = 0;
    if (row_blocks > 1) {
        const int per = (int)(blocks / kPlaceXcds), id = (int)(block % kPlaceXcds) * per + (int)(block / kPlaceXcds);
        *unit = id / row_blocks;
        *rb = id - *unit * row_blocks;
    }
    return *unit < units;
}

// Either way.
struct Place {
    unsigned row_blocks;
    unsigned eighth;  // pairs that an XCD takes; 0: whole units
};
inline Place place(long long units, int row_blocks, long long *grid)
{
    const long long whole = (units + kPlaceXcds - 1) / kPlaceXcds * row_blocks, eighth = eighths_grid(units, row_blocks) / kPlaceXcds;
    const bool by_units = units % kPlaceXcds != 0 && (whole + kPlaceUnits - 1) / kPlaceUnits == (eighth + kPlaceUnits - 1) / kPlaceUnits;  // (units by eights: eighths are whole units, without the last step below)
    *grid = (by_units ? whole : eighth) * kPlaceXcds;
    return {(unsigned)row_blocks, by_units ? 0u : (unsigned)eighth};
}
__host__ __device__ inline bool place_of(const Place &p, unsigned block, int units, int *unit, int *rb)
{
    *unit = (int)block;
    *rb = 0;
    if (__builtin_expect((int)p.row_blocks > 1, 1)) {  // (with other branches the prologue of a launch of many short workgroups shows: up to 2 %)
        const unsigned xcd = block % kPlaceXcds, id = block / kPlaceXcds + xcd * p.eighth;
        unsigned u = id / p.row_blocks;
        *rb = (int)(id - u * p.row_blocks);
        if (p.eighth == 0) {
            const unsigned each = (unsigned)units / kPlaceXcds, more = (unsigned)units % kPlaceXcds;  // the first `more` XCDs have a unit more
            u = u < each + (xcd < more ? 1 : 0) ? u + xcd * each + (xcd < more ? xcd : more) : (unsigned)units;  // (past the XCD's last unit: past them all)
        }
        *unit = (int)u;
    }
    return *unit < units;
}

}  // namespace w4a16
