"""Which workgroup takes which (column tile and K slice, row block): csrc/w4a16_place.h, compiled for the host."""
import os
import subprocess

import numpy as np
import pytest

from oracle import w4a16_oracle as orc
from paper_2601_16536_amd import build
from paper_2601_16536_amd import workloads as wl

SOURCE = """
#define __host__
#define __device__
#include <cstdio>
#include <cstdlib>
#include "w4a16_place.h"
int main(int argc, char **argv)
{
    using namespace w4a16;
    for (int i = 1; i + 1 < argc; i += 2) {
        const int units = atoi(argv[i]), row_blocks = atoi(argv[i + 1]);
        long long grid;
        const Place p = place(units, row_blocks, &grid);
        const long long eighths = eighths_grid(units, row_blocks);
        for (int way = 0; way < 2; ++way) {
            const long long n = way ? eighths : grid;
            for (long long b = 0; b < n; ++b) {
                int unit, rb;
                const bool any = way ? place_in_eighths((unsigned)b, (unsigned)n, units, row_blocks, &unit, &rb) : place_of(p, (unsigned)b, units, &unit, &rb);
                if (any) printf("%d %d %d %d %lld %d %d\\n", units, row_blocks, way, p.eighth != 0, b, unit, rb);
            }
        }
    }
}
"""
# units and row blocks: fewer units than XCDs, multiples of eight and one more or less, several rounds, one row block
SHAPES = [(1, 2), (7, 3), (8, 7), (9, 16), (30, 7), (33, 5), (50, 5), (63, 4), (64, 4), (65, 4), (49, 3), (141, 3), (84, 6), (256, 2), (113, 9), (44, 1), (13, 40)]


@pytest.fixture(scope="module")
def placed(tmp_path_factory):
    folder = tmp_path_factory.mktemp("place")
    (folder / "place.cpp").write_text(SOURCE)
    program = str(folder / "place")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-I", build.CSRC, str(folder / "place.cpp"), "-o", program])
    out = subprocess.run([program] + [str(v) for shape in SHAPES for v in shape], stdout=subprocess.PIPE, check=True, text=True).stdout
    return np.array([[int(v) for v in line.split()] for line in out.splitlines()])


@pytest.mark.parametrize("units,row_blocks", SHAPES)
def test_every_row_block_of_every_unit_once(placed, units, row_blocks):
    for way in (0, 1):
        rows = placed[(placed[:, 0] == units) & (placed[:, 1] == row_blocks) & (placed[:, 2] == way)]
        pairs = rows[:, 5] * row_blocks + rows[:, 6]
        assert sorted(pairs) == list(range(units * row_blocks)) and (rows[:, 6] < row_blocks).all()


@pytest.mark.parametrize("units,row_blocks", [s for s in SHAPES if s[1] > 1])
def test_units_are_divided_among_xcds_only_where_that_saves_a_round(placed, units, row_blocks):
    """64-column tiles.  No XCD has a round of 32 workgroups more than an even share of the pairs, and where whole units per XCD keep to
    that too, the row blocks of a unit are on one XCD, next to each other."""
    rows = placed[(placed[:, 0] == units) & (placed[:, 1] == row_blocks) & (placed[:, 2] == 0)]
    per_xcd = np.bincount(rows[:, 4] % 8, minlength=8)
    even = -(-units * row_blocks // 8)
    assert -(-per_xcd.max() // 32) == -(-even // 32)
    whole = -(-units // 8) * row_blocks
    divided = -(-whole // 32) > -(-even // 32)
    assert bool(rows[0, 3]) == (divided or units % 8 == 0)  # (units by eights: eighths are whole units)
    if not divided:
        for unit in range(units):
            blocks = np.sort(rows[rows[:, 5] == unit, 4])
            assert (np.diff(blocks) == 8).all()
        assert per_xcd.max() - per_xcd.min() <= row_blocks


@pytest.mark.gpu
@pytest.mark.parametrize("rows,M,K,N,group", [(16, 48, 256, 5376, 128), (32, 190, 256, 5376, 128), (64, 300, 256, 3160, 128), (64, 300, 256, 3160, 32)])
def test_64_column_tiles_dealt_out_in_eighths(rows, M, K, N, group):
    """Units whose row blocks are on two XCDs (in whole units: tests of the other forms and tests/test_gpu_pair.py)."""
    import torch
    from paper_2601_16536_amd import binding
    X, Wp, s, Zp = wl.make(M, K, N, index=9970 + M, group=group)
    Xb = wl.make_x_bf16(M, K, index=9970 + M)
    _, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    for knob, value in (("tile_rows", rows), ("panel", 2), ("pair", 2)):
        binding.tune(knob, value)
    try:
        for x, ref in ((torch.from_numpy(X).cuda(), orc.gemm(X, Wp, s, Zp, group)),
                       (torch.from_numpy(Xb.view(np.int16)).cuda().view(torch.bfloat16), orc.gemm_bf16(Xb, Wp, s, Zp, group))):
            print("[case] eighths", rows, (M, K, N, group), x.dtype, flush=True)
            bf16 = x.dtype == torch.bfloat16
            p = binding.query_plan(M, N, K, group, binding.KERNEL_TILE, 1, bf16=bf16)
            assert (p["tile_n"], p["tile_m"]) == (64, rows)
            units, row_blocks = -(-N // 64), -(-M // rows)
            assert -(-(-(-units // 8) * row_blocks) // 32) > -(-(-(-units * row_blocks // 8)) // 32)
            Y = torch.full((M + 1, N), 7.0, dtype=x.dtype, device="cuda")  # a row beyond: not written
            (binding.gemm_bf16 if bf16 else binding.gemm_ex)(x, dW, dS, dZ, group, kernel=binding.KERNEL_TILE, split=1, out=Y[:M])
            torch.cuda.synchronize()
            err = np.abs(Y[:M].double().cpu().numpy() - ref) / (1e-2 * (1.0 + np.abs(ref)))
            assert float(err.max()) <= 1.0 and (Y[M] == 7.0).all()
    finally:
        for knob in ("tile_rows", "panel", "pair"):
            binding.tune(knob, 0)
