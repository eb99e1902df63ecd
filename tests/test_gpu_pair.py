"""Tiles of 32 or 64 rows x 128 columns (w4a16_pair.hip) against the oracle at the edges of its tiles, chunks, runs and slices, and the
TILE forms with several row blocks where the column tiles are no multiple of the eight XCDs."""
import sys

import numpy as np
import pytest

from oracle import w4a16_oracle as orc
from paper_2601_16536_amd import workloads as wl

TOL = 1e-2
KNOBS = ("pair", "pair_split", "tile_rows", "panel")


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture
def gpu():
    import torch
    from paper_2601_16536_amd import binding
    assert torch.cuda.is_available()
    binding.lib()
    yield torch, binding
    for knob in KNOBS:
        binding.tune(knob, 0)


def test_plans_of_128_columns_cover_the_problem():
    """Whatever the shape: slices cover K and none is empty, no more workgroups than compute units where K is split, and the
    workspace is the FP32 partials."""
    from paper_2601_16536_amd import binding
    rng = np.random.default_rng(11)
    seen = set()
    for _ in range(3000):
        group = int(rng.choice([32, 64, 96, 128, 256, 384]))
        G = int(rng.integers(1, 300))
        K, N, M = G * group, 8 * int(rng.integers(1, 3600)), int(rng.integers(1, 700))
        bf16 = bool(rng.integers(0, 2))
        p = binding.query_plan(M, N, K, group, bf16=bf16)
        if p["tile_n"] != 128:
            continue
        assert M > 16 and group != 96 and p["tile_m"] in (32, 64) and p["threads"] == 512
        S, gps = p["split"], p["groups_per_split"]
        assert S * gps >= G > (S - 1) * gps
        assert p["workgroups"] == -(-N // 128) * -(-M // p["tile_m"]) * S and (S == 1 or p["workgroups"] <= 256)
        assert p["workspace_bytes"] == (S * M * N * 4 if S > 1 else 0)
        seen.add((p["tile_m"], S > 1))
    assert len(seen) == 4


@pytest.mark.parametrize("M,K,N,group,bf16,tile_n", [
    (155, 27200, 5624, 64, True, 256), (154, 11648, 6120, 128, True, 256), (194, 8960, 8088, 128, True, 256),  # slices of PANEL: 4 to 10 % faster than PAIR
    (1027, 17984, 3952, 64, True, 256), (393, 17152, 9648, 64, True, 256),  # unsplit PANEL: 9 %
    (141, 1536, 3576, 128, False, 64), (135, 1536, 3352, 128, False, 64),  # unsplit tiles of 16 rows: 7 %
    (24, 9472, 10840, 128, True, 128), (348, 4992, 2760, 128, True, 128), (37, 10240, 4608, 64, False, 128), (20, 4096, 16616, 256, False, 128), (28, 13312, 15912, 256, True, 128),
    (467, 20224, 968, 32, True, 128), (69, 17408, 1480, 128, False, 128), (26, 21760, 3456, 128, True, 128), (480, 2048, 4112, 256, True, 128)])  # PAIR: 2 to 35 % faster
def test_the_faster_form_is_chosen(M, K, N, group, bf16, tile_n):
    """Timed both ways; PAIR's model alone has it a little cheaper on all of them."""
    from paper_2601_16536_amd import binding
    assert binding.query_plan(M, N, K, group, bf16=bf16)["tile_n"] == tile_n


def is_pair(plan, K, group, rows, split):
    """Whether a plan is tiles of `rows` x 128 in `split` slices, or as many as K has groups for."""
    gps = -(-(K // group) // min(split, K // group))
    return (plan["tile_n"], plan["tile_m"], plan["threads"], plan["split"]) == (128, rows, 512, -(-(K // group) // gps))


# M: row blocks of 1, 31, 32 rows and one more (with 64 rows to a tile: up to half of it); N: one column group, either half of a tile, a tile and more; K: less than the four runs,
# runs of unequal length, a chunk that the matrix ends in (groups of 32), groups longer than a run
CASES = [(17, 128, 8, 128), (32, 64, 64, 64), (33, 96, 72, 32), (64, 1280, 136, 128), (65, 1056, 264, 32), (31, 832, 120, 64),
         (100, 2176, 520, 128), (130, 2304, 392, 384), (50, 3072, 256, 256), (97, 640, 1032, 64)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,group", CASES)
def test_pair_against_the_oracle(gpu, M, K, N, group):
    torch, binding = gpu
    index = 9800 + M + K + N
    X, Wp, s, Zp = wl.make(M, K, N, index=index, group=group, outliers=K >= 128)
    Xb = wl.make_x_bf16(M, K, index=index)
    eights = wl.pack_along_n(np.full((K // group, N), 8, np.uint8))
    dX, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    dXb = torch.from_numpy(Xb.view(np.int16)).cuda().view(torch.bfloat16)
    refs = {(False, False): orc.gemm(X, Wp, s, Zp, group), (False, True): orc.gemm(X, Wp, s, eights, group),
            (True, False): orc.gemm_bf16(Xb, Wp, s, Zp, group), (True, True): orc.gemm_bf16(Xb, Wp, s, eights, group)}
    binding.tune("pair", 1)
    for rows in (32, 64):
        binding.tune("tile_rows", rows)
        for split in (1, 2, 3):
            binding.tune("pair_split", split)
            for (bf16, symmetric), ref in refs.items():
                say("pair", (M, K, N, group), "rows", rows, "split", split, "bf16" if bf16 else "fp16", "symmetric" if symmetric else "")
                assert is_pair(binding.query_plan(M, N, K, group, bf16=bf16), K, group, rows, split)
                Y = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16 if bf16 else torch.float16, device="cuda")  # a row beyond: not written
                gemm = binding.gemm_bf16 if bf16 else binding.gemm
                gemm(dXb if bf16 else dX, dW, dS, None if symmetric else dZ, group, out=Y[:M])
                first = Y.clone()
                Y.fill_(7.0)
                gemm(dXb if bf16 else dX, dW, dS, None if symmetric else dZ, group, out=Y[:M])
                torch.cuda.synchronize()
                assert torch.equal(first, Y) and (Y[M] == 7.0).all()
                err = np.abs(Y[:M].double().cpu().numpy() - ref) / (TOL * (1.0 + np.abs(ref)))
                assert float(err.max()) <= 1.0


@pytest.mark.gpu
def test_pair_whole_numbers_and_rows_that_are_not_finite(gpu):
    """Scales that are powers of two and small whole X: every output is exact.  A row of NaN or infinities stays in its own row, also
    where the matrix ends inside a chunk."""
    torch, binding = gpu
    M, K, N, group = 75, 928, 264, 32
    rng = np.random.default_rng(6)
    _, Wp, _, Zp = wl.make(1, K, N, index=9900, group=group)
    s = (2.0 ** rng.integers(-8, -3, (K // group, N))).astype(np.float16)
    X = rng.integers(-3, 4, (M, K)).astype(np.float16)
    exact = orc.gemm(X, Wp, s, Zp, group)
    X[40], X[74] = np.nan, np.inf
    _, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    keep = [m for m in range(M) if m not in (40, 74)]
    binding.tune("pair", 1)
    for rows in (32, 64):
        for split in (1, 3):
            for dtype in (torch.float16, torch.bfloat16):
                say("pair whole numbers", rows, split, dtype)
                binding.tune("tile_rows", rows)
                binding.tune("pair_split", split)
                assert is_pair(binding.query_plan(M, N, K, group, bf16=dtype == torch.bfloat16), K, group, rows, split)
                Y = torch.full((M, N), 7.0, dtype=dtype, device="cuda")
                (binding.gemm if dtype == torch.float16 else binding.gemm_bf16)(torch.from_numpy(X).cuda().to(dtype), dW, dS, dZ, group, out=Y)
                out = Y.float().cpu().numpy()
                assert np.isnan(out[40]).all() and not np.isfinite(out[74]).any()
                assert np.array_equal(out[keep], torch.from_numpy(exact).to(torch.float32).to(dtype).float().numpy()[keep])


@pytest.mark.gpu
@pytest.mark.parametrize("rows,M,K,N,group", [(16, 40, 512, 328, 128), (32, 90, 1024, 456, 128), (32, 90, 512, 264, 64), (64, 200, 1024, 584, 128),
                                              (64, 130, 768, 200, 32)])
def test_row_blocks_of_column_tiles_that_are_no_multiple_of_eight(gpu, rows, M, K, N, group):
    torch, binding = gpu
    X, Wp, s, Zp = wl.make(M, K, N, index=9950 + M, group=group)
    Xb = wl.make_x_bf16(M, K, index=9950 + M)
    _, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    binding.tune("tile_rows", rows)
    binding.tune("panel", 2)
    binding.tune("pair", 2)
    for x, ref in ((torch.from_numpy(X).cuda(), orc.gemm(X, Wp, s, Zp, group)),
                   (torch.from_numpy(Xb.view(np.int16)).cuda().view(torch.bfloat16), orc.gemm_bf16(Xb, Wp, s, Zp, group))):
        for split in (1, 2):
            say("row blocks", rows, (M, K, N, group), split, x.dtype)
            plan = binding.query_plan(M, N, K, group, binding.KERNEL_TILE, split, bf16=x.dtype == torch.bfloat16)
            assert (plan["tile_n"], plan["tile_m"], plan["split"]) == (64, rows, split)
            Y = torch.full((M + 1, N), 7.0, dtype=x.dtype, device="cuda")
            f = binding.gemm_bf16 if x.dtype == torch.bfloat16 else binding.gemm_ex
            f(x, dW, dS, dZ, group, kernel=binding.KERNEL_TILE, split=split, out=Y[:M])
            torch.cuda.synchronize()
            err = np.abs(Y[:M].double().cpu().numpy() - ref) / (TOL * (1.0 + np.abs(ref)))
            assert float(err.max()) <= 1.0 and (Y[M] == 7.0).all()
