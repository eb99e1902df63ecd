"""The form for many rows (tiles of 128 rows x 256 columns, w4a16_panel.hip) against the oracle at the edges of its tiles,
stages (128 k), slices and row blocks, in both formats and at every length of scale segment it has."""
import sys

import numpy as np
import pytest

from oracle import w4a16_oracle as orc
from paper_2601_16536_amd import workloads as wl

TOL = 1e-2


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2601_16536_amd import binding
    assert torch.cuda.is_available()
    binding.lib()
    return torch, binding


def err_ratio(Y, ref):
    return float(np.max(np.abs(Y - ref) / (TOL * (1.0 + np.abs(ref)))))


def pieces_of(p, M, N):
    """Pieces of rows (1, 2, 4) that a plan of 128 x 256 tiles cuts the tiles of 128 rows past the last whole round of 256 compute units into, from its
    workgroups; None where they, or the partials, one place per piece and slice, are those of no cut."""
    tiles_n = -(-N // 256)
    tiles, last_rows = -(-M // 128) * tiles_n, ((M - 1) % 128 + 32) // 32 * 32
    small, rest, S = tiles_n if last_rows < 128 else 0, tiles % 256, p["split"]
    for pieces in (1, 2, 4):
        if pieces > 1 and (rest <= small or (small and last_rows != 128 // pieces)):
            continue
        count = max(rest - small, 0) * pieces + min(rest, small)
        if p["workgroups"] == tiles - rest + count * S and p["workspace_bytes"] == (count * S * (128 * 256 // pieces) * 4 if S > 1 else 0):
            return pieces
    return None


def test_plans_beyond_128_rows_cover_the_problem():
    """Whatever the shape: slices cover K and none is empty, the grid is the whole tiles and the slices of the pieces, and the
    workspace is their FP32 partials, no more, and at most one tile per compute unit."""
    from paper_2601_16536_amd import binding
    rng = np.random.default_rng(7)
    seen = set()
    for _ in range(3000):
        group = int(rng.choice([32, 64, 96, 128, 256, 384]))
        G = int(rng.integers(1, 200))
        K, N, M = G * group, 8 * int(rng.integers(1, 3600)), int(rng.integers(129, 2500))
        p = binding.query_plan(M, N, K, group)
        assert p["kernel"] == binding.KERNEL_TILE
        if p["tile_n"] != 256:
            continue
        assert group != 96
        tiles = -(-M // 128) * -(-N // 256)
        S, gps = p["split"], p["groups_per_split"]
        assert S * gps >= G > (S - 1) * gps
        assert S == 1 or (gps * group) % 128 == 0
        pieces = pieces_of(p, M, N)
        assert pieces is not None
        assert p["workspace_bytes"] <= 256 * 128 * 256 * 4
        seen.add((S > 1, tiles < 256, pieces))
    assert seen >= {(False, False, 1), (True, False, 1), (True, True, 1), (False, False, 2), (False, True, 2), (False, False, 4), (True, False, 2), (True, False, 4)}


# M: last row blocks of 1, 32, 33, 64, 65, 96, 97, 128 rows; N: one column group, a tile less and more than one piece, several
# tiles; K: one stage, a slice that ends inside a stage (groups of 32 and 64), groups longer than a stage
CASES = [(129, 128, 8, 128), (160, 640, 248, 128), (161, 1024, 256, 64), (192, 832, 264, 64), (193, 64, 520, 64), (224, 96, 72, 32),
         (225, 1056, 512, 32), (256, 1280, 1032, 256), (385, 1152, 264, 384), (130, 2048, 768, 128), (65, 256, 520, 128), (17, 384, 264, 128)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,group", CASES)
def test_panel_against_the_oracle(gpu, M, K, N, group):
    torch, binding = gpu
    index = 9100 + M + K + N
    X, Wp, s, Zp = wl.make(M, K, N, index=index, group=group, outliers=K >= 128)
    Xb = wl.make_x_bf16(M, K, index=index)
    eights = wl.pack_along_n(np.full((K // group, N), 8, np.uint8))
    dX, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    dXb = torch.from_numpy(Xb.view(np.int16)).cuda().view(torch.bfloat16)
    refs = {(False, False): orc.gemm(X, Wp, s, Zp, group), (False, True): orc.gemm(X, Wp, s, eights, group),
            (True, False): orc.gemm_bf16(Xb, Wp, s, Zp, group), (True, True): orc.gemm_bf16(Xb, Wp, s, eights, group)}
    binding.tune("panel", 1)
    try:
        for split in (1, 2, 5, 0):  # of the tiles, where K has as many stages; 0: the planner's
            binding.tune("panel_split", split)
            for (bf16, symmetric), ref in refs.items():
                say("panel", (M, K, N, group), "split", split, "bf16" if bf16 else "fp16", "symmetric" if symmetric else "")
                Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16 if bf16 else torch.float16, device="cuda")
                (binding.gemm_bf16 if bf16 else binding.gemm)(dXb if bf16 else dX, dW, dS, None if symmetric else dZ, group, out=Y)
                first = Y.clone()
                Y.fill_(float("nan"))
                (binding.gemm_bf16 if bf16 else binding.gemm)(dXb if bf16 else dX, dW, dS, None if symmetric else dZ, group, out=Y)
                torch.cuda.synchronize()
                assert torch.equal(first, Y)
                assert err_ratio(Y.double().cpu().numpy(), ref) <= 1.0
    finally:
        binding.tune("panel", 0)
        binding.tune("panel_split", 0)


# Tiles of 128 rows cut into pieces of 64 and 32: a last row block of as many rows, none, and pieces that end at or past the last row
PIECES = [(2, 192, 1024, 264, 64), (2, 256, 640, 520, 128), (2, 225, 832, 248, 64), (4, 160, 1056, 512, 32), (4, 128, 1280, 264, 256),
          (4, 97, 384, 72, 128), (4, 481, 640, 1032, 128), (2, 320, 2048, 768, 128)]


@pytest.mark.gpu
@pytest.mark.parametrize("pieces,M,K,N,group", PIECES)
def test_panel_pieces_of_rows_against_the_oracle(gpu, pieces, M, K, N, group):
    torch, binding = gpu
    X, Wp, s, Zp = wl.make(M, K, N, index=9700 + M + K, group=group, outliers=True)
    Xb = wl.make_x_bf16(M, K, index=9700 + M + K)
    _, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    cases = [(torch.from_numpy(X).cuda(), orc.gemm(X, Wp, s, Zp, group)),
             (torch.from_numpy(Xb.view(np.int16)).cuda().view(torch.bfloat16), orc.gemm_bf16(Xb, Wp, s, Zp, group))]
    binding.tune("panel", 1)
    binding.tune("panel_pieces", pieces)
    try:
        for split in (1, 2, 3):
            binding.tune("panel_split", split)
            for x, ref in cases:
                say("panel pieces", pieces, (M, K, N, group), "split", split, x.dtype)
                plan = binding.query_plan(M, N, K, group, bf16=x.dtype == torch.bfloat16)
                assert plan["split"] == split and pieces_of(plan, M, N) == pieces
                Y = torch.full((M + 1, N), 7.0, dtype=x.dtype, device="cuda")  # a row beyond: not written
                (binding.gemm_bf16 if x.dtype == torch.bfloat16 else binding.gemm)(x, dW, dS, dZ, group, out=Y[:M])
                torch.cuda.synchronize()
                assert err_ratio(Y[:M].double().cpu().numpy(), ref) <= 1.0 and (Y[M] == 7.0).all()
    finally:
        for knob in ("panel", "panel_pieces", "panel_split"):
            binding.tune(knob, 0)


# Whole tiles before the cut ones (43 column tiles, six or seven row blocks, 256 whole): two tiles of 128 rows and a shorter row block, or 45 of 128 rows
MIXED = [(4, 777, (1, 2, 5)), (2, 832, (1, 2, 3)), (2, 896, (1, 2)), (4, 896, (1,)), (1, 777, (2, 3)), (1, 896, (5,))]


@pytest.mark.gpu
@pytest.mark.parametrize("pieces,M,splits", MIXED)
def test_panel_whole_tiles_and_pieces_of_others(gpu, pieces, M, splits):
    """Every output against 64-bit sums; with a workspace of just the plan's size, beyond which nothing is written."""
    torch, binding = gpu
    K, N, group = 640, 11008, 64
    gen = torch.Generator(device="cuda").manual_seed(M + pieces)
    words = lambda *shape: torch.randint(-(1 << 31), 1 << 31, shape, dtype=torch.int32, device="cuda", generator=gen)
    X, Wp, Zp = torch.randn((M, K), device="cuda", generator=gen), words(K // 8, N), words(K // group, N // 8)
    s = torch.rand((K // group, N), device="cuda", generator=gen).to(torch.float16) * 0.019 + 0.001
    shift = torch.arange(0, 32, 4, device="cuda", dtype=torch.int32)
    q = ((Wp.unsqueeze(1) >> shift.view(1, 8, 1)) & 15).reshape(K, N).double()
    z = ((Zp.unsqueeze(2) >> shift.view(1, 1, 8)) & 15).reshape(K // group, N).double()
    W = (q - z.repeat_interleave(group, 0)) * s.double().repeat_interleave(group, 0)
    binding.tune("panel", 1)
    binding.tune("panel_pieces", pieces)
    try:
        for split in splits:
            binding.tune("panel_split", split)
            for dtype in (torch.float16, torch.bfloat16):
                say("whole tiles and pieces", pieces, M, "split", split, dtype)
                bf16, x = dtype == torch.bfloat16, X.to(dtype)
                plan = binding.query_plan(M, N, K, group, bf16=bf16)
                assert plan["split"] == split and pieces_of(plan, M, N) == pieces and plan["workgroups"] > 256
                size = plan["workspace_bytes"]
                ws = torch.full((size + 4096,), 0x55, dtype=torch.uint8, device="cuda")
                Y = torch.full((M + 1, N), 7.0, dtype=dtype, device="cuda")
                rc = binding.lib().w4a16_gemm_scratch(x.data_ptr(), Wp.data_ptr(), s.data_ptr(), Zp.data_ptr(), group, M, N, K, Y.data_ptr(),
                                                      torch.cuda.current_stream().cuda_stream, int(bf16), ws.data_ptr(), size)
                assert rc == binding.OK
                torch.cuda.synchronize()
                ref = x.double() @ W
                assert float(((Y[:M].double() - ref).abs() / (TOL * (1.0 + ref.abs()))).max()) <= 1.0 and bool((Y[M] == 7.0).all())
                assert bool((ws[size:] == 0x55).all()) and (split == 1 or bool((ws[:size] != 0x55).any()))
    finally:
        for knob in ("panel", "panel_pieces", "panel_split"):
            binding.tune(knob, 0)


@pytest.mark.gpu
def test_panel_whole_numbers_and_rows_that_are_not_finite(gpu):
    """Scales that are powers of two and small whole X: every output is exact.  A row of NaN or infinities stays in its own
    row, also where a slice's last stage reaches beyond K (K = 832, groups of 64: half a stage)."""
    torch, binding = gpu
    M, K, N, group = 257, 832, 264, 64
    rng = np.random.default_rng(5)
    _, Wp, _, Zp = wl.make(1, K, N, index=9300, group=group)
    s = (2.0 ** rng.integers(-8, -3, (K // group, N))).astype(np.float16)
    X = rng.integers(-3, 4, (M, K)).astype(np.float16)
    want = orc.to_fp16(orc.gemm(X, Wp, s, Zp, group))
    X[100], X[256] = np.nan, np.inf
    _, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    binding.tune("panel", 1)
    try:
        for split in (1, 3):
            for dtype in (torch.float16, torch.bfloat16):
                say("panel whole numbers", split, dtype)
                binding.tune("panel_split", split)
                dX = torch.from_numpy(X).cuda().to(dtype)
                Y = torch.full((M, N), 7.0, dtype=dtype, device="cuda")
                (binding.gemm if dtype == torch.float16 else binding.gemm_bf16)(dX, dW, dS, dZ, group, out=Y)
                out = Y.float().cpu().numpy()
                assert np.isnan(out[100]).all() and not np.isfinite(out[256]).any()
                keep = [m for m in range(M) if m not in (100, 256)]
                ref = want.astype(np.float32) if dtype == torch.float16 else torch.from_numpy(want).to(torch.float32).to(dtype).float().numpy()
                if dtype == torch.bfloat16:  # the sums are exact in FP32 and have more bits than the format: one rounding
                    exact = orc.gemm(np.nan_to_num(X, nan=0, posinf=0), Wp, s, Zp, group)
                    ref = torch.from_numpy(exact).to(torch.float32).to(dtype).float().numpy()
                assert np.array_equal(out[keep], ref[keep])
    finally:
        binding.tune("panel", 0)
        binding.tune("panel_split", 0)


@pytest.mark.gpu
def test_panel_without_room_for_its_partials(gpu):
    """A plan that would split runs without the split where its workspace is not to be had: brought by the call and too small,
    registered and too small, the array of the entry point that allocates nothing, and a capture with each.  The same bits as
    the unsplit plan."""
    torch, binding = gpu
    M, K, N = 400, 4096, 7168
    plan = binding.query_plan(M, N, K, 128)
    assert plan["tile_n"] == 256 and plan["split"] > 1 and plan["workspace_bytes"] > 4 << 20, plan
    X, Wp, s, Zp = wl.make(M, K, N, index=9400)
    ref = orc.gemm(X, Wp, s, Zp, 128)
    args = binding.to_device(X, Wp, s, Zp)
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    binding.gemm(*args, 128, out=Y)  # with scratch of its own: split
    assert err_ratio(Y.double().cpu().numpy(), ref) <= 1.0
    binding.tune("panel_split", 1)
    try:
        assert binding.query_plan(M, N, K, 128)["tile_n"] == 256
        unsplit = binding.gemm(*args, 128)
    finally:
        binding.tune("panel_split", 0)
    assert err_ratio(unsplit.double().cpu().numpy(), ref) <= 1.0
    ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")

    def through_c():
        st = torch.cuda.current_stream().cuda_stream
        assert binding.raw_gemm(*[t.data_ptr() for t in args], 128, M, N, K, Y.data_ptr(), st) == binding.OK

    binding.set_workspace(ws)
    try:
        for name, call in (("its own", lambda: binding.gemm_ws(*args, 128, ws, out=Y)), ("registered", through_c),
                           ("registered, binding", lambda: binding.gemm(*args, 128, out=Y)),
                           ("noalloc", lambda: binding.gemm_noalloc(*args, 128, out=Y))):
            say("panel without room", name)
            Y.fill_(float("nan"))
            call()
            torch.cuda.synchronize()
            assert torch.equal(Y, unsplit)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                call()
            for _ in range(3):
                Y.fill_(float("nan"))
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(Y, unsplit)
    finally:
        binding.set_workspace(None)


@pytest.mark.gpu
def test_panel_gives_way_to_tiles_that_need_less(gpu):
    """M = 48, K = 14336, N = 7168: the 256-column plan needs more than the 4 MiB of the entry point that allocates nothing and would
    be slow unsplit; there, and in a workspace of the 64-column plan's size, the 64-column plan runs, with its own finish."""
    torch, binding = gpu
    M, K, N = 48, 14336, 7168
    plan = binding.query_plan(M, N, K, 128)
    assert plan["tile_n"] == 256 and plan["workspace_bytes"] > 4 << 20, plan
    binding.tune("panel", 2)
    small = binding.query_plan(M, N, K, 128)
    binding.tune("panel", 0)
    assert small["split"] > 1 and 0 < small["workspace_bytes"] <= 4 << 20, small
    X, Wp, s, Zp = wl.make(M, K, N, index=9410)
    rows = [0, 31, 32, 47]
    ref = orc.gemm(np.ascontiguousarray(X[rows]), Wp, s, Zp, 128)
    args = binding.to_device(X, Wp, s, Zp)
    ws = torch.empty(small["workspace_bytes"], dtype=torch.uint8, device="cuda")
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    outs = []
    for name, call in (("noalloc", lambda: binding.gemm_noalloc(*args, 128, out=Y)), ("workspace", lambda: binding.gemm_ws(*args, 128, ws, out=Y)),
                       ("256 columns", lambda: binding.gemm(*args, 128, out=Y))):
        say("less room", name)
        Y.fill_(float("nan"))
        call()
        torch.cuda.synchronize()
        outs.append(Y.clone())
        assert err_ratio(Y.double().cpu().numpy()[rows], ref) <= 1.0
    assert torch.equal(outs[0], outs[1])


# Beyond eight row blocks of 128 the tiles are numbered in bands of eight: a second band, a shorter last one, a last block of 33 rows,
# several column tiles, split tiles on both sides of a band's edge
BANDS = [(1185, 128, 520, 64), (1100, 384, 264, 128), (1281, 256, 776, 32), (2049, 160, 520, 32)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,group", BANDS)
def test_panel_bands_of_row_blocks_against_the_oracle(gpu, M, K, N, group):
    torch, binding = gpu
    X, Wp, s, Zp = wl.make(M, K, N, index=9500 + M, group=group)
    Xb = wl.make_x_bf16(M, K, index=9500 + M)
    _, dW, dS, dZ = binding.to_device(X[:1], Wp, s, Zp)
    dX, dXb = torch.from_numpy(X).cuda(), torch.from_numpy(Xb.view(np.int16)).cuda().view(torch.bfloat16)
    refs = orc.gemm(X, Wp, s, Zp, group), orc.gemm_bf16(Xb, Wp, s, Zp, group)
    binding.tune("panel", 1)
    try:
        for split in (1, 2):
            binding.tune("panel_split", split)
            plan = binding.query_plan(M, N, K, group)
            assert plan["tile_n"] == 256 and plan["split"] == (split if K > 128 else 1)
            for x, gemm, ref in ((dX, binding.gemm, refs[0]), (dXb, binding.gemm_bf16, refs[1])):
                say("panel bands", (M, K, N, group), "split", split, x.dtype)
                Y = torch.full((M, N), float("nan"), dtype=x.dtype, device="cuda")
                gemm(x, dW, dS, dZ, group, out=Y)
                assert err_ratio(Y.double().cpu().numpy(), ref) <= 1.0
    finally:
        binding.tune("panel", 0)
        binding.tune("panel_split", 0)


# K: fewer stages than waves, a run that ends inside a stage, runs of unequal length, groups longer than a stage
TALL = [(64, 128, 64, 128), (33, 640, 72, 128), (128, 832, 136, 64), (65, 96, 264, 32), (100, 1056, 200, 32), (130, 1536, 64, 384),
        (70, 5376, 1032, 128), (61, 2048, 2056, 256)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,group", TALL)
def test_sixty_four_rows_per_workgroup_against_the_oracle(gpu, M, K, N, group):
    """The 64-row form (w4a16_tile_tall.hip) in both formats, with its three finishes: direct, accumulator, second pass."""
    torch, binding = gpu
    index = 9600 + M + K + N
    X, Wp, s, Zp = wl.make(M, K, N, index=index, group=group)
    Xb = wl.make_x_bf16(M, K, index=index)
    eights = wl.pack_along_n(np.full((K // group, N), 8, np.uint8))
    _, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    dX, dXb = torch.from_numpy(X).cuda(), torch.from_numpy(Xb.view(np.int16)).cuda().view(torch.bfloat16)
    G = K // group
    binding.tune("tile_rows", 64)
    try:
        for split in sorted({1, min(2, G), min(5, G)}):
            for finish in ((0,) if split == 1 else (1, 2)):
                binding.tune("stripe_finish", finish)
                for bf16, zeros, zp in ((False, dZ, Zp), (True, dZ, Zp), (False, None, eights), (True, None, eights)):
                    say("64 rows", (M, K, N, group), "split", split, "finish", finish, "bf16" if bf16 else "fp16", "zeros" if zeros is not None else "symmetric")
                    plan = binding.query_plan(M, N, K, group, binding.KERNEL_TILE, split)
                    assert plan["tile_m"] == 64 and plan["waves_k"] == 4
                    ref = orc.gemm_bf16(Xb, Wp, s, zp, group) if bf16 else orc.gemm(X, Wp, s, zp, group)
                    outs = []
                    for _ in range(2):
                        Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16 if bf16 else torch.float16, device="cuda")
                        (binding.gemm_bf16 if bf16 else binding.gemm_ex)(dXb if bf16 else dX, dW, dS, zeros, group, kernel=binding.KERNEL_TILE, split=split, out=Y)
                        torch.cuda.synchronize()
                        outs.append(Y)
                    assert torch.equal(outs[0], outs[1])
                    assert err_ratio(outs[0].double().cpu().numpy(), ref) <= 1.0
    finally:
        binding.tune("tile_rows", 0)
        binding.tune("stripe_finish", 0)


@pytest.mark.gpu
def test_sixty_four_rows_keep_rows_that_are_not_finite_apart(gpu):
    torch, binding = gpu
    M, K, N, group = 66, 480, 72, 32  # the slice ends inside a stage, and row 65's X starts where row 64's ends
    X, Wp, s, Zp = wl.make(M, K, N, index=9700, group=group)
    X[64], X[65, ::2] = 0.5, np.nan
    ref = orc.gemm(X[:65], Wp, s, Zp, group)
    args = binding.to_device(X, Wp, s, Zp)
    binding.tune("tile_rows", 64)
    try:
        for split in (1, 3):
            say("64 rows, NaN in one row", split)
            Y = binding.gemm_ex(*args, group, kernel=binding.KERNEL_TILE, split=split).double().cpu().numpy()
            assert np.isnan(Y[65]).all() and err_ratio(Y[:65], ref) <= 1.0
    finally:
        binding.tune("tile_rows", 0)


@pytest.mark.gpu
def test_sixty_four_rows_where_the_partials_have_no_room(gpu):
    """A 64-row plan whose slices go to FP32 partials, with a workspace that holds them, one that holds 64-bit sums only, and
    one that holds neither: the plans that need less."""
    torch, binding = gpu
    M, K, N, group = 91, 5696, 1408, 64
    plan = binding.query_plan(M, N, K, group)
    assert plan["tile_m"] == 64 and plan["split"] > 1 and plan["workspace_bytes"] > M * N * 8, plan
    X, Wp, s, Zp = wl.make(M, K, N, index=9800, group=group)
    ref = orc.gemm(X, Wp, s, Zp, group)
    args = binding.to_device(X, Wp, s, Zp)
    for size in (plan["workspace_bytes"], M * N * 8, 256):
        say("64 rows, workspace of", size)
        ws = torch.full((size + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        ws = ws[-ws.data_ptr() % 256:][:size]
        Y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        binding.gemm_ws(*args, group, ws, out=Y)
        assert err_ratio(Y.double().cpu().numpy(), ref) <= 1.0


@pytest.mark.gpu
def test_prompts_on_two_streams_at_once(gpu):
    """Shapes whose 64-column plan needs no buffer may overlap: calls of different inputs on two streams, through the binding
    (a scratch of each call's own) and through the C entry (a plan that needs none), give what they give one at a time."""
    torch, binding = gpu
    M, K, N = 400, 4096, 7168
    assert binding.query_plan(M, N, K, 128)["workspace_bytes"] > 0
    _, Wp, s, Zp = wl.make(1, K, N, index=9900)
    _, dW, dS, dZ = binding.to_device(np.zeros((1, K), np.float16), Wp, s, Zp)
    Xs = [torch.from_numpy(wl.make_x(M, K, index=9901 + i)).cuda() for i in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]

    def through_binding(X, Y, st):
        with torch.cuda.stream(st):
            binding.gemm(X, dW, dS, dZ, 128, out=Y)

    def through_c(X, Y, st):
        assert binding.raw_gemm(X.data_ptr(), dW.data_ptr(), dS.data_ptr(), dZ.data_ptr(), 128, M, N, K, Y.data_ptr(), st.cuda_stream) == binding.OK

    for call in (through_binding, through_c):
        say("two streams", call.__name__)
        alone = []
        for X in Xs:
            Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
            torch.cuda.synchronize()
            call(X, Y, streams[0])
            torch.cuda.synchronize()
            alone.append(Y)
        outs = [[torch.empty((M, N), dtype=torch.float16, device="cuda") for _ in range(6)] for _ in Xs]
        torch.cuda.synchronize()
        for r in range(6):
            for X, Y, st in zip(Xs, outs, streams):
                call(X, Y[r], st)
        torch.cuda.synchronize()
        for want, got in zip(alone, outs):
            assert all(torch.equal(want, Y) for Y in got)
    assert err_ratio(alone[0].double().cpu().numpy()[:8], orc.gemm(wl.make_x(M, K, index=9901)[:8], Wp, s, Zp, 128)) <= 1.0
