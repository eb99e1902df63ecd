"""The TILE ticket kernel's forms by rows of X (compiled for 1, 2, 4, 8 and 16 rows) and by blocks per unit (groups of 32, 64
and 128), at their edges: every form keeps other outputs of the MFMA's result per lane."""
import numpy as np
import pytest

from oracle import w4a16_oracle as orc
from paper_2601_16536_amd import workloads as wl
from test_gpu_parity import err_ratio, gpu, run_gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("bf16", [False, True])
def test_every_form_gives_the_rows_of_the_largest(gpu, group, bf16):
    """Against the oracle at 16 rows; fewer rows give the same bits, as neither the rows of an MFMA nor the sums meet."""
    torch, binding = gpu
    G = {32: 35, 64: 19, 128: 6}[group]  # short groups: a last unit with fewer than its four or two of them
    K, N = G * group, 136  # two whole tiles and one of 8 columns
    X, Wp, s, Zp = wl.make(16, K, N, index=7100 + group, group=group)
    if bf16:
        X = wl.make_x_bf16(16, K, index=7100 + group)
    ref = (orc.gemm_bf16 if bf16 else orc.gemm)(X, Wp, s, Zp, group)
    dX, dW, dS, dZ = binding.to_device(X.view(np.float16), Wp, s, Zp)
    if bf16:
        dX = dX.view(torch.bfloat16)
    run = binding.gemm_bf16 if bf16 else binding.gemm_ex
    try:
        for split in (1, 2, 6):
            full = None
            for blocks in (0, 4):  # the scheduler's units; of several groups
                binding.tune("tile_unit", blocks)
                for M in (16, 9, 8, 7, 5, 4, 3, 2, 1):
                    say("ticket forms", "bf16" if bf16 else "fp16", "group", group, "blocks", blocks, "M", M, "split", split)
                    Y = torch.full((M, N), float("nan"), dtype=dX.dtype, device="cuda")
                    run(dX[:M].contiguous(), dW, dS, dZ, group, kernel=binding.KERNEL_TILE, split=split, out=Y)
                    torch.cuda.synchronize()
                    if full is None:
                        full = Y
                        assert err_ratio(Y.float().cpu().numpy(), ref) <= 1.0
                    assert torch.equal(Y.view(torch.int16), full[:M].view(torch.int16)), (M, split, blocks)
    finally:
        binding.tune("tile_unit", 0)


@pytest.mark.parametrize("group", [32, 64])
def test_last_unit_of_several_groups_reads_no_other_row(gpu, group):
    """A last unit with fewer groups than it has room for ends at the row's end: an infinity at the start of the next row of X
    stays in its row."""
    torch, binding = gpu
    K, N = 33 * 32 if group == 32 else 17 * 64, 72
    X, Wp, s, Zp = wl.make(8, K, N, index=7200 + group, group=group)
    X[1::2, :128] = np.inf
    clean = X.copy()
    clean[1::2] = 1.0
    out = []
    try:
        binding.tune("tile_unit", 4)
        for x in (X, clean):
            say("several groups, infinity in the next row", group)
            dX, dW, dS, dZ = binding.to_device(x, Wp, s, Zp)
            for M in (8, 4):
                Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
                out.append(binding.gemm_ex(dX[:M].contiguous(), dW, dS, dZ, group, kernel=binding.KERNEL_TILE, split=1, out=Y))
        torch.cuda.synchronize()
    finally:
        binding.tune("tile_unit", 0)
    for y, c in zip(out[:2], out[2:]):
        assert bool(torch.isfinite(y[::2]).all()) and torch.equal(y[::2], c[::2])
        assert bool(torch.isnan(y[1::2]).all())


@pytest.mark.parametrize("odd,step", [(1, 0), (3, 2), (5, 2)])
@pytest.mark.parametrize("kernel", ["TILE", "STRIPE"])
def test_contributions_halfway_between_two_steps(gpu, kernel, odd, step):
    """Units that contribute an odd multiple of 2^-25, halfway between two values of the exact sums: they round to the even one, by
    themselves, whatever has been summed before.  64 units in one column per sign: the sum is known."""
    torch, binding = gpu
    group, G, N = 128, 64, 16
    K = group * G
    q = np.full((K, N), 7 + odd, np.uint8)
    q[:, 1::2] = 7 - odd  # with z = 7: contributions of +odd and -odd times x s
    X = np.zeros((4, K), np.float16)
    X[:, ::group] = 2.0 ** -14
    s = np.full((G, N), 2.0 ** -11, np.float16)
    Wp, Zp = wl.pack_along_k(q), wl.pack_along_n(np.full((G, N), 7, np.uint8))
    for M in (1, 2, 4):
        for split in (1, 2, 8):
            say("halves", kernel, M, split)
            Y = run_gpu(gpu, X[:M], Wp, s, Zp, group, kernel=getattr(binding, "KERNEL_" + kernel), split=split).astype(np.float64)
            assert np.array_equal(Y[:, ::2], np.full((M, N // 2), 64 * step * 2.0 ** -24)), (M, split, Y)
            assert np.array_equal(Y[:, 1::2], np.full((M, N // 2), -64 * step * 2.0 ** -24)), (M, split, Y)


def _known_contributions(units, group):
    """X of 16 rows (the even ones +, the odd ones -), weights and scales such that group g of column n contributes units[g, n], a pair
    (kind, count): kind 0 is count times 2^-24, kind 1 count times 2^13, kind 2 count times 2^25; |count| <= 7.  All of Eq. 2 is exact."""
    kind, count = units
    G, N = kind.shape
    q = np.full((G * group, N), 7, np.uint8)  # z = 7
    q[::group] = np.where(kind < 2, 7 + count, 7)
    q[1::group] = np.where(kind == 2, 7 + count, 7)
    s = np.choose(kind, [2.0 ** -24, 2.0 ** 13, 2.0 ** 13]).astype(np.float16)
    X = np.zeros((16, G * group), np.float32)
    X[:, ::group], X[:, 1::group] = 1.0, 4096.0
    X[1::2] *= -1
    return X, wl.pack_along_k(q), s, wl.pack_along_n(np.full((G, N), 7, np.uint8))


def _steps_of(gpu, X, Wp, s, Zp, group, bf16, M, kernel, split):
    """Rows 0 .. M - 1 of the multiply, in units of 2^-24 and with the rows' signs taken out."""
    torch, binding = gpu
    dX, dW, dS, dZ = binding.to_device(X[:M].astype(np.float16), Wp, s, Zp)
    if bf16:
        dX = dX.to(torch.bfloat16)
    Y = torch.full((M, Wp.shape[1]), float("nan"), dtype=dX.dtype, device="cuda")
    (binding.gemm_bf16 if bf16 else binding.gemm_ex)(dX, dW, dS, dZ, group, kernel=kernel, split=split, out=Y)
    torch.cuda.synchronize()
    return Y.float().cpu().numpy().astype(np.float64) * 2.0 ** 24 * np.where(np.arange(M) % 2, -1, 1)[:, None]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("group", [32, 128])
def test_large_contributions_that_cancel_leave_the_small_ones(gpu, group, bf16):
    """Contributions of +-32768 (odd multiples of 2^39 steps) among ones of a few steps of 2^-24, in another order in every column: the
    large ones cancel and the small ones are whole, so that every order, and every share of the units among the waves, gives their sum."""
    torch, binding = gpu
    G, N, rng = 64, 200, np.random.default_rng(5)
    kind, count = np.zeros((G, N), np.int64), np.zeros((G, N), np.int64)
    for n in range(N):
        small = rng.integers(1, 4, 32)
        row = [(1, 4)] * 16 + [(1, -4)] * 16 + [(0, int(v)) for v in small]
        for g, at in enumerate(rng.permutation(G)):
            kind[g, n], count[g, n] = row[at]
    want = np.where(kind == 0, count, 0).sum(0).astype(np.float64)  # below 256: exact in both formats
    args = _known_contributions((kind, count), group)
    for kernel in ("TILE", "STRIPE"):
        for M in (1, 2, 4) if kernel == "STRIPE" else (1, 2, 4, 8, 16):
            for split in (1, 3):
                say("cancelling", kernel, "group", group, "bf16", bf16, "M", M, "split", split)
                for _ in range(3):
                    Y = _steps_of(gpu, *args, group, bf16, M, getattr(binding, "KERNEL_" + kernel), split)
                    assert np.array_equal(Y, np.tile(want, (M, 1))), (kernel, M, split, int((Y != want).sum()))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("knob", ["tile_unit", "stripe_waves"])
def test_sums_of_one_wave_beyond_the_clamp_and_back(gpu, knob, bf16):
    """A wave whose sum passes 1.5 2^27, four times the clamp of its final sum, and comes back has lost nothing: its sum is exact up to 2^29.
    One wave has all of it: a unit of four groups (TILE), or one wave per workgroup (STRIPE)."""
    torch, binding = gpu
    group, N, rng = 32, 72, np.random.default_rng(6)
    G = 8 * 4
    kind, count = np.zeros((G, N), np.int64), np.zeros((G, N), np.int64)
    for n in range(N):
        for u in range(0, G, 4):
            a, b = (int(v) for v in rng.integers(1, 4, 2))
            for g, (k, c) in zip(range(u, u + 4), rng.permutation([(2, 6), (2, -6), (0, a), (0, b)])):
                kind[g, n], count[g, n] = k, c
    want = np.where(kind == 0, count, 0).sum(0).astype(np.float64)
    args = _known_contributions((kind, count), group)
    kernel = binding.KERNEL_TILE if knob == "tile_unit" else binding.KERNEL_STRIPE
    try:
        binding.tune(knob, 4 if knob == "tile_unit" else 1)
        for M in (1, 2, 4) if knob == "stripe_waves" else (1, 2, 4, 8, 16):
            say("beyond the clamp and back", knob, "bf16", bf16, "M", M)
            Y = _steps_of(gpu, *args, group, bf16, M, kernel, 1)
            assert np.array_equal(Y, np.tile(want, (M, 1))), (M, int((Y != want).sum()))
    finally:
        binding.tune(knob, 0)


@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("bf16", [False, True])
def test_every_form_gives_the_same_bits_on_every_run(gpu, group, bf16):
    """Which wave takes which unit differs from run to run: the forms by rows, and the units of several groups, five times each."""
    torch, binding = gpu
    K, N = 40 * 128, 264
    X, Wp, s, Zp = wl.make(16, K, N, index=7300 + group, group=group)
    dX, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    if bf16:
        dX = dX.to(torch.bfloat16)
    run = binding.gemm_bf16 if bf16 else binding.gemm_ex
    for kernel in (binding.KERNEL_TILE, binding.KERNEL_STRIPE):
        for M in (1, 2, 4) if kernel == binding.KERNEL_STRIPE else (1, 2, 4, 8, 16):
            say("same bits", "bf16" if bf16 else "fp16", "group", group, "kernel", kernel, "M", M)
            x, first = dX[:M].contiguous(), None
            for _ in range(5):
                Y = torch.full((M, N), float("nan"), dtype=dX.dtype, device="cuda")
                run(x, dW, dS, dZ, group, kernel=kernel, split=2, out=Y)
                first = Y if first is None else first
                assert torch.equal(Y.view(torch.int16), first.view(torch.int16)), (kernel, M)


def test_most_columns_at_few_rows(gpu):
    """N = 2^22, more 64-column tiles than a grid's second dimension has: the multiply runs (as STRIPE) at 3 and 4 rows.  First and last
    columns against the oracle."""
    torch, binding = gpu
    K, N = 32, 1 << 22
    X, Wp, s, Zp = wl.make(4, K, 128, index=7400, group=K)
    dX, dW, dS, dZ = binding.to_device(X, Wp, s, Zp)
    W = torch.zeros((K // 8, N), dtype=torch.int32, device="cuda")
    S, Z = torch.zeros((1, N), dtype=torch.float16, device="cuda"), torch.zeros((1, N // 8), dtype=torch.int32, device="cuda")
    for big, small, n in ((W, dW, 64), (S, dS, 64), (Z, dZ, 8)):
        big[:, :n], big[:, -n:] = small[:, :n].view(big.dtype), small[:, -n:].view(big.dtype)
    ref = orc.gemm(X, Wp, s, Zp, K)
    for M in (3, 4):
        say("most columns", M)
        Y = binding.gemm(dX[:M].contiguous(), W, S, Z, K)
        torch.cuda.synchronize()
        got = torch.cat([Y[:, :64], Y[:, -64:]], 1).cpu().numpy()
        assert err_ratio(got, ref[:M]) <= 1.0, M
        assert bool((Y[:, 64:-64] == 0).all())


# M, K, N, group, blocks of 32 k per unit: both sides of every line of the rule (one workgroup per compute unit, K not split below 16384 columns)
UNITS = [(m, k, 8256, 32, 4 if k >= edge else 1) for m, edge in ((1, 1024), (4, 1024), (5, 1600), (8, 1600), (9, 3072), (16, 3072)) for k in (edge - 32, edge)] + \
        [(m, k, 8256, 64, 4 if k >= edge else 2) for m, edge in ((2, 1728), (3, 2048), (4, 2048), (8, 2816), (16, 14336)) for k in (edge - 64, edge)] + \
        [(4, 2048, 16448, 32, 1), (4, 2112, 16448, 64, 2), (16, 256, 8256, 128, 4)]


def test_units_of_several_groups_from_the_slices_where_they_are_faster(gpu, capfd):
    """Several groups per unit on long slices only, with no more workgroups than compute units: the rule as launched (the log's unit=)."""
    torch, binding = gpu
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sizes for 256 compute units")
    try:
        binding.tune("log", 1)
        for M, K, N, group, blocks in UNITS:
            X = torch.zeros((M, K), dtype=torch.float16, device="cuda")
            W = torch.zeros((K // 8, N), dtype=torch.int32, device="cuda")
            s = torch.zeros((K // group, N), dtype=torch.float16, device="cuda")
            capfd.readouterr()
            binding.gemm_ex(X, W, s, None, group, kernel=binding.KERNEL_TILE)
            torch.cuda.synchronize()
            line = capfd.readouterr().err
            assert "unit=%d\n" % blocks in line, (M, K, N, group, blocks, line)
    finally:
        binding.tune("log", 0)
