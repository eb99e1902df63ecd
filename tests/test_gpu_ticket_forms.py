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


@pytest.mark.parametrize("kernel", ["TILE", "STRIPE"])
def test_contributions_halfway_between_two_steps(gpu, kernel):
    """Units that contribute an odd multiple of 2^-25, halfway between two values of the exact sums: they round away from zero, by
    themselves, whatever has been summed before.  64 units in one column per sign: the sum is known."""
    torch, binding = gpu
    group, G, N = 128, 64, 16
    K = group * G
    q = np.full((K, N), 8, np.uint8)
    q[:, 1::2] = 6  # with z = 7: contributions of +1 and -1 times x s
    X = np.zeros((4, K), np.float16)
    X[:, ::group] = 2.0 ** -14
    s = np.full((G, N), 2.0 ** -11, np.float16)
    Wp, Zp = wl.pack_along_k(q), wl.pack_along_n(np.full((G, N), 7, np.uint8))
    for M in (1, 2, 4):
        for split in (1, 2, 8):
            say("halves", kernel, M, split)
            Y = run_gpu(gpu, X[:M], Wp, s, Zp, group, kernel=getattr(binding, "KERNEL_" + kernel), split=split).astype(np.float64)
            assert np.array_equal(Y[:, ::2], np.full((M, N // 2), 64 * 2.0 ** -24)), (M, split, Y)
            assert np.array_equal(Y[:, 1::2], np.full((M, N // 2), -64 * 2.0 ** -24)), (M, split, Y)
