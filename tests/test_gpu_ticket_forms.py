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
    K, N = 6 * group, 136  # two whole tiles and one of 8 columns
    X, Wp, s, Zp = wl.make(16, K, N, index=7100 + group, group=group)
    if bf16:
        X = wl.make_x_bf16(16, K, index=7100 + group)
    ref = (orc.gemm_bf16 if bf16 else orc.gemm)(X, Wp, s, Zp, group)
    dX, dW, dS, dZ = binding.to_device(X.view(np.float16), Wp, s, Zp)
    if bf16:
        dX = dX.view(torch.bfloat16)
    run = binding.gemm_bf16 if bf16 else binding.gemm_ex
    for split in (1, 2, 6):
        full = None
        for M in (16, 9, 8, 7, 5, 4, 3, 2, 1):
            say("ticket forms", "bf16" if bf16 else "fp16", "group", group, "M", M, "split", split)
            Y = torch.full((M, N), float("nan"), dtype=dX.dtype, device="cuda")
            run(dX[:M].contiguous(), dW, dS, dZ, group, kernel=binding.KERNEL_TILE, split=split, out=Y)
            torch.cuda.synchronize()
            if full is None:
                full = Y
                assert err_ratio(Y.float().cpu().numpy(), ref) <= 1.0
            assert torch.equal(Y.view(torch.int16), full[:M].view(torch.int16)), (M, split)


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
