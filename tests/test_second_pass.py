"""The second pass alone: FP32 partials added in slice order, then one rounding."""
import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("S", list(range(1, 18)) + [24, 31, 32, 33])
def test_every_number_of_slices_is_added_in_order(S):
    """Eight slices' loads are in flight, and the one to seven left over together: the bits of one addition after another, whatever S.
    The last row's sums cancel: another order would show."""
    import torch
    from paper_2601_16536_amd import binding
    M, N = 5, 328  # 410 threads: a second workgroup that is not full
    rng = np.random.default_rng(S)
    P = rng.standard_normal((S, M, N)).astype(np.float32) * np.float32(2.0) ** rng.integers(-6, 7, (S, M, N)).astype(np.float32)
    if S > 1:
        P[-1, M - 1] = -P[0, M - 1]
    acc = P[0].copy()
    for s in range(1, S):
        acc += P[s]  # FP32
    Y = torch.full((M + 1, N), 7.0, dtype=torch.float16, device="cuda")
    print("[case] second pass", S, flush=True)
    binding.reduce(torch.from_numpy(P).cuda(), out=Y[:M])
    assert np.array_equal(Y[:M].cpu().numpy().view(np.uint16), acc.astype(np.float16).view(np.uint16)) and bool((Y[M] == 7.0).all())
