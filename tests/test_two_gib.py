"""Weights of close to 2 GiB: offsets run on past the end of a slice, and those of columns past N may come back into the matrix."""
import numpy as np
import pytest


def test_the_largest_weights_keep_their_form():
    """128 x 256 tiles are for all weights below 2 GiB, whatever is asked for ahead of the last stage."""
    from paper_2601_16536_amd import binding
    for M, K, N in ((128, 512, 1 << 22), (128, 512, (1 << 22) - 8), (300, 3968, 1 << 20), (2048, 122880, 34600)):
        assert K // 8 * N * 4 < 0x7F000000 <= (K // 8 + 64) * N * 4
        p = binding.query_plan(M, N, K, 128)
        assert (p["kernel"], p["tile_n"]) == (binding.KERNEL_TILE, 256), (M, K, N, p)


@pytest.mark.gpu
@pytest.mark.parametrize("form,K,group", [("panel", 992, 32), ("panel", 896, 896), ("tall", 896, 896), ("tall", 992, 32), ("pair", 896, 128)])
def test_columns_past_n_of_the_largest_weights(form, K, group):
    """N = 2^22 - 8, so that the last tile has columns past N.  Columns at the edges, where a wrapped offset could show, against 64-bit
    sums; every output is written and the row beyond is not."""
    import torch
    from paper_2601_16536_amd import binding
    M, N = 40, (1 << 22) - 8
    gen = torch.Generator(device="cuda").manual_seed(5)
    words = lambda *shape: torch.randint(-(1 << 31), 1 << 31, shape, dtype=torch.int32, device="cuda", generator=gen)
    X = torch.randn((M, K), device="cuda", generator=gen).to(torch.float16)
    Wp, Zp = words(K // 8, N), words(K // group, N // 8)
    s = torch.rand((K // group, N), device="cuda", generator=gen, dtype=torch.float16) * 0.019 + 0.001
    knobs = {"panel": {"panel": 1, "pair": 2}, "tall": {"panel": 2, "pair": 2, "tile_rows": 64}, "pair": {"pair": 1, "pair_split": 1}}[form]
    Y = torch.full((M + 1, N), float("nan"), dtype=torch.float16, device="cuda")
    try:
        for knob, value in knobs.items():
            binding.tune(knob, value)
        plan = binding.query_plan(M, N, K, group)
        assert (plan["tile_n"], plan["split"]) == ({"panel": 256, "tall": 64, "pair": 128}[form], 1) and (form != "tall" or plan["waves_k"] == 4)
        print("[case] 2 GiB", form, K, group, flush=True)
        binding.gemm(X, Wp, s, Zp, group, out=Y[:M])
        torch.cuda.synchronize()
    finally:
        for knob in knobs:
            binding.tune(knob, 0)
    assert bool(torch.isfinite(Y[:M]).all()) and bool(torch.isnan(Y[M]).all())
    cols = torch.cat([torch.arange(0, 264), torch.arange(N // 2, N // 2 + 64), torch.arange(N - 320, N)]).cuda()
    shift = torch.arange(0, 32, 4, device="cuda", dtype=torch.int32)
    q = ((Wp[:, cols].unsqueeze(1) >> shift.view(1, 8, 1)) & 15).reshape(K, -1).double()
    z = ((Zp[:, cols // 8] >> (cols % 8 * 4).to(torch.int32)) & 15).double().repeat_interleave(group, 0)
    ref = X.double() @ ((q - z) * s[:, cols].double().repeat_interleave(group, 0))
    err = (Y[:M][:, cols].double() - ref).abs() / (1e-2 * (1.0 + ref.abs()))
    assert float(err.max()) <= 1.0
