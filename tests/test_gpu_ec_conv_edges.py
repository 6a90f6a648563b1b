"""The kernels of the conv error correction at the edges of their dispatch: the
matrix form of the Gram blocks (d_k^2 C's <= 64 in tiles of 16, maps up to 32
KB), the fused pass (<= 128, maps up to 48 KB for both sub-spaces) and the
kernels behind them, channel blocks of 64, more images than Gram chunks, and
the solve's sizes in K.  Against the float64 oracle with the bounds of
test_gpu_ec_conv.py (both sides are float64; codes must be equal).
"""
import numpy as np
import pytest
import torch

from paper_1512_06473_amd import api as api_mod
from test_gpu_ec_conv import problem, run_gpu

pytestmark = pytest.mark.gpu

# N, C_s, H, W, C_t, d_k, stride, pad, C's, K
CASES = [
    (1, 2, 3, 3, 5, 1, 1, 0, 1, 2),       # one (p, j)
    (2, 16, 5, 6, 65, 1, 1, 0, 8, 7),     # a channel past a block of 64
    (9, 4, 5, 5, 17, 3, 1, 1, 2, 64),     # 2 tiles; more images than chunks; K a whole wave
    (3, 8, 7, 5, 33, 4, 2, 1, 4, 65),     # 64: the Gram tiles' limit; K one past a wave
    (2, 16, 6, 6, 40, 3, 1, 1, 8, 128),   # 72: past it, fused pass of 5 tiles
    (2, 8, 8, 8, 64, 5, 1, 2, 4, 130),    # 100: 7 tiles
    (2, 16, 6, 7, 24, 4, 1, 1, 8, 50),    # 128: the pass's limit
    (2, 10, 6, 7, 24, 5, 1, 2, 5, 200),   # 125, ragged; K = 200
    (2, 12, 7, 7, 24, 5, 1, 2, 6, 40),    # 150: past it
    (1, 8, 36, 36, 20, 3, 1, 1, 4, 32),   # map of 23 KB: fused
    (1, 8, 40, 40, 20, 3, 1, 1, 4, 32),   # 28 KB: past the pass's
    (1, 8, 48, 44, 20, 3, 1, 1, 4, 32),   # 37 KB: past the Gram's as well
    (1, 6, 24, 24, 30, 7, 2, 2, 3, 20),   # 49 positions: four groups of counts
    (7001, 4, 3, 3, 5, 3, 1, 0, 4, 8),    # one output an image: two images per workgroup, the last alone
    (1240, 2, 4, 3, 70, 3, 1, 0, 2, 6),   # the same with five channel blocks
    (2, 8, 4, 4, 1050, 3, 1, 0, 8, 256),  # 9450 pairs at the largest K and C's
]


# The codes at the start: drawn, all the same, or one half the same.
@pytest.mark.parametrize("start", ["drawn", "one", "half"])
@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_ec_conv_edges(case, start):
    if start != "drawn" and case[9] > 130:
        pytest.skip("long in the oracle")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import ec_conv
    N, Cs, H, W, Ct, dk, st, pd, Csp, K = case
    print("ec_conv edge", case, flush=True)
    rng = np.random.Generator(np.random.PCG64(9400 + CASES.index(case)))
    S, T, D0, c0 = problem(rng, N, Cs, H, W, Ct, dk, st, pd, Csp, K)
    if start == "one":
        c0[...] = K - 1
    elif start == "half":  # rows made from the list and from counts in one layer
        c0[: Ct // 2] = 1 % K
    D, c, obj = run_gpu(api_mod, torch.device("cuda:0"), S, T, D0, c0, st, pd, 1, 1)
    Dr, cr, hr = ec_conv.ec_conv(S, T, D0, c0, st, pd, 1, 1)
    assert np.array_equal(c, cr), int((c != cr).sum())
    assert np.allclose(D, Dr, rtol=1e-6, atol=1e-7 * float(np.abs(Dr).max())), float(np.abs(D - Dr).max())
    assert np.allclose(obj, hr, rtol=1e-9, atol=1e-9 * hr[0])


@pytest.mark.parametrize("case", [(1, 16, 5, 5, 655, 5, 1, 2, 8, 193), (2, 16, 4, 4, 1820, 3, 1, 1, 8, 256),
                                  (1, 7, 4, 4, 16384, 1, 1, 0, 7, 256),
                                  (1536, 1, 78, 78, 1, 1, 1, 0, 1, 2),  # 73 KB of LDS in the pass
                                  (2, 1, 90, 90, 4, 7, 1, 0, 1, 5)], ids=str)  # 93 KB for the Gram blocks
def test_ec_conv_largest(case):
    """The largest pair counts (C_t d_k^2 up to 16384) with K and C's at their
    largest, and the largest LDS of the pass and of the Gram kernel: the objective falls step by step and ends at the error of the
    sub-codebooks and codes that were returned (float64, on sub-codebooks
    rounded to fp32)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle
    N, Cs, H, W, Ct, dk, st, pd, Csp, K = case
    print("ec_conv largest", case, flush=True)
    rng = np.random.Generator(np.random.PCG64(9500 + Ct))
    S, T, D0, c0 = problem(rng, N, Cs, H, W, Ct, dk, st, pd, Csp, K)
    D, c, obj = run_gpu(api_mod, torch.device("cuda:0"), S, T, D0, c0, st, pd, 1, 1)
    assert np.all(np.diff(obj) <= 1e-9 * obj[0])
    for Dx, cx, want in ((D0, c0, obj[0]), (D, c, obj[-1])):
        err = ((T - oracle.conv_direct(S, Dx, cx, st, pd)) ** 2).sum()
        assert abs(err - want) <= 1e-5 * obj[0], (err, want)


def test_ec_conv_scratch_of_many_images():
    """The partial correlations do not grow with the images: 20000 of one output
    each, 64 channels, C's = 8 (one set per image would be 737 MB)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    N, Ct = 20000, 64
    g = torch.Generator(device=dev).manual_seed(9600)
    S = torch.randn((N, 8, 3, 3), generator=g, device=dev)
    T = torch.randn((N, Ct, 1, 1), generator=g, device=dev)
    D = torch.randn((1, 4, 8), generator=g, device=dev)
    c = torch.randint(0, 4, (Ct, 3, 3, 1), generator=g, device=dev, dtype=torch.uint8)
    s = torch.cuda.Stream(dev)  # a scratch buffer of its own
    s.wait_stream(torch.cuda.current_stream(dev))
    with torch.cuda.stream(s):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info(dev)[0]
        obj = api_mod.ec_conv(S, T, D, c, 1, 0, 1, 1)
        torch.cuda.synchronize()
        used = before - torch.cuda.mem_get_info(dev)[0]
    assert bool(torch.isfinite(obj).all())
    assert used <= 200 << 20, used
