"""GPU parity of the dense conv kernel (weights rebuilt from the codebooks,
split-fp16 matrix products) at the edges of its tiles and of its number range.

Held to the fp32 bound abs(gpu - oracle) <= 1e-5 A + 1e-6 (A: sum of the
magnitudes of an output's products) on float data; equal bit for bit on small
integers, which the split represents and sums exactly.  The tile is 96 output
positions x 64 or 128 channels, a chunk 16 channels per kernel tap, and the
tiles' units are cut into runs at any unit.
"""
import numpy as np
import pytest
import torch

from paper_1512_06473_amd import workloads as wl

pytestmark = pytest.mark.gpu

RTOL, ATOL = 1e-5, 1e-6

SHAPES = [
    # N, Cs, H, W, Ct, dk, stride, pad, Csp, K
    (1, 16, 14, 14, 32, 3, 1, 1, 4, 16),      # one chunk, fewer runs than CUs
    (1, 16, 1, 96, 65, 1, 1, 0, 4, 32),       # exactly one tile of positions, 65 channels
    (1, 20, 1, 97, 64, 1, 1, 0, 5, 32),       # one position more; a chunk of 4 channels only
    (2, 17, 9, 11, 129, 3, 1, 1, 1, 7),       # channels past a group of 8, C's = 1
    (3, 36, 9, 11, 40, 3, 2, 1, 4, 64),       # stride 2
    (2, 24, 13, 12, 33, 1, 2, 0, 4, 64),      # strided 1x1: only read positions are staged
    (2, 24, 13, 12, 33, 1, 3, 0, 8, 256),
    (1, 40, 7, 90, 48, 3, 1, 1, 8, 128),      # column strips
    (1, 32, 5, 130, 20, 5, 1, 2, 16, 200),    # strips, C's = 16, K > 128
    (2, 96, 15, 14, 96, 5, 1, 2, 4, 128),
    (4, 64, 8, 8, 130, 2, 1, 1, 4, 128),      # even kernel
    (1, 48, 12, 12, 24, 3, 1, 2, 6, 100),     # pad 2
    (5, 128, 7, 7, 256, 3, 1, 1, 4, 128),     # tiles across images
    (40, 48, 13, 13, 200, 3, 1, 1, 4, 64),    # whole tiles and shared ones
    (2, 3, 45, 47, 97, 11, 4, 2, 3, 64),      # few input channels: kernel rows packed into positions
    (3, 4, 20, 23, 40, 5, 1, 2, 4, 32),
    (1, 6, 17, 19, 33, 3, 2, 1, 2, 50),
    (1, 1, 9, 120, 5, 3, 1, 1, 1, 9),
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(autouse=True)
def dense(monkeypatch):
    monkeypatch.setenv("QCNN_CONV_KERNEL", "dense")


def T(a, dev):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def conv(dev, x, D, codes, s, p, bias=None, relu=False):
    from paper_1512_06473_amd import api
    return api.conv_forward(T(x, dev), T(D, dev), T(codes, dev), s, p, T(bias, dev), relu).cpu().numpy()


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_dense_edges(dev, oracle, shape, integer):
    N, Cs, H, W, Ct, dk, s, p, Csp, K = shape
    rng = np.random.Generator(np.random.PCG64(11))
    x, D, codes = wl.random_conv(rng, N, Cs, H, W, Ct, dk, s, p, Csp, K, integer=integer)
    bias = (rng.integers(-3, 4, Ct) if integer else rng.standard_normal(Ct)).astype(np.float32)
    y = conv(dev, x, D, codes, s, p, bias, True)
    ref, A = oracle.conv_lut(x, D, codes, s, p, with_bound=True)
    ref = np.maximum(ref + bias[None, :, None, None].astype(np.float64), 0.0)
    if integer:
        assert np.array_equal(y.astype(np.float64), ref)
    else:
        A = A + np.abs(bias)[None, :, None, None]
        assert np.all(np.abs(y - ref) <= RTOL * A + ATOL)


def _layer(seed=5, N=2, Cs=64, H=13, Ct=96):
    rng = np.random.Generator(np.random.PCG64(seed))
    return rng, *wl.random_conv(rng, N, Cs, H, H, Ct, 3, 1, 1, 4, 128)


@pytest.mark.parametrize("scale", [2.0 ** -118, 1e-30, 1e-12, 1e12, 1e30])
def test_dense_scale(dev, oracle, scale):
    """Results do not depend on the inputs' magnitude: each is as close as at
    magnitude one (the bound scaled with it, no absolute part but fp32's
    smallest normal number)."""
    _, x, D, codes = _layer()
    x = (x * np.float32(scale)).astype(np.float32)
    y = conv(dev, x, D, codes, 1, 1)
    ref, A = oracle.conv_lut(x, D, codes, 1, 1, with_bound=True)
    assert np.all(np.abs(y.astype(np.float64) - ref) <= RTOL * A + 1.2e-38)


@pytest.mark.parametrize("kind", ["channels", "images", "positions", "codewords", "tiny"])
def test_dense_wide_range(dev, oracle, kind):
    """Inputs or codewords over many orders of magnitude, each output held to
    the bound of its own products: growing channel by channel (the scale is
    changed between chunks), image by image, position by position (some span
    more than the split holds: those tiles run in fp32), codeword by codeword,
    and next to single values of 1e-25."""
    rng, x, D, codes = _layer()
    N, Cs, H, W = x.shape
    if kind == "channels":
        x *= np.float32(2.0) ** (np.arange(Cs) // 2 - 16)[None, :, None, None].astype(np.float32)
    elif kind == "images":
        x *= np.float32(10.0) ** (-12 * np.arange(N))[:, None, None, None].astype(np.float32)
    elif kind == "positions":
        x *= (np.float32(10.0) ** rng.integers(-15, 16, (H, W)).astype(np.float32))[None, None]
    elif kind == "codewords":
        D *= (np.float32(10.0) ** rng.integers(-15, 1, D.shape[:2]).astype(np.float32))[:, :, None]
    else:
        x[rng.random(x.shape) < 0.01] = 1e-25
    y = conv(dev, x, D, codes, 1, 1)
    ref, A = oracle.conv_lut(x, D, codes, 1, 1, with_bound=True)
    assert np.all(np.abs(y.astype(np.float64) - ref) <= RTOL * A + 1e-30)


@pytest.mark.parametrize("ratio", [1e6, 1e8, 1e10, 1e12, 1e15, 1e20])
@pytest.mark.parametrize("where", ["x", "D", "packed rows"])
def test_dense_small_beside_large(dev, oracle, where, ratio):
    """A small value beside a large one, of which the result is made alone
    because the other factor is zero on the large one: channel by channel,
    within a codeword, and column by column where kernel rows are packed (the 8
    values of a staged group are neighbouring channels, or columns)."""
    rng, x, D, codes = _layer(21)
    if where == "packed rows":
        x, D, codes = wl.random_conv(rng, 2, 4, 21, 22, 70, 3, 1, 1, 4, 128)
        x[:, :, ::3, ::4] *= np.float32(ratio)
        D[:, :, :2] = 0.0
        x[:, 2:] /= np.float32(ratio)
    elif where == "x":
        x[:, np.arange(64) % 8 < 4] *= np.float32(ratio)
        D[::2] = 0.0            # the subspaces on the large channels
    else:
        D[:, :, :2] *= np.float32(ratio)
        x[:, np.arange(64) % 4 < 2] = 0.0
    y = conv(dev, x, D, codes, 1, 1)
    ref, A = oracle.conv_lut(x, D, codes, 1, 1, with_bound=True)
    assert np.all(np.abs(y.astype(np.float64) - ref) <= RTOL * A + 1e-30)


@pytest.mark.parametrize("what", ["all chunks", "last subspace", "codewords"])
@pytest.mark.parametrize("power", [-20, -40, -70, -100])
@pytest.mark.parametrize("shape", [SHAPES[i] for i in (0, 2, 3, 4, 6, 8, 10, 13, 14, 15, 17)], ids=str)
def test_dense_range_bands(dev, oracle, shape, power, what):
    """Results made only of inputs far below the largest, small integers times
    2^power, equal bit for bit, bias and ReLU included: the first pass alone, in
    a second and a third pass over all chunks or over the last one, and past
    those, or with codewords of that range, the fp32 form; per call and through
    a plan, with tiles of one run and of several."""
    from paper_1512_06473_amd import api
    N, Cs, H, W, Ct, dk, s, p, Csp, K = shape
    rng = np.random.Generator(np.random.PCG64(31))
    x, D, codes = wl.random_conv(rng, N, Cs, H, W, Ct, dk, s, p, Csp, K, integer=True)
    M, f = Cs // Csp, np.float32(2.0 ** power)
    bias = rng.integers(-3, 4, Ct).astype(np.float32) * f
    if what == "codewords":
        if M == 1:
            pytest.skip("one subspace")
        D[M - 1] *= f
        x[:, :(M - 1) * Csp] = 0.0
    else:
        # the small channels: within each subspace, so that both lie side by side, or the last one's
        small = np.arange(Cs) % 2 == 1 if what == "all chunks" else np.arange(Cs) >= Cs - Csp
        if small.all() or not small.any():
            pytest.skip("no channels of both kinds")
        x[:, small] *= f
        for m in range(M):
            D[m][:, ~small[m * Csp:(m + 1) * Csp]] = 0.0
    y = conv(dev, x, D, codes, s, p, bias, True)
    ref = np.maximum(oracle.conv_lut(x, D, codes, s, p) + bias[None, :, None, None].astype(np.float64), 0.0)
    assert ref.any()
    assert np.array_equal(y.astype(np.float64), ref), float(np.abs(y - ref).max() / float(f))
    plan = api.ConvPlan(x.shape, T(D, dev), T(codes, dev), s, p, T(bias, dev), True)
    assert np.array_equal(plan(T(x, dev)).cpu().numpy(), y)


def _exact(x, D, codes, s, p):
    """The dense correlation with the rebuilt weights, float64 on the GPU."""
    W = torch.stack([D[m][codes[..., m].long()] for m in range(D.shape[0])], -2).flatten(-2).permute(0, 3, 1, 2)
    dk = codes.shape[1]
    out = [(n - dk + 2 * p) // s + 1 for n in x.shape[2:]]
    cols = torch.nn.functional.unfold(x.double(), dk, padding=p, stride=s)
    Wm = W.reshape(W.shape[0], -1).double().contiguous()
    return torch.stack([Wm @ c for c in cols]).reshape(x.shape[0], -1, *out)


@pytest.mark.parametrize("shape", [
    # N, Cs, H, W, Ct, dk, stride, pad, Csp, K: chains of 48 to 64 table entries
    (47, 40, 20, 20, 324, 5, 1, 2, 8, 128),   # 25 steps a chunk, whole tiles and pieces
    (9, 232, 8, 8, 131, 5, 1, 2, 8, 128),     # tiles of many pieces
    (22, 160, 12, 12, 56, 5, 1, 2, 8, 128),   # two reduction groups
    (28, 140, 14, 12, 356, 3, 2, 1, 4, 64),   # stride 2
    (41, 396, 49, 48, 156, 1, 1, 0, 4, 16),   # 1x1
], ids=str)
def test_dense_error_not_above_the_tables(dev, shape, monkeypatch):
    """Layers with the shortest chains of table entries that still go to this
    kernel: its relative error (2-norm, against float64, mean of three inputs) is
    not larger than the table kernel's."""
    from paper_1512_06473_amd import api
    N, Cs, H, W, Ct, dk, s, p, Csp, K = shape
    err = {}
    for seed in range(3):
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        x = torch.randn((N, Cs, H, W), generator=g, device=dev).clamp_min_(0.0)
        D = 0.05 * torch.randn((Cs // Csp, K, Csp), generator=g, device=dev)
        codes = torch.randint(0, K, (Ct, dk, dk, Cs // Csp), generator=g, device=dev, dtype=torch.uint8)
        ref = _exact(x, D, codes, s, p)
        for kernel in ("dense", "flat"):
            monkeypatch.setenv("QCNN_CONV_KERNEL", kernel)
            y = api.conv_forward(x, D, codes, s, p).double()
            err[kernel] = err.get(kernel, 0.0) + float((y - ref).norm() / ref.norm()) / 3.0
    assert err["dense"] <= err["flat"], err


@pytest.mark.parametrize("Cs", [16, 64])
@pytest.mark.parametrize("tail", [4093, 4097, 4095, 2049, 1])
def test_dense_significands(dev, Cs, tail):
    """Factors that all lose the most in the split (every significand 1 + tail
    2^-23): a factor keeps 23 bits (2^-23 of it), and the product of the two low
    parts is left out (2^-22), 2^-21 of a product in all.  On top of that the sums
    of Cs products: two roundings a step of 16 channels, three folds and joins,
    the MFMA's own no finer than 2^-23 each."""
    rng = np.random.Generator(np.random.PCG64(tail))
    x, D, codes = wl.random_conv(rng, 2, Cs, 9, 11, 70, 1, 1, 0, 4, 32)
    v = np.float32(1.0 + tail * 2.0 ** -23)
    x = (v * np.float32(2.0) ** rng.integers(-3, 4, x.shape)).astype(np.float32)
    D = (v * np.float32(2.0) ** rng.integers(-3, 4, D.shape)).astype(np.float32)
    y = conv(dev, x, D, codes, 1, 0).astype(np.float64)
    W = np.concatenate([D[m][codes[:, 0, 0, m]] for m in range(Cs // 4)], 1).astype(np.float64)
    ref = np.einsum("tc,nchw->nthw", W, x.astype(np.float64))  # every product is positive: A = ref
    assert np.all(np.abs(y - ref) <= (2.0 ** -21 + (2 * Cs / 16 + 3) * 2.0 ** -23) * ref)


@pytest.mark.parametrize("where", ["x", "D", "packed rows"])
def test_dense_non_finite(dev, where, monkeypatch):
    """Infinities and NaN reach exactly the outputs they reach through the
    table kernel; the others stay within the bound of it."""
    rng, x, D, codes = _layer(7)
    if where == "packed rows":
        x, D, codes = wl.random_conv(rng, 2, 4, 21, 22, 70, 3, 1, 1, 4, 128)
        x[0, 1, 3, 4], x[0, 3, 20, 0], x[1, 2, 20, 21] = np.inf, -np.inf, np.nan
    elif where == "x":
        x[0, 5, 3, 4], x[0, 40, 12, 0], x[1, 63, 12, 12] = np.inf, -np.inf, np.nan
    else:
        D[3, 17, 1], D[9, 100, 0] = np.inf, np.nan
    y = conv(dev, x, D, codes, 1, 1)
    monkeypatch.setenv("QCNN_CONV_KERNEL", "flat")
    t = conv(dev, x, D, codes, 1, 1)
    assert np.array_equal(np.isnan(y), np.isnan(t)) and np.array_equal(np.isinf(y), np.isinf(t))
    fin = np.isfinite(t)
    assert fin.any() and not fin.all()
    assert np.array_equal(np.sign(y[np.isinf(t)]), np.sign(t[np.isinf(t)]))
    assert np.all(np.abs(y[fin] - t[fin]) <= 2e-5 * np.abs(t[fin]) + 2e-4)


def test_dense_zero_input(dev):
    _, x, D, codes = _layer()
    assert not conv(dev, np.zeros_like(x), D, codes, 1, 1).any()
    x[:, :32] = 0.0  # the first chunks hold nothing to scale by
    y = conv(dev, x, D, codes, 1, 1)
    assert np.isfinite(y).all() and y.any()


@pytest.mark.parametrize("seed", range(12))
def test_dense_random_against_generic(dev, seed, monkeypatch):
    """Random layers of every form the dense kernel takes against the generic
    table kernel: per call, packed, through a plan and pooled."""
    from paper_1512_06473_amd import api
    rng = np.random.Generator(np.random.PCG64(100 + seed))
    dk, Csp = int(rng.choice([1, 2, 3, 5, 7])), int(rng.choice([1, 2, 3, 4, 8, 12, 16]))
    M, K, stride = int(rng.integers(1, 12)), int(rng.integers(1, 257)), int(rng.choice([1, 1, 2, 3]))
    pad, N, Ct = int(rng.integers(0, dk)), int(rng.integers(1, 5)), int(rng.integers(1, 180))
    H, W = int(rng.integers(dk, 30)), int(rng.integers(dk, 40))
    x, D, codes = wl.random_conv(rng, N, M * Csp, H, W, Ct, dk, stride, pad, Csp, K)
    xd, Dd, cd = T(x, dev), T(D, dev), T(codes, dev)
    y = api.conv_forward(xd, Dd, cd, stride, pad)
    assert torch.equal(y, api.conv_forward_packed(xd, Dd, api.pack_codes(cd, K), Ct, dk, stride, pad))
    assert torch.equal(y, api.ConvPlan(xd.shape, Dd, cd, stride, pad)(xd))
    if min(y.shape[2:]) >= 2:
        assert torch.equal(api.maxpool2d(y, 2, 1), api.conv_pool_forward(xd, Dd, cd, stride, pad, 2, 1))
    A = api.conv_forward(xd.abs(), Dd.abs(), cd, stride, pad)
    monkeypatch.setenv("QCNN_CONV_KERNEL", "generic")
    t = api.conv_forward(xd, Dd, cd, stride, pad)
    assert bool(((y - t).abs() <= 2 * RTOL * A + 2 * ATOL).all())
