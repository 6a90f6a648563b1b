"""The FC kernels that read the code stream itself (csrc/fc_few.hip, and
csrc/fc_gather.hip for few subspaces and many images), at the sizes where they
can go wrong, against the CPU oracle (Eq. (5)).

Byte codes, packed codes and a plan of either must agree bit for bit; against
the oracle, integer data is exact and float data is within the bound of a sum
of M products of C's terms in fp32 taken relative to the sum of magnitudes A:
a table entry is C's fused steps, and the longest chain of lookups is M / 4 + 2
plus one step per split (at most 256 of at most 32 groups each, never more
than M / 32) and the bias, so (C's + M / 4 + M / 32 + 4) 2^-24 A bounds it.  The
other kernel adds its M lookups in one chain: (C's + M + 4) 2^-24 A.
"""
import numpy as np
import pytest
import torch

from paper_1512_06473_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, M, C's, K, C_t
CASES = [
    (1, 1, 4, 1, 1),         # K = 1: no stream to read in packed form
    (1, 31, 4, 2, 255),      # one channel block less one; a short group of 1-bit codes
    (1, 32, 4, 3, 256),      # exactly a group, a block; entries past K
    (2, 33, 4, 8, 257),      # a subspace into the next group; a channel into the next block
    (2, 65, 3, 16, 300),     # single loads (C's = 3)
    (3, 97, 4, 31, 511),     # an image past the last of four
    (4, 200, 8, 64, 64),
    (5, 1153, 4, 32, 700),   # several groups per workgroup, a ragged last split
    (8, 130, 2, 100, 40),    # K > 64: 7-bit codes
    (9, 64, 12, 128, 129),
    (70, 77, 4, 256, 300),   # byte codes; a table of one group
    (300, 70, 16, 32, 1030), # more blocks than CUs: no split
    (1, 2304, 4, 32, 4096),  # fc6 of AlexNet
]
# few subspaces, images for 128, 256 or 512 workgroups: the two sides of each line
GATHER = [
    (8193, 3, 9, 32, 3),     # 129 workgroups
    (8200, 4, 9, 32, 3),     # 129 workgroups, past 3 subspaces: fc_few
    (16383, 32, 16, 16, 7),  # 256 workgroups, the last image missing
    (16383, 33, 16, 16, 7),
    (8131, 16, 16, 16, 257), # two channel blocks, 256 workgroups
    (16321, 17, 16, 16, 257),
    (16321, 8, 4, 200, 300),
    (32769, 2, 16, 256, 65), # 513 workgroups, byte codes
    (65535, 30, 9, 33, 2),   # 1024 workgroups, 64 channels or fewer
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def api():
    from paper_1512_06473_amd import api as a
    return a


def T(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def bits(t):
    return t.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("case", CASES + GATHER, ids=str)
def test_fc_few(api, dev, oracle, case, integer):
    N, M, Csp, K, Ct = case
    print("fc few", case, integer, flush=True)
    rng = np.random.Generator(np.random.PCG64(9100 + (CASES + GATHER).index(case)))
    x, D, codes = wl.random_fc(rng, N, M * Csp, Ct, Csp, K, integer=integer)
    bias = rng.integers(-3, 4, size=Ct).astype(np.float32)
    relu = N % 2 == 0
    xd, Dd, cd, bd = T(x, dev), T(D, dev), T(codes, dev), T(bias, dev)
    y = api.fc_forward(xd, Dd, cd, bd, relu)
    plan = api.FcPlan(N, Dd, cd, bd, relu)
    packed = api.pack_codes(cd, K)
    yq = api.fc_forward_packed(xd, Dd, packed, Ct, bd, relu)
    for other in (plan(xd), yq):
        assert np.array_equal(bits(y), bits(other))
    # inputs that start off a 16-byte boundary: the same values by single loads
    off = torch.empty(x.size + 1, device=dev)[1:].view(x.shape)
    off.copy_(xd)
    assert np.array_equal(bits(y), bits(api.fc_forward(off, Dd, cd, bd, relu)))
    ref, A = oracle.fc_lut(x, D, codes, bias=bias, relu=relu, with_bound=True)
    err = np.abs(y.cpu().numpy().astype(np.float64) - ref)
    tol = 0 if integer else (Csp + (M if case in GATHER else M / 4 + M / 32) + 4) * 2.0 ** -24
    assert np.all(err <= tol * A), float(err.max())
    plan.close()


def test_fc_few_non_finite(api, dev):
    """An infinite or NaN input reaches every channel whose codeword meets it
    and no other image."""
    rng = np.random.Generator(np.random.PCG64(9200))
    x, D, codes = wl.random_fc(rng, 4, 40 * 4, 70, 4, 32)
    y0 = api.fc_forward(T(x, dev), T(D, dev), T(codes, dev)).cpu().numpy()
    x[1, 5], x[2, 159] = np.inf, np.nan
    y = api.fc_forward(T(x, dev), T(D, dev), T(codes, dev)).cpu().numpy()
    assert np.array_equal(y[[0, 3]], y0[[0, 3]])
    assert not np.isfinite(y[1:3]).any()
