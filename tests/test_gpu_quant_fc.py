"""The update that takes four subspaces per workgroup (pq_update_fc_kernel in
csrc/quantize.hip), at the edges of its chunks, sets and codes: sub-codewords
and counts equal the CPU oracle's bit for bit (each cluster is summed in
float64 in sub-vector order and rounded once), and those of weights that start
off a 16-byte boundary, which the general kernel updates.
"""
import numpy as np
import pytest
import torch

from paper_1512_06473_amd import api as api_mod
from paper_1512_06473_amd import workloads as wl

pytestmark = pytest.mark.gpu

# C_t, M, C's, K
CASES = [
    (1, 768, 4, 32),     # one row; the smallest M
    (511, 769, 4, 32),   # a chunk less a row; a set of one subspace, codes off dword bounds
    (512, 770, 4, 5),    # a whole chunk
    (513, 771, 4, 64),   # a row into the next; 6-bit codes
    (1100, 768, 4, 1),   # K = 1
    (255, 768, 8, 32),   # C's = 8: chunks of 256 rows
    (257, 771, 8, 17),
]


@pytest.mark.parametrize("skew", [False, True])
@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_update_fc(oracle, case, skew):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    Ct, M, Csp, K = case
    print("update fc", case, skew, flush=True)
    rng = np.random.Generator(np.random.PCG64(9300 + CASES.index(case)))
    W, D = wl.random_quant(rng, Ct, M * Csp, 1, Csp, K)
    codes = rng.integers(0, K, size=(Ct, 1, 1, M)).astype(np.uint8)
    if skew:  # most of a subspace in one sub-codeword, others unused
        codes[rng.random(codes.shape) < 0.9] = K // 2
        codes[codes == 0] = K // 2
    codes = codes.reshape(tuple(api_mod._codes_shape(torch.from_numpy(W), M)))
    Wd, cd = torch.from_numpy(W).to(dev), torch.from_numpy(codes).to(dev)
    Dn, cnt = api_mod.pq_update(Wd, cd, torch.from_numpy(D).to(dev))
    rD, rcnt = oracle.pq_update(W, codes, D)
    assert np.array_equal(cnt.cpu().numpy(), rcnt)
    assert np.array_equal(Dn.cpu().numpy().view(np.uint32), rD.view(np.uint32))
    off = torch.empty(W.size + 1, device=dev)[1:].view(Wd.shape)
    off.copy_(Wd)
    D2, cnt2 = api_mod.pq_update(off, cd, torch.from_numpy(D).to(dev))
    assert torch.equal(D2, Dn) and torch.equal(cnt2, cnt)
