"""Look-ups over short and empty lists in shapes without a kernel of their own (d / M = 2; 4-bit codes, 48 sub-quantizers),
against the CPU oracle."""
import numpy as np
import pytest

import oracle
from parity_util import EXTRA, check_search

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

L2, IP = 0, 1


@pytest.fixture(scope="module")
def vs():
    import paper_2401_08281_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return m


@pytest.mark.parametrize("matrix", [-1, 1])
@pytest.mark.parametrize("M,nbits,metric,form", [(64, 4, IP, 0), (64, 4, L2, 1), (64, 4, L2, 0), (32, 4, IP, 0),
                                                 (16, 8, IP, 0), (48, 8, L2, 1), (32, 8, IP, 0)])
def test_short_lists(vs, M, nbits, metric, form, matrix):
    """Lists of no, one and up to several hundred codes next to each other, query by query and, where there is a kernel
    for it, on the matrix cores."""
    rng = np.random.default_rng(M + nbits)
    d = 2 * M
    sizes = [0, 1, 255, 0, 0, 256, 257, 63, 64, 65, 511, 513, 2, 0, 31, 700] * 2
    cent = (30 * rng.standard_normal((len(sizes), d))).astype(np.float32)
    x = np.concatenate([cent[l] + rng.standard_normal((n, d)).astype(np.float32) for l, n in enumerate(sizes)])
    cb = rng.standard_normal((M, 1 << nbits, 2)).astype(np.float32)
    q = (cent[rng.integers(0, len(sizes), 9)] + rng.standard_normal((9, d))).astype(np.float32)
    ix = vs.IVFPQ(d, metric, torch.from_numpy(cent).cuda(), torch.from_numpy(cb).cuda(), nbits)
    if form:
        ix.set_search_type(form)
    ix.add(torch.from_numpy(x).cuda())
    orc = oracle.OracleIVFPQ(d, metric, cent, cb, nbits)
    orc.add(x)
    vs.vs_set_option("matrix_scan", matrix)
    try:
        for k, nprobe in ((1, 1), (10, 7), (100, 32), (200, 32)):
            D, I = ix.search(torch.from_numpy(q).cuda(), k, nprobe)
            Do, Io = orc.search(q, k + EXTRA, nprobe)
            big = np.sqrt((x ** 2).sum(1).max())
            # (stored norms: |q|^2 + |x'|^2 cancel)
            cancel = (q.astype(np.float64) ** 2).sum(1) + 4 * float(big) ** 2 if form else None
            check_search(D.cpu().numpy(), I.cpu().numpy(), Do, Io, metric, q, big, cancel)
    finally:
        vs.vs_set_option("matrix_scan", 0)
        ix.close()
