"""Few-row distance tiles, the selection's first bound, the re-rank's single sort and left-out rows, at the edges of their
tiles, steps and slots.  Distances against the CPU oracle (the tolerances of parity_util); the two exact routes against
each other bit for bit."""
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


def bits(t):
    return t.view(torch.int32) if t.is_floating_point() else t


def both_routes(vs, x, q, k, metric):
    out = []
    for path in (1, 2):
        vs.vs_set_option("knn_path", path)
        try:
            out.append([t.clone() for t in vs.vs_flat_search(x, q, k, metric)])
        finally:
            vs.vs_set_option("knn_path", 0)
    (D, I), (D2, I2) = out
    assert torch.equal(I, I2) and torch.equal(bits(D), bits(D2))
    return D, I


# rows, columns, d, k: rows at the tiles of 4, 16 and 64; columns at a tile of 64, a step of 2048 values (512 per
# wavefront) and the one after it; k at the sorts' widths
@pytest.mark.parametrize("metric", [L2, IP])
@pytest.mark.parametrize("nq,nb,d,k", [
    (1, 63, 33, 1), (1, 4096, 128, 16), (4, 65, 32, 64), (5, 2047, 100, 48), (3, 2049, 31, 49), (16, 8193, 128, 128),
    (17, 4159, 99, 127), (64, 6145, 36, 129), (65, 1025, 96, 10), (333, 2000, 96, 24), (1, 20000, 40, 150)])
def test_few_rows(vs, metric, nq, nb, d, k):
    rng = np.random.default_rng(nq * 10007 + nb)
    for kind in ("float", "integer", "equal"):
        x = rng.standard_normal((nb, d)).astype(np.float32)
        q = rng.standard_normal((nq, d)).astype(np.float32)
        if kind == "integer":        # exact in bf16: approximate values are the canon values, many of them equal
            x, q = np.round(3 * x), np.round(3 * q)
        elif kind == "equal":        # nothing tells the columns apart: the smallest numbers win
            x[:] = x[0]
        xt, qt = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
        D, I = both_routes(vs, xt, qt, k, metric)
        Do, Io = oracle.flat_search(x, q, k + EXTRA, metric)
        if kind == "equal":
            assert (I.cpu().numpy() == Io[:, :k]).all()
        else:
            check_search(D.cpu().numpy(), I.cpu().numpy(), Do, Io, metric, q, np.sqrt((x ** 2).sum(1).max()))


@pytest.mark.parametrize("metric", [L2, IP])
def test_few_rows_infinities_and_nan(vs, metric):
    """Rows with NaN or infinite components, and fewer finite ones than k: both routes agree bit for bit."""
    rng = np.random.default_rng(7)
    x = rng.standard_normal((4200, 64)).astype(np.float32)
    x[::3, 5] = np.nan
    x[1::3, 6] = np.inf
    x[40:4190, 7] = 3e38
    q = rng.standard_normal((5, 64)).astype(np.float32)
    q[1] = 0
    q[2, 3] = np.inf
    both_routes(vs, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), 32, metric)


@pytest.mark.parametrize("nq,nb,d,k", [(300, 16384, 160, 32), (2000, 4096, 128, 16), (300, 40000, 64, 100), (257, 16390, 96, 48)])
@pytest.mark.parametrize("data", ["near", "integer", "gauss"])
def test_rerank(vs, nq, nb, d, k, data):
    """near: columns in tight bunches, so that many lie within the error of the k-th best."""
    rng = np.random.default_rng(nb + k)
    x = rng.standard_normal((nb, d)).astype(np.float32)
    if data == "near":
        x = x[rng.integers(0, nb // 200, nb)] + 1e-3 * x
    elif data == "integer":
        x = np.round(2 * x)
    q = x[rng.integers(0, nb, nq)] + (0 if data == "integer" else 0.1) * rng.standard_normal((nq, d)).astype(np.float32)
    xt, qt = torch.from_numpy(x.astype(np.float32)).cuda(), torch.from_numpy(q.astype(np.float32)).cuda()
    for metric in (L2, IP):
        D, I = both_routes(vs, xt, qt, k, metric)
        fx = vs.Flat(d, metric)      # a kept operand: one product on the fp16 heads
        fx.add(xt)
        vs.vs_set_option("knn_path", 2)
        try:
            Df, If = fx.search(qt, k)
        finally:
            vs.vs_set_option("knn_path", 0)
        assert torch.equal(I, If) and torch.equal(bits(D), bits(Df))
