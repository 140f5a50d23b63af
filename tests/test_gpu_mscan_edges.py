"""Where the matrix-core scan of inverted lists can go wrong beyond the sizes of its tiles: every distance and id bit for
bit that of the query-major scan."""
import numpy as np
import pytest

from test_gpu_mscan import IP, L2, lists_of, make, same

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def vs():
    import paper_2401_08281_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return m


@pytest.fixture(autouse=True)
def options(vs):
    yield
    for name, value in (("matrix_scan", 0), ("list_major_candidates", 1024), ("knn_eps_scale", 1.0)):
        vs.vs_set_option(name, value)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def both_scans(vs, ix, q, k, nprobe, tell=""):
    """Results of the matrix-core scan, which are those of the query-major scan."""
    vs.vs_set_option("matrix_scan", -1)
    D0, I0 = [t.clone() for t in ix.search(q, k, nprobe)]
    vs.vs_set_option("matrix_scan", 1)
    D1, I1 = ix.search(q, k, nprobe)
    torch.cuda.synchronize()
    assert same(D0, D1) and same(I0, I1), tell
    return D1, I1


# (d, M, bits): a shape with a kernel of its own, one without, 4-bit codes
@pytest.mark.parametrize("d,M,nbits", [(128, 16, 8), (100, 20, 8), (64, 32, 4)])
@pytest.mark.parametrize("what", ["equal vectors", "queries that are not finite"])
def test_survivors_beyond_their_list(vs, d, M, nbits, what):
    """More survivors per query than their common list has room for on average, 4 k + 128, and fewer than a query's own
    buffer holds; behind a larger search, whose values lie where the list is."""
    rng = np.random.default_rng(d)
    k, nprobe, nq = 10, 8, 200
    cent, x = lists_of(rng, d, [60] * 24)
    if what == "equal vectors":
        x = np.repeat(x[rng.permutation(len(x))[:24]], 300, axis=0)       # every vector 300 times
    ix = make(vs, "pq", d, M, nbits, L2, cent, x, rng)
    try:
        ix.add(dev(x))
        other = (x[rng.integers(0, len(x), 777)] + 20 * rng.standard_normal((777, d))).astype(np.float32)
        q = (x[rng.integers(0, len(x), nq)] + 0.1 * rng.standard_normal((nq, d))).astype(np.float32)
        if what != "equal vectors":
            q[:, 3] = np.where(np.arange(nq) % 2, np.nan, np.inf)
        print("survivors", d, M, nbits, what, flush=True)
        both_scans(vs, ix, dev(other), 100, 24)
        both_scans(vs, ix, dev(q), k, nprobe)
        n = ix.search_stats(dev(q), k, nprobe)[2]["list_major_rescanned"]
        assert 0 < n <= nq, n        # (some had no room and were scanned again)
    finally:
        ix.close()
