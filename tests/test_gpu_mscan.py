"""The matrix-core scan of inverted lists against the query-major scan: every distance and id bit for bit (parity with
the oracle is the query-major scan's, checked elsewhere).  Sizes at the edges of its blocks of 16 and units of 32
codes, its groups of 16 to 64 queries, its selection widths and its candidate buffers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

L2, IP = 0, 1


@pytest.fixture(scope="module")
def vs():
    import paper_2401_08281_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return m


def lists_of(rng, d, sizes):
    """Centroids far apart and `sizes[l]` vectors around each."""
    cent = (40.0 * rng.standard_normal((len(sizes), d))).astype(np.float32)
    x = np.concatenate([cent[l] + rng.standard_normal((n, d)).astype(np.float32) for l, n in enumerate(sizes)])
    return cent, x[rng.permutation(len(x))]


def make(vs, kind, d, M, nbits, metric, cent, x, rng):
    cent_d = torch.from_numpy(cent).cuda()
    if kind == "pq":
        cb = rng.standard_normal((M, 1 << nbits, d // M)).astype(np.float32)
        ix = vs.IVFPQ(d, metric, cent_d, torch.from_numpy(cb).cuda(), nbits=nbits)
    elif kind == "flat":
        ix = vs.IVFFlat(d, metric, cent_d)
    else:
        ok = x[np.isfinite(x).all(1)]
        lo, hi = ok.min(0), ok.max(0)
        ix = vs.IVFSQ8(d, metric, cent_d, torch.from_numpy(lo).cuda(), torch.from_numpy((hi - lo) / 255).cuda())
    return ix


def same(a, b):
    return bool((a.view(torch.int32) == b.view(torch.int32)).all()) if a.is_floating_point() else torch.equal(a, b)


# kind, d, M, bits, metric, search type, queries, k, probes
CASES = [
    ("pq", 32, 8, 8, L2, 0, 65, 10, 9), ("pq", 32, 8, 8, L2, 1, 333, 64, 9), ("pq", 32, 8, 8, IP, 0, 130, 65, 64),
    ("pq", 128, 16, 8, L2, 0, 333, 1, 9), ("pq", 128, 16, 8, L2, 2, 129, 100, 33), ("pq", 128, 16, 8, IP, 0, 64, 128, 9),
    ("pq", 96, 32, 8, L2, 0, 333, 100, 33), ("pq", 96, 32, 8, L2, 1, 65, 16, 9), ("pq", 96, 32, 8, IP, 0, 63, 17, 1),
    ("pq", 100, 20, 8, L2, 0, 130, 10, 9), ("pq", 64, 32, 4, L2, 0, 333, 33, 9), ("pq", 64, 32, 4, IP, 0, 17, 128, 64),
    # 4-bit inner products as one-hot rows: 2, 4 and 8 code bytes of a lane, sub-vectors of 1 to 12 dimensions
    ("pq", 768, 64, 4, IP, 0, 333, 10, 33), ("pq", 320, 64, 4, IP, 0, 65, 128, 9), ("pq", 160, 32, 4, IP, 0, 130, 65, 64),
    ("pq", 16, 16, 4, IP, 0, 333, 1, 9), ("pq", 144, 16, 4, IP, 0, 17, 100, 33),
    ("flat", 32, 0, 0, L2, 0, 333, 10, 9), ("flat", 128, 0, 0, L2, 0, 65, 128, 33), ("flat", 161, 0, 0, IP, 0, 130, 5, 9),
    ("flat", 250, 0, 0, L2, 0, 16, 1, 64),
    ("sq8", 33, 0, 0, L2, 0, 333, 10, 9), ("sq8", 96, 0, 0, IP, 0, 129, 65, 33), ("sq8", 256, 0, 0, L2, 0, 17, 64, 9),
]


@pytest.mark.parametrize("kind,d,M,nbits,metric,form,nq,k,nprobe", CASES)
def test_matrix_scan_equals_query_major(vs, kind, d, M, nbits, metric, form, nq, k, nprobe):
    rng = np.random.default_rng(d * 1000 + nq + k)
    edges = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 255, 256, 257, 1023, 1025]
    sizes = edges * 3 + list(rng.integers(0, 300, 16))
    cent, x = lists_of(rng, d, sizes)
    # queries near the vectors, one far from everything, one on a centroid, one that is not finite
    q = (x[rng.integers(0, len(x), nq)] + 0.3 * rng.standard_normal((nq, d))).astype(np.float32)
    q[0], q[1] = 1e4, cent[1]
    q[-1, 0] = np.nan if metric == L2 else np.inf
    if kind == "flat":
        x[:3, 1] = (np.nan, np.inf, 1e30)                       # no fp16 images
    x[-40:] = x[-1]                                             # ties
    ix = make(vs, kind, d, M, nbits, metric, cent, x, rng)
    try:
        if form:
            ix.set_search_type(form)
        xd, qd = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
        for part in xd.split((len(x) + 2) // 3):                # several calls: the copy of the codes is made again
            ix.add(part.contiguous())
        vs.vs_set_option("matrix_scan", -1)
        D0, I0 = [t.clone() for t in ix.search(qd, k, nprobe)]
        vs.vs_set_option("matrix_scan", 1)
        # (64 candidates: buffers overflow; a negative scale: every query is left to the query-major scan)
        for cand, eps in ((1024, 1.0), (64, 1.0), (1024, -1.0), (1024, 1.0)):
            vs.vs_set_option("list_major_candidates", cand)
            vs.vs_set_option("knn_eps_scale", eps)
            D1, I1 = ix.search(qd, k, nprobe)
            torch.cuda.synchronize()
            assert same(D0, D1) and same(I0, I1), (cand, eps)
            if kind == "pq":
                n = ix.search_stats(qd, k, nprobe)[2]["list_major_rescanned"]
                assert n == nq if eps < 0 else (n < nq or cand < 1024), (cand, eps, n)
        # captured: every replay against the eager query-major search of the same queries
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            ix.search(qd, k, nprobe)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            D1, I1 = ix.search(qd, k, nprobe)
        for rep in range(3):
            qd.copy_(qd.flip(0).clone())
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            vs.vs_set_option("matrix_scan", -1)
            D2, I2 = ix.search(qd, k, nprobe)
            vs.vs_set_option("matrix_scan", 1)
            torch.cuda.synchronize()
            assert same(D1, D2) and same(I1, I2), "replay %d" % rep
    finally:
        for name, value in (("matrix_scan", 0), ("list_major_candidates", 1024), ("knn_eps_scale", 1.0)):
            vs.vs_set_option(name, value)
        ix.close()
