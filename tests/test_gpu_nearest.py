"""Nearest rows, nearest codewords and ragged exact search on the matrix cores against the canon
tiles (option knn_path = 1) and the CPU oracle.  Every comparison of ids, codes and distances is exact:
the matrix cores only shortlist, the canon chain decides.  Needs a real MI355X."""
import numpy as np
import pytest

from test_gpu_parity import dev, host, say, vs  # noqa: F401  (vs: fixture)

pytestmark = pytest.mark.gpu

L2, IP = 0, 1


def rows(kind, n, d, seed):
    rng = np.random.default_rng(seed)
    if kind == "sift":
        return np.rint(np.clip(rng.uniform(0, 255, (50, d))[rng.integers(0, 50, n)] + 20 * rng.standard_normal((n, d)),
                               0, 255)).astype(np.float32)
    x = rng.standard_normal((n, d)).astype(np.float32)
    return x * np.float32({"gauss": 1.0, "beyond_fp16": 3e5, "tiny": 1e-18}[kind])


def both_routes(vs, call, counted=None):
    """call() by the canon tiles, and by the matrix cores: where the library chooses them and wherever there
    is a kernel (the results of these two agree).  counted: the rows that the latter has to count."""
    def by(path):
        try:
            vs.vs_set_option("knn_path", path)
            vs.vs_counters_read()
            out = [host(t).copy() for t in call()]
            return out, vs.vs_counters_read()[0]
        finally:
            vs.vs_set_option("knn_path", 0)
    canon, rows_canon = by(1)
    chosen, _ = by(0)
    forced, rows_forced = by(2)
    assert rows_canon == 0
    if counted is not None:
        assert rows_forced == counted
    for a, b in zip(chosen, forced):
        np.testing.assert_array_equal(a, b)
    return canon, forced


# Parts of an add below n * rows * d = 2e9, where the canon tiles are chosen, go to the sweep by knn_path = 2.
# d: both ends of the range, every padded length, remainders of 4, 2 and 1; rows of B: one step and a
# remainder, one past a step, a split; n: one past a tile, remainders.
NEAREST_CASES = [
    ("d17", 131_073, 300, 17, L2, "gauss"), ("d30_ip", 80_001, 300, 30, IP, "gauss"),
    ("d32", 60_033, 321, 32, L2, "sift"), ("d64_ip", 30_001, 320, 64, IP, "gauss"),
    ("d66", 40_960, 257, 66, L2, "gauss"), ("d96", 20_001, 350, 96, L2, "gauss"),
    ("d100", 25_700, 256, 100, L2, "sift"), ("d128", 65_537, 129, 128, L2, "sift"),
    ("d127_ip", 20_481, 260, 127, IP, "gauss"), ("b_split", 700, 8_193, 128, L2, "sift"),
    ("few_rows", 600_001, 9, 128, L2, "gauss"),
    ("beyond_fp16", 30_001, 333, 72, L2, "beyond_fp16"), ("beyond_fp16_ip", 30_001, 333, 128, IP, "beyond_fp16"),
    ("tiny", 20_001, 300, 128, L2, "tiny"),
]


@pytest.mark.parametrize("name,n,nb,d,metric,kind", NEAREST_CASES, ids=[c[0] for c in NEAREST_CASES])
@pytest.mark.parametrize("special", ["plain", "ties_and_nonfinite"])
def test_nearest_row_sweep_equals_canon_tiles(vs, name, n, nb, d, metric, kind, special):
    """List assignment, in two parts.  Second variant: centroids that occur twice (the smaller one wins), and
    in both parts vectors that are a centroid, hold an infinity, a NaN or only zeros, the last one too."""
    say("nearest %s n=%d nb=%d d=%d metric=%d %s" % (name, n, nb, d, metric, special))
    x = rows(kind, n, d, 1)
    cent = rows(kind, nb, d, 2)
    if special != "plain":
        cent[nb // 2:] = cent[:nb - nb // 2]
        for part in (x[:n // 3], x[n // 3:]):
            part[5:5 + nb // 2:2] = cent[:len(part[5:5 + nb // 2:2])]
            part[1, d - 1], part[2, 0], part[3], part[-1, 0] = np.inf, np.nan, 0.0, -np.inf
    xd, cd = dev(x), dev(cent)

    def call():
        ix = vs.IVFFlat(d, metric, cd)
        ix.add(xd[:n // 3])
        ix.add(xd[n // 3:])
        out = ix.list_sizes(), ix.storage()[0]
        ix.close()
        return out
    canon, got = both_routes(vs, call, n)
    for a, b in zip(canon, got):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("d", [17, 31, 32, 33, 48, 63, 64, 65, 80, 96, 97, 112, 127, 128])
def test_small_sweeps_equal_canon_tiles(vs, d):
    """Fewer vectors than a wavefront, a workgroup, a tile has, and one more; rows of B around one step of 64,
    and enough for splits of several sizes; fp16 heads, bf16 (values beyond fp16), exact operands."""
    for n in (1, 31, 65, 256, 257, 641):
        for nb, kind, metric in ((1, "gauss", L2), (2, "sift", IP), (63, "beyond_fp16", L2), (64, "gauss", IP),
                                 (65, "sift", L2), (513, "gauss", L2), (2_000, "beyond_fp16", IP), (2_049, "gauss", L2)):
            say("small sweep n=%d nb=%d d=%d metric=%d %s" % (n, nb, d, metric, kind))
            x, cent = rows(kind, n, d, 15), rows(kind, nb, d, 16)
            cent[nb // 2:] = cent[:nb - nb // 2]
            x[-1] = cent[-1]
            xd, cd = dev(x), dev(cent)

            def call():
                ix = vs.IVFFlat(d, metric, cd)
                ix.add(xd)
                out = ix.list_sizes(), ix.storage()[0]
                ix.close()
                return out
            canon, got = both_routes(vs, call, n)
            for a, b in zip(canon, got):
                np.testing.assert_array_equal(a, b)


def test_knn_path_2_takes_small_assignments_to_the_matrix_cores(vs):
    x, cent = dev(rows("gauss", 100, 64, 17)), dev(rows("gauss", 50, 64, 18))
    ix = vs.IVFFlat(64, L2, cent)
    try:
        for path, rows_counted in ((0, 0), (2, 100), (1, 0)):
            vs.vs_set_option("knn_path", path)
            assert add_and_count(vs, ix, x)[0] == rows_counted
            vs.vs_kmeans(x, cent.clone(), 3)
            assert vs.vs_counters_read()[0] == 3 * rows_counted
    finally:
        vs.vs_set_option("knn_path", 0)
    ix.close()


@pytest.mark.parametrize("kind", ["all_nan", "one_inf", "huge", "inf_among_few_ip"])
def test_nearest_row_sweep_with_nonfinite_centroids(vs, kind):
    say("nearest, centroids %s" % kind)
    n, nb, metric = (1_100_000, 9, IP) if kind == "inf_among_few_ip" else (40_001, 257, L2)
    x, cent = rows("gauss", n, 64, 3), rows("gauss", nb, 64, 4)
    if kind == "all_nan":
        cent[:] = np.nan
    elif kind == "huge":
        cent[::2] *= np.float32(1e19)
    else:
        cent[7, 3] = -np.inf
    xd, cd = dev(x), dev(cent)

    def call():
        ix = vs.IVFFlat(64, metric, cd)
        ix.add(xd)
        return ix.list_sizes(), ix.storage()[0]
    canon, got = both_routes(vs, call)
    for a, b in zip(canon, got):
        np.testing.assert_array_equal(a, b)


# Ordinary centroids (fp16 heads) next to vectors of which one, a few or all components are beyond the
# fp16 range: only 12 rows of B have positive partners of these components (score +infinity), the
# others have zeros (NaN).  The last vector is among them and n leaves lanes past the list's end.
@pytest.mark.parametrize("metric", [L2, IP])
@pytest.mark.parametrize("d", [32, 96, 100, 128])
@pytest.mark.parametrize("which", ["one", "few", "all", "infinite"])
def test_vectors_beyond_the_fp16_range_next_to_ordinary_centroids(vs, which, d, metric):
    say("nearest, %s component(s) beyond fp16, d=%d metric=%d" % (which, d, metric))
    n, nb = 701, 16_500                                 # (more than 16384 rows of B: always the sweep)
    x, cent = rows("gauss", n, d, 12), rows("gauss", nb, d, 13)
    cols = np.arange(d) if which == "all" else np.arange(3, d, d // 5)[:{"one": 1, "few": 5, "infinite": 1}[which]]
    some = np.random.default_rng(14).choice(nb, 12, replace=False)
    positive = np.abs(cent[some][:, cols])
    if which != "all":
        cent[:, cols] = 0.0
    cent[np.ix_(some, cols)] = positive
    large = np.arange(n) if which == "all" else np.arange(n - 1, 0, -3)
    x[np.ix_(large, cols)] = np.inf if which == "infinite" else 1e5
    xd, cd = dev(x), dev(cent)

    def call():
        ix = vs.IVFFlat(d, metric, cd)
        ix.add(xd)
        out = ix.list_sizes(), ix.storage()[0]
        ix.close()
        return out
    canon, got = both_routes(vs, call)
    for a, b in zip(canon, got):
        np.testing.assert_array_equal(a, b)


# runs of lists that get nothing: as long as one lane fills, one shorter, one longer, and the whole table
# before, between and behind the vectors of one or two lists; more ranks than one workgroup has
@pytest.mark.parametrize("nlist,hit", [(1, [0]), (70_001, [0]), (70_001, [70_000]), (70_001, [40_000]),
                                       (70_001, [3, 35, 66, 99, 131, 70_000]), (1_100, [0, 1_099] * 600),
                                       (5_000, list(range(31, 5_000, 33)) * 9)])
def test_offsets_of_adds_that_leave_most_lists_as_they_are(vs, nlist, hit):
    say("placement, %d vectors into %d lists" % (len(hit), nlist))
    cent = np.zeros((nlist, 2), dtype=np.float32)
    cent[:, 0] = np.arange(nlist)
    ix = vs.IVFFlat(2, L2, dev(cent))
    lists, ids = [[] for _ in range(nlist)], 0
    for batch in (hit, hit[:1], hit[::-1]):
        ix.add(dev(cent[batch]))
        for l in batch:
            lists[l].append(ids)
            ids += 1
    np.testing.assert_array_equal(host(ix.list_sizes()), [len(l) for l in lists])
    got = ix.storage()
    np.testing.assert_array_equal(host(got[0]), [i for l in lists for i in l])
    ix.close()


def well_separated(n, nb, d, seed, far=3):
    """Vectors near centroids that are far apart, so that the first sweep is certain of every one, but for
    the first `far`: their first component, which only centroid 5 has, is beyond what the fp16 heads
    may hold, while bf16 products are certain of them.  The number of exact fallbacks thus tells which
    products a call used: `far` by fp16 heads, none by bf16."""
    cent = 10 * rows("gauss", nb, d, seed)
    cent[:, 0] = 0.0
    x = cent[np.random.default_rng(seed).integers(6, nb, n)] + rows("gauss", n, d, seed + 1)
    x[:, 0] = 0.0
    cent[5, 0] = 1000.0
    x[:far, 0] = 40_000.0
    return dev(x), dev(cent)


def add_and_count(vs, ix, x):
    vs.vs_counters_read()
    ix.add(x)
    return vs.vs_counters_read()


def test_counters_cover_the_one_sweep_route_and_forced_fallbacks_teach_nothing(vs):
    n, nb, d = 75_000, 300, 96
    say("counters of the sweep n=%d nb=%d d=%d" % (n, nb, d))
    x, cent = well_separated(n, nb, d, 20)
    ix = vs.IVFFlat(d, L2, cent)
    assert add_and_count(vs, ix, x) == (n, 3)
    try:
        vs.vs_set_option("knn_eps_scale", -1.0)
        assert add_and_count(vs, ix, x) == (n, n)
    finally:
        vs.vs_set_option("knn_eps_scale", 1.0)
    assert add_and_count(vs, ix, x) == (n, 3)          # (0 had the forced call moved the index to bf16)
    c = cent.clone()
    vs.vs_kmeans(x, c, 2)
    assert vs.vs_counters_read()[0] == 2 * n
    ix.close()


def tight_groups(n, d, size, share, seed):
    """Groups of `size` centroids whose squared distances to the group's centre are 0, 0.95, 1.9, ..., the
    centres some 100 times that apart, and vectors at the centres (`share` of them; the others are at
    centroids that stand alone).  |a|^2 + max |b|^2 is about 200 d: the fp16 bound, 9.8e-4 of it (19 at
    d = 96), takes in a whole group of 20, the bf16 bound, some 1.2e-4 of it, three or four."""
    g = np.random.default_rng(seed)
    centres = 10 * g.standard_normal((30, d))
    centres *= 10 * np.sqrt(d) / np.linalg.norm(centres, axis=1, keepdims=True)
    step = g.standard_normal((30, size, d))
    step *= np.sqrt(0.95 * np.arange(size))[None, :, None] / np.linalg.norm(step, axis=2, keepdims=True)
    alone = 10 * g.standard_normal((100, d))
    alone *= 10 * np.sqrt(d) / np.linalg.norm(alone, axis=1, keepdims=True)
    cent = np.concatenate([(centres[:, None] + step).reshape(-1, d), alone])
    x = alone[g.integers(0, 100, n)]
    at = g.random(n) < share
    x[at] = centres[g.integers(0, 30, at.sum())]
    x += 0.01 * g.standard_normal((n, d))
    return dev(x.astype(np.float32)), dev(cent.astype(np.float32)), int(at.sum())


@pytest.mark.parametrize("d,metric", [(96, L2), (96, IP), (60, L2)])
def test_vectors_that_the_heads_leave_are_swept_with_more_products(vs, d, metric):
    """40 % of the vectors have more rows within the fp16 bound than the candidate list holds: they are
    not redone by the canon chain over all rows, in no call."""
    n = 12_001
    say("tight groups n=%d d=%d metric=%d" % (n, d, metric))
    x, cent, tight = tight_groups(n, d, 20, 0.4, 24)
    assert tight * 512 > n

    def call():
        ix = vs.IVFFlat(d, metric, cent)
        ix.add(x)
        out = ix.list_sizes(), ix.storage()[0]
        ix.close()
        return out
    canon, got = both_routes(vs, call, n)
    for a, b in zip(canon, got):
        np.testing.assert_array_equal(a, b)
    ix = vs.IVFFlat(d, metric, cent)
    vs.vs_set_option("knn_path", 2)
    try:
        for _ in range(2):
            rows_counted, redone = add_and_count(vs, ix, x)
            assert rows_counted == n
            if metric == L2 and d == 96:
                assert redone * 512 <= n, redone
    finally:
        vs.vs_set_option("knn_path", 0)
    ix.close()


def test_a_search_with_one_probe_teaches_the_sweep_nothing(vs):
    """A search at nprobe = 1 gives up the fp16 heads for its own kind after one row in 512 redone; the
    one-sweep route, which has a rule of its own, still begins with them (3 vectors left, see above)."""
    n, nb, d = 75_000, 300, 96
    say("one-probe search, then an add: n=%d nb=%d d=%d" % (n, nb, d))
    x, cent = well_separated(n, nb, d, 20)
    q, tight, _ = tight_groups(2_000, d, 64, 1.0, 25)
    import torch
    cent = torch.cat([cent, tight + 0.0])
    ix = vs.IVFFlat(d, L2, cent)
    assert add_and_count(vs, ix, x)[1] == 3
    vs.vs_set_option("knn_path", 2)
    try:
        vs.vs_counters_read()
        ix.search(q, 1, 1)
        assert vs.vs_counters_read()[1] * 512 > 2_000          # the rule's condition
    finally:
        vs.vs_set_option("knn_path", 0)
    assert add_and_count(vs, ix, x)[1] == 3
    ix.close()


@pytest.mark.parametrize("n,d,K", [(20_001, 128, 300), (130_001, 17, 300), (1_500, 32, 16_385)])
def test_kmeans_sweep_equals_canon_tiles(vs, n, d, K):
    """Three rounds: objective, assignment and centroids, with the bookkeeping on the device and
    (K > 16384) on the host."""
    say("kmeans n=%d d=%d K=%d" % (n, d, K))
    x = rows("sift", n, d, 5)
    init = np.resize(x, (K, d)) + (np.arange(K) // n)[:, None].astype(np.float32)
    xd = dev(x)

    def call():
        c = dev(init)
        obj, assign = vs.vs_kmeans(xd, c, 3, return_assign=True)
        return c, assign, dev(np.array(obj))
    canon, got = both_routes(vs, call)
    for a, b in zip(canon, got):
        np.testing.assert_array_equal(a, b)


# d: both ends of the lanes of 8, 16 and 32 and of one and two wavefronts of dimensions
@pytest.mark.parametrize("d", [1, 8, 9, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("sizes", ["edges", "one_holds_most", "only_the_last", "many_centroids"])
def test_means_of_clusters_of_all_sizes(vs, d, sizes):
    """The mean of a cluster is its float64 sum in blocks of 4096 vectors, in their order, over its size;
    a centroid without vectors keeps its place."""
    say("means of clusters, %s d=%d" % (sizes, d))
    size = {"edges": [0, 1, 31, 32, 33, 0, 4_095, 4_096, 4_097, 8_191, 8_192, 8_193, 12_289, 64, 0],
            "one_holds_most": [3, 0, 70_001, 0, 0, 5] + [1] * 70, "only_the_last": [0] * 9 + [20_481],
            "many_centroids": [0, 2, 0, 3] * 1_100 + [4_100] + [1] * 20}[sizes]
    K, g = len(size), np.random.default_rng(31)
    cent = np.zeros((K, d), dtype=np.float32)
    cent[:, 0] = 1000.0 * np.arange(K)
    own = g.permutation(np.repeat(np.arange(K), size))
    x = (cent[own] + g.standard_normal((len(own), d))).astype(np.float32)
    want = cent.copy()
    for j in range(K):
        mine = x[own == j].astype(np.float64)
        if len(mine):
            sums = [np.cumsum(mine[b:b + 4096], axis=0)[-1] for b in range(0, len(mine), 4096)]
            want[j] = np.cumsum(sums, axis=0)[-1] / len(mine)
    got = dev(cent)
    _, assign = vs.vs_kmeans(dev(x), got, 1, return_assign=True)
    np.testing.assert_array_equal(host(assign), own)
    np.testing.assert_array_equal(host(got), want)


# dsub: one and two groups of eight dimensions, both with remainders; 17 takes the vector kernel.
# n: below one group of 32 vectors, one past a workgroup's 128.
@pytest.mark.parametrize("nbits", [4, 8])
@pytest.mark.parametrize("dsub", [1, 2, 3, 4, 7, 8, 9, 12, 15, 16, 17])
@pytest.mark.parametrize("n,M", [(19, 4), (4_225, 6)])
def test_nearest_codewords_match_oracle(vs, oracle, n, M, dsub, nbits):
    say("encode n=%d M=%d dsub=%d nbits=%d" % (n, M, dsub, nbits))
    d, K = M * dsub, 1 << nbits
    x, cent = rows("sift", n, d, 6), rows("sift", 7, d, 7)
    cb = rows("sift", K, d, 8).reshape(K, M, dsub).transpose(1, 0, 2) - 128.0
    cb[0, K // 2:] = cb[0, :K // 2]                    # every codeword of the first one twice
    cb[1, 1:] *= np.float32(1e4)                       # one small codeword among large ones
    cb = np.ascontiguousarray(cb, dtype=np.float32)
    ix = vs.IVFPQ(d, L2, dev(cent), dev(cb), nbits)
    ix.add(dev(x))
    orc = oracle.OracleIVFPQ(d, L2, cent, cb, nbits)
    orc.add(x)
    np.testing.assert_array_equal(host(ix.codes()), orc.codes)


@pytest.mark.parametrize("nbits", [4, 8])
@pytest.mark.parametrize("dsub", [1, 3, 4, 8, 9, 16])
@pytest.mark.parametrize("gap", [1, 2, 3, 4, 8, 13])
def test_twin_codewords_of_one_four_and_of_two(vs, oracle, dsub, nbits, gap):
    """The kernel selects fours of consecutive codewords: twins `gap` apart lie in one or in two of them, equal (the
    smaller number wins) or one rounding apart, where the canon chain decides."""
    say("twins dsub=%d nbits=%d gap=%d" % (dsub, nbits, gap))
    n, M, K = 2_113, 4, 1 << nbits
    d = M * dsub
    x, cent = rows("gauss", n, d, 60), rows("gauss", 3, d, 61)
    cb = np.ascontiguousarray(rows("gauss", K, d, 62).reshape(K, M, dsub).transpose(1, 0, 2))
    for j in range(0, K - gap, 2 * gap):
        cb[0, j + gap] = cb[0, j]
        cb[1, j + gap] = np.nextafter(cb[1, j], np.float32(9), dtype=np.float32)
        cb[2, j] = np.nextafter(cb[2, j + gap], np.float32(-9), dtype=np.float32)
    ix = vs.IVFPQ(d, L2, dev(cent), dev(cb), nbits)
    ix.add(dev(x))
    orc = oracle.OracleIVFPQ(d, L2, cent, cb, nbits)
    orc.add(x)
    np.testing.assert_array_equal(host(ix.codes()), orc.codes)


@pytest.mark.parametrize("nbits", [4, 8])
@pytest.mark.parametrize("dsub", [2, 5, 8, 12, 16])
@pytest.mark.parametrize("kind", ["gauss", "tiny", "huge", "nonfinite_vectors", "nonfinite_codewords"])
def test_nearest_codewords_on_all_routes(vs, kind, dsub, nbits):
    """Codes by the canon chain alone (knn_path = 1), by the matrix cores, and by their canon branch for every
    sub-vector (knn_eps_scale < 0); training likewise."""
    say("codes on all routes, %s dsub=%d nbits=%d" % (kind, dsub, nbits))
    n, M, K = 1_061, 4, 1 << nbits
    d = M * dsub
    scale = np.float32({"tiny": 1e-20, "huge": 3e18}.get(kind, 1.0))
    x, cent = rows("gauss", n, d, 40) * scale, rows("gauss", 5, d, 41) * scale
    cb = np.ascontiguousarray(rows("gauss", K, d, 42).reshape(K, M, dsub).transpose(1, 0, 2)) * scale
    cb[0, K // 2] = cb[0, 1]
    if kind == "nonfinite_vectors":
        x[5, 0], x[6, 1], x[7, d - 1], x[8] = np.nan, np.inf, -np.inf, np.nan
    if kind == "nonfinite_codewords":
        cb[0, 3, 0], cb[0, 0, 1], cb[1, 0, 0], cb[1, K - 1, 1] = np.nan, np.inf, np.nan, -np.inf
        cb[2, :, 0] = np.inf
        cb[2, 0, 0] = np.nan
    xd, cd, bd = dev(x), dev(cent), dev(cb)

    def codes():
        ix = vs.IVFPQ(d, L2, cd, bd, nbits)
        ix.add(xd)
        out = host(ix.codes()).copy(), host(ix.list_sizes()).copy()
        ix.close()
        return out

    def trained():
        c, b = cd.clone(), bd.clone()
        vs.vs_ivfpq_train(xd, L2, c, b, nbits, 2)
        return host(c).copy(), host(b).copy()
    for call in (codes, trained):
        got = {}
        for path, eps in ((0, 1.0), (1, 1.0), (0, -1.0)):
            try:
                vs.vs_set_option("knn_path", path)
                vs.vs_set_option("knn_eps_scale", eps)
                got[path, eps] = call()
            finally:
                vs.vs_set_option("knn_path", 0)
                vs.vs_set_option("knn_eps_scale", 1.0)
        for other in ((0, 1.0), (0, -1.0)):
            for a, b in zip(got[1, 1.0], got[other]):
                np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n,d,M,nbits,niter", [(5_003, 12, 4, 8, 3), (5_003, 24, 2, 4, 3), (9_001, 34, 2, 8, 2),
                                               (3_000_001, 32, 32, 4, 2)])
def test_subquantizers_together_equal_one_at_a_time(vs, n, d, M, nbits, niter):
    """The last shape's work space is beyond one group of sub-quantizers; 17 dimensions are not taken
    together."""
    say("train n=%d d=%d M=%d nbits=%d" % (n, d, M, nbits))
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    x = torch.randn((n, d), generator=g, device="cuda")
    cent = x[:16].clone()
    cb = torch.randn((M, 1 << nbits, d // M), generator=g, device="cuda")

    def call():
        c, b = cent.clone(), cb.clone()
        obj = vs.vs_ivfpq_train(x, L2, c, b, nbits, niter)
        return c, b, torch.tensor(obj, dtype=torch.float64, device="cuda")
    canon, got = both_routes(vs, call)
    for a, b in zip(canon, got):
        np.testing.assert_array_equal(a, b)


# rows of B on both sides of one canon tile (16384), lengths between the padded ones
@pytest.mark.parametrize("nb,nq,d,k,metric", [
    (16_384, 3, 100, 10, L2), (16_385, 3, 100, 10, L2), (20_003, 130, 17, 1, IP), (20_003, 65, 33, 100, L2),
    (9_001, 700, 129, 10, IP), (4_097, 600, 257, 10, L2), (1_201, 700, 770, 150, L2)])
def test_ragged_exact_search_equals_canon_tiles(vs, nb, nq, d, k, metric):
    say("ragged flat nb=%d nq=%d d=%d k=%d metric=%d" % (nb, nq, d, k, metric))
    x, q = dev(rows("gauss", nb, d, 10)), dev(rows("gauss", nq, d, 11))
    ix = vs.Flat(d, metric)
    ix.add(x)
    for call in (lambda: vs.vs_flat_search(x, q, k, metric), lambda: ix.search(q, k)):
        canon, got = both_routes(vs, call)
        for a, b in zip(canon, got):
            np.testing.assert_array_equal(a, b)


# both list sizes of the canon tiles' selection and the values of k between which they change
@pytest.mark.parametrize("k", [47, 48, 49, 63, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("nb", [40, 64, 3_001, 16_500])
def test_selection_at_the_sizes_of_its_lists(vs, nb, k):
    say("selection nb=%d k=%d" % (nb, k))
    x, q = rows("sift", nb, 40, 47), dev(rows("sift", 70, 40, 48))
    x[nb // 2:] = x[:nb - nb // 2]                      # ties
    xd = dev(x)
    canon, got = both_routes(vs, lambda: vs.vs_flat_search(xd, q, k, L2))
    for a, b in zip(canon, got):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("d", [33, 50, 64])
def test_products_that_underflow_tie_alike_on_all_routes(vs, d):
    """Inner products of +0 and, in some rows, of a product that underflows to -0 in the last dimension, far
    ahead of all others: where rows are padded to whole blocks of 32 the zeros make both +0 (a tie)."""
    say("underflowing products d=%d" % d)
    nb, nq = 20_003, 40
    x, q = np.zeros((nb, d), dtype=np.float32), np.zeros((nq, d), dtype=np.float32)
    x[:, 0] = -1.0
    special = np.arange(100, 112)
    x[special, 0] = 0.0
    x[special, d - 1] = np.where(special % 2 == 0, np.float32(-1e-23), np.float32(1e-23))
    q[:, 0], q[:, d - 1] = 1.0, 1e-23
    xd, qd = dev(x), dev(q)

    def assigned():
        ix = vs.IVFFlat(d, IP, xd)
        ix.add(qd)
        out = (ix.list_sizes(),)
        ix.close()
        return out
    for call in (lambda: vs.vs_flat_search(xd, qd, 8, IP), assigned):
        canon, got = both_routes(vs, call)
        for a, b in zip(canon, got):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("d", [33, 64, 100])
@pytest.mark.parametrize("metric", [L2, IP])
@pytest.mark.parametrize("scale", [1e-18, 1e-19, 1e-20, 1e-22])
def test_exact_search_of_tiny_values(vs, scale, d, metric):
    """Products near and below the smallest normal number, which the matrix cores may drop."""
    say("tiny values %g d=%d metric=%d" % (scale, d, metric))
    x, q = dev(rows("gauss", 5_001, d, 45) * np.float32(scale)), dev(rows("gauss", 300, d, 46) * np.float32(scale))
    canon, got = both_routes(vs, lambda: vs.vs_flat_search(x, q, 10, metric))
    for a, b in zip(canon, got):
        np.testing.assert_array_equal(a, b)


def test_static_search_accepts_what_fits_by_the_matrix_core_route(vs):
    """The canon tiles of a small problem can be larger than the fixed work space (600 x 16384 scores:
    40 MiB) where the matrix-core route's shortlist fits it: the call is served, with the same results."""
    import ctypes
    import torch
    d, nlist, M, nq = 32, 16384, 8, 600
    say("static search nlist=%d nq=%d d=%d" % (nlist, nq, d))
    x = dev(rows("gauss", 40_000, d, 5))
    q = dev(rows("gauss", nq, d, 6))
    ix = vs.IVFPQ(d, L2, x[:nlist].contiguous(), x[:256].view(256, M, d // M).permute(1, 0, 2).contiguous(), 8)
    ix.add(x)
    D, I = ix.search(q, 3, 1)
    d2, i2 = torch.empty_like(D), torch.empty_like(I)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = vs.lib().vs_ivfpq_search_static(ix.h, p(q), nq, 3, 1, p(d2), p(i2),
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    np.testing.assert_array_equal(host(I), host(i2))
    np.testing.assert_array_equal(host(D), host(d2))


@pytest.mark.parametrize("niter", [255, 256, 257, 600])
def test_objective_of_many_rounds(vs, niter):
    """The sums of the objective are kept for 256 rounds: a long run's objective is that of its parts."""
    import torch
    say("objective of %d rounds" % niter)
    n, d, K, first = 700, 6, 90, 100
    x = dev(rows("gauss", n, d, 33))
    whole, parts = x[:K].clone(), x[:K].clone()
    obj = vs.vs_kmeans(x, whole, niter)
    want = list(vs.vs_kmeans(x, parts, first)) + list(vs.vs_kmeans(x, parts, niter - first))
    np.testing.assert_array_equal(obj, want)
    np.testing.assert_array_equal(host(whole), host(parts))
    cent = torch.zeros((1, d), device="cuda")
    cb = x[:16].reshape(16, 2, 3).permute(1, 0, 2).contiguous()
    got = vs.vs_ivfpq_train(x, L2, cent, cb.clone(), 4, niter)
    res = (x - cent).reshape(n, 2, 3)
    for m in range(2):
        np.testing.assert_array_equal(np.array(got)[1 + m], vs.vs_kmeans(res[:, m].contiguous(), cb[m].clone(), niter))


def hold_memory(need):
    """Tensors that leave `need` bytes of device memory (what the driver reports as free is not all there is)."""
    import torch
    chunk, held = 16 << 20, []
    free = torch.cuda.mem_get_info()[0]
    if free > need + (4 << 30):
        held.append(torch.empty(free - need - (4 << 30), dtype=torch.uint8, device="cuda"))
    try:
        while True:
            held.append(torch.empty(chunk, dtype=torch.uint8, device="cuda"))
    except torch.cuda.OutOfMemoryError:
        pass
    del held[-(-(-need // chunk)):]
    torch.cuda.empty_cache()
    return held


@pytest.mark.parametrize("left", [300, 60, 14])
def test_training_with_little_memory_free(vs, left):
    """The work space of 32 sub-quantizers of 2M vectors is 576 MB together, 18 MB of one.  `left` MB more
    than the coarse part needs leave room for half of them, for two, for none."""
    import torch
    n, d, M, nbits = 2_000_001, 32, 32, 4
    say("train n=%d M=%d with %d MB to spare" % (n, M, left))
    g = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn((n, d), generator=g, device="cuda")
    cent, cb = x[:64].clone(), torch.randn((M, 1 << nbits, 1), generator=g, device="cuda")

    def call():
        c, b = cent.clone(), cb.clone()
        obj = vs.vs_ivfpq_train(x, L2, c, b, nbits, 2)
        return [host(c).copy(), host(b).copy(), np.array(obj)]
    want = call()
    vs.vs_trim()
    torch.cuda.empty_cache()
    # the coarse part, per vector: three numbers, the residual, and 97 bytes of its assignment's scratch
    need = n * (3 * 4 + 4 * d + 97) + (left << 20)
    hold = hold_memory(need)
    say("driver reports %d MB free of %d" % (torch.cuda.mem_get_info()[0] >> 20, need >> 20))
    try:
        got = call()
    finally:
        del hold
        torch.cuda.empty_cache()
        vs.vs_trim()
    for a, b in zip(want, got):
        np.testing.assert_array_equal(a, b)


def test_ragged_rows_that_leave_no_room_for_planes_use_canon_tiles(vs):
    """Operand planes of 1M x 100 take 768 MB; with less than that free the search and the index still work."""
    import torch
    n, d, nq, k = 1_000_000, 100, 40, 5
    say("ragged rows n=%d d=%d with little memory free" % (n, d))
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((n, d), generator=g, device="cuda")
    q = torch.randn((nq, d), generator=g, device="cuda")
    want = [host(t).copy() for t in vs.vs_flat_search(x, q, k, L2)]
    vs.vs_trim()
    torch.cuda.empty_cache()
    hold = torch.empty(max(0, torch.cuda.mem_get_info()[0] - (700 << 20)), dtype=torch.uint8, device="cuda")
    try:
        once = [host(t).copy() for t in vs.vs_flat_search(x, q, k, L2)]
        vs.vs_trim()
        ix = vs.Flat(d, L2)
        ix.add(x)
        kept = [host(t).copy() for t in ix.search(q, k)]
    finally:
        del hold
        torch.cuda.empty_cache()
        vs.vs_trim()
    for got in (once, kept):
        for a, b in zip(want, got):
            np.testing.assert_array_equal(a, b)
