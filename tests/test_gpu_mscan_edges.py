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
    """More survivors than their common list has room for, 4 k + 128 per query and half a million at least, and fewer of a query
    than its own buffer holds; behind another search, whose values lie where the list is."""
    rng = np.random.default_rng(d)
    k, nprobe, nq = 10, 8, 20_000
    cent, x = lists_of(rng, d, [60] * 24)
    if what == "equal vectors":
        x = np.repeat(x[rng.permutation(len(x))[:24]], 300, axis=0)       # every vector 300 times
    ix = make(vs, "pq", d, M, nbits, L2, cent, x, rng)
    try:
        ix.add(dev(x))
        other = (x[rng.integers(0, len(x), 7777)] + 20 * rng.standard_normal((7777, d))).astype(np.float32)
        q = (x[rng.integers(0, len(x), nq)] + 0.1 * rng.standard_normal((nq, d))).astype(np.float32)
        if what != "equal vectors":
            q[:, 3] = np.where(np.arange(nq) % 2, np.nan, np.inf)
        print("survivors", d, M, nbits, what, flush=True)
        both_scans(vs, ix, dev(other), 100, 24)
        both_scans(vs, ix, dev(q), k, nprobe)
        n = ix.search_stats(dev(q), k, nprobe)[2]["list_major_rescanned"]
        assert 0 < n < nq, n         # (some had no room and were scanned again)
    finally:
        ix.close()


# 32 x 3 holds |t|^2 / 2 of a codeword in its table, 16 x 8 and 20 x 5 its components only
@pytest.mark.parametrize("d,M,big", [(96, 32, 400.0), (128, 16, 1e5), (100, 20, 1e5)])
@pytest.mark.parametrize("metric", [L2, IP])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_codewords_that_are_not_finite(vs, d, M, big, metric, bad):
    """Such a codeword is never chosen; a large finite one beside it is, and its vectors are found."""
    rng = np.random.default_rng(d + M)
    cent, x = lists_of(rng, d, [150] * 16)
    cb = rng.standard_normal((M, 256, d // M)).astype(np.float32)
    cb[:, 0] = big
    cb[0, 1, 0] = bad
    x[:200] = cent[rng.integers(0, 16, 200)] + big             # coded with the large codewords
    ix = vs.IVFPQ(d, metric, dev(cent), dev(cb), nbits=8)
    try:
        ix.add(dev(x))
        q = np.concatenate([x[:60], x[300:400]]) + 0.1 * rng.standard_normal((160, d))
        D, I = both_scans(vs, ix, dev(q.astype(np.float32)), 20, 16)
        assert (I[:60, 0] < 200).float().mean() > 0.9          # (they are among the results)
    finally:
        ix.close()


# sizes at which squares overflow or vanish, sums of codewords do, or the scale itself leaves its range
@pytest.mark.parametrize("size", [1e-30, 1e-22, 1e-13, 1e-6, 1e12, 3e14, 1e19, 1e24, 1e36])
@pytest.mark.parametrize("metric", [L2, IP])
@pytest.mark.parametrize("kind,d,M,form", [("pq", 96, 32, 0), ("pq", 128, 16, 1), ("pq", 100, 20, 0), ("flat", 64, 0, 0),
                                           ("sq8", 64, 0, 0)])
def test_data_of_any_size(vs, kind, d, M, form, metric, size):
    """Distances that are infinite, vanish or are not numbers in the exact arithmetic: the same ties."""
    if form and metric == IP:
        pytest.skip("stored norms serve L2")
    rng = np.random.default_rng(d)
    cent, x = lists_of(rng, d, [100] * 12)
    with np.errstate(over="ignore", under="ignore"):
        cent, x = (cent * np.float32(size)).astype(np.float32), (x * np.float32(size)).astype(np.float32)
        q = (x[rng.integers(0, len(x), 150)] * rng.uniform(0.99, 1.01, (150, d))).astype(np.float32)
    if kind == "pq":
        cb = (rng.standard_normal((M, 256, d // M)) * size).astype(np.float32)
        ix = vs.IVFPQ(d, metric, dev(cent), dev(cb), nbits=8)
    else:
        ix = make(vs, kind, d, M, 8, metric, cent, x, rng)
    try:
        if form:
            ix.set_search_type(form)
        ix.add(dev(x))
        both_scans(vs, ix, dev(q), 10, 6)
    finally:
        ix.close()


@pytest.mark.parametrize("size", [1e-43, 1e-30, 1e-19, 1e-6, 1.0, 1e12, 1e18, 1e30])
@pytest.mark.parametrize("d,M", [(320, 64), (192, 32), (16, 16)])
@pytest.mark.parametrize("what", ["plain", "one large sub-quantizer", "equal codewords", "not finite"])
def test_one_hot_sums_of_any_size(vs, d, M, size, what):
    """4-bit inner products: tables whose entries vanish, overflow, are all equal, or of which one sub-quantizer's set the
    step of all others."""
    rng = np.random.default_rng(d + M)
    cent, x = lists_of(rng, d, [100] * 12)
    cb = rng.standard_normal((M, 16, d // M)).astype(np.float32)
    if what == "one large sub-quantizer":
        cb[3] *= 1000
    if what == "equal codewords":
        cb[:] = cb[:, :1]
    if what == "not finite":
        cb[0, 1, 0], cb[M - 1, 15, 0] = np.nan, np.inf
    with np.errstate(over="ignore", under="ignore"):
        cent, x, cb = [(a * np.float32(size)).astype(np.float32) for a in (cent, x, cb)]
        q = (x[rng.integers(0, len(x), 150)] * rng.uniform(0.9, 1.1, (150, d))).astype(np.float32)
    q[0], q[1, 0], q[2, 0] = 0, np.nan, np.inf
    ix = vs.IVFPQ(d, IP, dev(cent), dev(cb), nbits=4)
    try:
        ix.add(dev(x))
        both_scans(vs, ix, dev(q), 10, 6)
    finally:
        ix.close()


@pytest.mark.parametrize("kind,d,M", [("pq", 128, 16), ("pq", 100, 20), ("flat", 64, 0), ("sq8", 96, 0)])
def test_centroids_far_larger_than_residuals(vs, kind, d, M):
    """Stored norms and inner products whose terms are near the end of fp32 while residuals are of ordinary size."""
    rng = np.random.default_rng(d)
    for metric in (L2, IP):
        for size in (1e4, 1e12, 1e17, 4e18, 1e25):
            cent = (size * rng.standard_normal((12, d))).astype(np.float32)
            x = (cent[rng.integers(0, 12, 1200)] * rng.uniform(1 - 1e-6, 1 + 1e-6, (1200, d))).astype(np.float32)
            q = (x[rng.integers(0, 1200, 150)] * rng.uniform(1 - 1e-6, 1 + 1e-6, (150, d))).astype(np.float32)
            ix = make(vs, kind, d, M, 8, metric, cent, x, rng)
            try:
                ix.add(dev(x))
                for form in (0, 1) if kind == "pq" and metric == L2 else (0,):
                    if form:
                        ix.set_search_type(form)
                    both_scans(vs, ix, dev(q), 10, 6, (metric, size, form))
            finally:
                ix.close()


@pytest.mark.parametrize("kind,d,M", [("pq", 128, 16), ("pq", 100, 20), ("flat", 64, 0), ("sq8", 96, 0)])
@pytest.mark.parametrize("metric", [L2, IP])
def test_no_error_bound_and_no_threshold(vs, kind, d, M, metric):
    """Fewer vectors than k in the probed lists: every one is a result, also where the error bounds are scaled to nothing."""
    rng = np.random.default_rng(d)
    cent, x = lists_of(rng, d, [20] * 12)
    ix = make(vs, kind, d, M, 8, metric, cent, x, rng)
    try:
        ix.add(dev(x))
        vs.vs_set_option("knn_eps_scale", 0.0)
        D, I = both_scans(vs, ix, dev(x[:100]), 100, 4)
        assert ((I >= 0).sum(1) == 80).all()
    finally:
        ix.close()


@pytest.mark.parametrize("kind,d,M", [("pq", 96, 32), ("flat", 64, 0), ("sq8", 96, 0)])
def test_no_memory_for_the_candidates(vs, kind, d, M):
    """With too little memory for a batch's candidates, about 1 GB, the query-major scan serves it: the first call finds
    out, the next ones only enqueue kernels (they can be captured).  vs_trim and a larger index try again."""
    from test_gpu_nearest import hold_memory
    rng = np.random.default_rng(d)
    nq, k, nprobe = 30_000, 10, 8
    cent, x = lists_of(rng, d, [400] * 40)
    q = dev((x[rng.integers(0, len(x), nq)] + 0.1 * rng.standard_normal((nq, d))).astype(np.float32))
    ix = make(vs, kind, d, M, 8, L2, cent, x, rng)
    vs.vs_set_option("matrix_scan", 1)

    def route():
        vs.vs_profile_enable(1)
        vs.vs_profile_read()
        D, I = ix.search(q, k, nprobe)
        torch.cuda.synchronize()
        n = vs.vs_profile_read()
        vs.vs_profile_enable(0)
        return D, I, n

    try:
        ix.add(dev(x))
        vs.vs_trim()
        torch.cuda.empty_cache()
        print("little memory", kind, flush=True)
        out = [torch.empty((nq, k), dtype=t, device="cuda") for t in (torch.float32, torch.int64) * 2]
        D0, I0, D1, I1 = out
        hold = hold_memory(600 << 20)
        try:
            ix.search(q, k, nprobe, D0, I0)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                ix.search(q, k, nprobe, D1, I1)
            for _ in range(3):
                D1.zero_()
                g.replay()
                torch.cuda.synchronize()
                assert bool((D0 == D1).all()) and bool((I0 == I1).all())
            del g
        finally:
            del hold
            torch.cuda.empty_cache()
        D2, I2, n = route()
        assert same(D0, D2) and same(I0, I2) and not n["scan_first"][1]
        vs.vs_trim()
        D2, I2, n = route()
        assert same(D0, D2) and same(I0, I2) and n["scan_first"][1]
    finally:
        ix.close()


def test_an_add_that_has_no_room_for_the_copy_of_the_codes(vs):
    """6M codes of 16 bytes take 144 MB with their ids, their copy for the matrix cores about 98 MB more: with some 210
    MB free the codes and the copy fit, the ids then do not, and the copy goes."""
    from test_gpu_nearest import hold_memory
    n, d, M, nlist = 3_000_000, 128, 16, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((n, d), generator=g, device="cuda")
    cb = torch.randn((M, 256, d // M), generator=g, device="cuda")
    q = x[:500] + 0.1
    ix = vs.IVFPQ(d, L2, x[:nlist].contiguous(), cb, nbits=8)
    vs.vs_set_option("matrix_scan", 1)
    try:
        ix.add(x)
        vs.vs_trim()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        print("adding with little memory", flush=True)
        hold = hold_memory(200 << 20)
        try:
            ix.add(x)
        finally:
            del hold
            torch.cuda.empty_cache()
        assert ix.ntotal == 2 * n
        D, I = [t.clone() for t in ix.search(q, 20, 4)]
        vs.vs_set_option("matrix_scan", -1)
        D0, I0 = ix.search(q, 20, 4)
        torch.cuda.synchronize()
        assert same(D, D0) and same(I, I0)
        vs.vs_set_option("matrix_scan", 1)
        ix.add(x[:1000].contiguous())                           # with room again, the copy is back
        assert (both_scans(vs, ix, q, 20, 4)[1] >= 0).all()
        vs.vs_profile_enable(1)
        vs.vs_profile_read()
        ix.search(q, 20, 4)
        torch.cuda.synchronize()
        n_first = vs.vs_profile_read()["scan_first"][1]
        vs.vs_profile_enable(0)
        assert n_first
    finally:
        ix.close()


@pytest.mark.parametrize("nq,k,nprobe", [(40, 100, 64), (256, 10, 64), (1000, 100, 32)])
def test_unstructured_data_is_not_scanned_twice(vs, nq, k, nprobe):
    """Gaussian vectors and queries, coarse codes: the first lists of a query are no nearer than the others, and several
    thousand vectors of each query pass the threshold.  Their buffers hold them."""
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((300_000, 64), generator=g, device="cuda")
    cb = torch.randn((32, 16, 2), generator=g, device="cuda") * 0.8
    q = torch.randn((nq, 64), generator=g, device="cuda")
    ix = vs.IVFPQ(64, L2, x[:64].contiguous(), cb, nbits=4)
    try:
        ix.add(x)
        both_scans(vs, ix, q, k, nprobe)
        assert ix.search_stats(q, k, nprobe)[2]["list_major_rescanned"] == 0
    finally:
        ix.close()


# (kind, nlist, queries, k, probes, whether the lists are scanned on the matrix cores): either side of the lines that
# pairs per list, list length, probes and k draw
@pytest.mark.parametrize("kind,d,M,nlist,metric,nq,k,nprobe,matrix", [
    ("pq", 96, 32, 1024, L2, 512, 10, 4, False), ("pq", 96, 32, 1024, L2, 128, 100, 16, True),
    ("pq", 96, 32, 1024, L2, 800, 10, 4, True), ("pq", 96, 32, 1024, IP, 2600, 10, 4, True),
    ("pq", 96, 32, 1024, IP, 800, 10, 16, True), ("pq", 128, 16, 8192, IP, 5300, 10, 16, True),
    ("pq", 32, 8, 8192, IP, 5300, 10, 16, False), ("flat", 96, 0, 1024, L2, 50, 10, 16, False),
    ("flat", 96, 0, 1024, L2, 50, 100, 16, True), ("flat", 96, 0, 1024, IP, 50, 10, 16, True),
    ("sq8", 96, 0, 1024, L2, 100, 10, 16, False), ("sq8", 96, 0, 1024, L2, 330, 10, 16, True),
    ("sq8", 100, 0, 1024, L2, 50, 10, 16, True)])
def test_lists_of_few_queries_are_scanned_query_by_query(vs, kind, d, M, nlist, metric, nq, k, nprobe, matrix):
    """Batches large enough for the matrix-core scan whose queries share their lists with too few others (that scan was
    up to 1.9 times as slow on them)."""
    n = 2_000_000
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn((n, d), generator=g, device="cuda")
    cent = x[:nlist].contiguous()
    if kind == "pq":
        ix = vs.IVFPQ(d, metric, cent, torch.randn((M, 256, d // M), generator=g, device="cuda"), nbits=8)
    elif kind == "flat":
        ix = vs.IVFFlat(d, metric, cent)
    else:
        ix = vs.IVFSQ8(d, metric, cent, torch.full((d,), -5.0, device="cuda"), torch.full((d,), 10.0 / 255, device="cuda"))
    try:
        ix.add(x)
        vs.vs_profile_enable(1)
        vs.vs_profile_read()
        ix.search(x[:nq].contiguous(), k, nprobe)
        torch.cuda.synchronize()
        assert (vs.vs_profile_read()["scan_first"][1] > 0) == matrix
    finally:
        vs.vs_profile_enable(0)
        ix.close()


# every form of VS_MS_PQ_FORMS that test_gpu_mscan does not reach, at the ends of its range of d / M, and the steps of raw
# vectors and scalar codes between those there
@pytest.mark.parametrize("kind,d,M,nbits,metric,form,nq,k,nprobe", [
    ("pq", 40, 8, 8, L2, 1, 333, 10, 9), ("pq", 64, 8, 8, IP, 0, 65, 100, 33), ("pq", 80, 16, 8, L2, 0, 130, 17, 9),
    ("pq", 112, 16, 8, IP, 0, 333, 1, 9), ("pq", 140, 20, 8, IP, 0, 65, 64, 33), ("pq", 120, 20, 8, L2, 1, 130, 10, 9),
    ("pq", 48, 16, 8, L2, 0, 65, 128, 64), ("pq", 64, 16, 8, L2, 1, 333, 33, 9), ("pq", 128, 32, 8, L2, 0, 130, 10, 9),
    ("pq", 128, 32, 8, IP, 0, 65, 65, 33), ("pq", 32, 32, 4, L2, 0, 130, 10, 9), ("pq", 64, 64, 4, IP, 0, 65, 16, 9),
    ("pq", 128, 64, 4, L2, 1, 333, 100, 33), ("pq", 48, 16, 4, L2, 0, 65, 10, 9), ("pq", 64, 16, 4, IP, 0, 130, 1, 64),
    ("pq", 96, 32, 4, L2, 1, 65, 64, 9), ("pq", 128, 32, 4, IP, 0, 333, 10, 9), ("pq", 192, 64, 4, L2, 0, 130, 17, 9),
    ("pq", 256, 64, 4, IP, 0, 65, 128, 33),
    ("flat", 50, 0, 0, IP, 0, 130, 10, 9), ("flat", 96, 0, 0, L2, 0, 65, 100, 33), ("flat", 160, 0, 0, L2, 0, 333, 1, 9),
    ("flat", 217, 0, 0, IP, 0, 65, 65, 9), ("sq8", 20, 0, 0, L2, 0, 130, 10, 9), ("sq8", 128, 0, 0, IP, 0, 65, 128, 33),
    ("sq8", 150, 0, 0, L2, 0, 333, 33, 9), ("sq8", 190, 0, 0, IP, 0, 65, 1, 64), ("sq8", 220, 0, 0, L2, 0, 130, 10, 9)])
def test_every_form(vs, kind, d, M, nbits, metric, form, nq, k, nprobe):
    import test_gpu_mscan
    test_gpu_mscan.test_matrix_scan_equals_query_major(vs, kind, d, M, nbits, metric, form, nq, k, nprobe)
    rng = np.random.default_rng(d)
    cent, x = lists_of(rng, d, [50] * 8)
    ix = make(vs, kind, d, M, nbits, metric, cent, x, rng)
    try:                                                        # that scan is the one that runs
        if form:
            ix.set_search_type(form)
        ix.add(dev(x))
        vs.vs_profile_enable(1)
        vs.vs_profile_read()
        both_scans(vs, ix, dev(x[:nq]), k, 4)
        assert vs.vs_profile_read()["scan_first"][1] == 1
    finally:
        vs.vs_profile_enable(0)
        ix.close()


@pytest.mark.parametrize("kind,d,M", [("pq", 32, 8), ("pq", 100, 20), ("flat", 40, 0), ("sq8", 64, 0)])
def test_more_lists_than_a_workgroup_takes(vs, kind, d, M):
    """The offsets' workgroups take 1024 lists each; most of these are empty or hold a few vectors."""
    rng = np.random.default_rng(d)
    cent, x = lists_of(rng, d, list(rng.integers(0, 4, 2047)) + [70] + list(rng.integers(0, 9, 1500)))
    ix = make(vs, kind, d, M, 8, L2, cent, x, rng)
    try:
        for part in dev(x).split(len(x) // 2 + 1):
            ix.add(part.contiguous())
        q = (x[rng.integers(0, len(x), 500)] + 5 * rng.standard_normal((500, d))).astype(np.float32)
        for k, nprobe in ((10, 64), (100, 200)):
            both_scans(vs, ix, dev(q), k, nprobe)
    finally:
        ix.close()


def test_one_list_holds_nearly_everything(vs):
    """Segments are doubled where there would be more than four million work items."""
    g = torch.Generator(device="cuda").manual_seed(4)
    rng = np.random.default_rng(4)
    d, M = 32, 8
    cent = np.concatenate([np.zeros((1, d)), 6 * rng.standard_normal((30, d))]).astype(np.float32)
    x = torch.cat([torch.randn((300_000, d), generator=g, device="cuda"),
                   dev(np.repeat(cent[1:], 100, axis=0)) + torch.randn((3000, d), generator=g, device="cuda")])
    ix = vs.IVFPQ(d, L2, dev(cent), torch.randn((M, 256, d // M), generator=g, device="cuda"), nbits=8)
    try:
        ix.add(x)
        q = torch.randn((12_000, d), generator=g, device="cuda")
        both_scans(vs, ix, q, 10, 11)
    finally:
        ix.close()


def test_copy_of_the_codes_in_memory_of_its_own(vs):
    """Above 128 MiB the copy lies apart; the index grows into that and on."""
    g = torch.Generator(device="cuda").manual_seed(5)
    d, M = 96, 32
    x = torch.randn((2_200_000, d), generator=g, device="cuda")
    ix = vs.IVFPQ(d, L2, x[:512].contiguous(), torch.randn((M, 256, d // M), generator=g, device="cuda"), nbits=8)
    try:
        q = x[:700] + 0.1
        vs.vs_profile_enable(1)
        for _ in range(3):                                      # 70, 141 and 211 MB
            ix.add(x)
            vs.vs_profile_read()
            both_scans(vs, ix, q, 20, 16)
            assert vs.vs_profile_read()["scan_first"][1] == 1
    finally:
        vs.vs_profile_enable(0)
        ix.close()


@pytest.mark.parametrize("kind,d,M", [("pq", 32, 8), ("flat", 40, 0), ("sq8", 40, 0)])
def test_batches_beyond_a_piece(vs, kind, d, M):
    """More than 65,536 queries are scanned in pieces, the last one shorter; each has room for the candidates of k = 100
    (as one batch each query had 256, and more than a quarter were scanned again)."""
    rng = np.random.default_rng(d)
    nq, k, nprobe = 262_145, 100, 24
    x = rng.standard_normal((24_000, d)).astype(np.float32)
    ix = make(vs, kind, d, M, 8, L2, x[:40], x, rng)
    try:
        ix.add(dev(x))
        g = torch.Generator(device="cuda").manual_seed(6)
        q = torch.randn((nq, d), generator=g, device="cuda")
        both_scans(vs, ix, q, k, nprobe)
        if kind == "pq":
            assert ix.search_stats(q, k, nprobe)[2]["list_major_rescanned"] < nq // 50
            vs.vs_set_option("knn_eps_scale", -1.0)             # (all of every piece are counted)
            assert ix.search_stats(q, k, nprobe)[2]["list_major_rescanned"] == nq
    finally:
        ix.close()
