"""4-bit inner products swept as one-hot rows: which indexes and batches go that way, and sizes at which its kernels can go
wrong.  Every distance and id bit for bit that of the query-major scan."""
import numpy as np
import pytest

from test_gpu_mscan import IP, same

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
    vs.vs_profile_enable(0)
    for name, value in (("matrix_scan", 0), ("list_major_candidates", 1024), ("knn_eps_scale", 1.0)):
        vs.vs_set_option(name, value)


def clusters(seed, d, nlist, n, scale=None, crowded=False):
    """(centroids, vectors around them, a generator): components in the sizes of `scale`, half of the vectors in one
    list if `crowded`."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    cent = torch.randn((nlist, d), generator=g, device="cuda")
    at = torch.randint(0, nlist, (n,), generator=g, device="cuda")
    if crowded:
        at[: n // 2] = 3
    x = cent[at] + 0.4 * torch.randn((n, d), generator=g, device="cuda")
    if scale is not None:
        cent, x = cent * scale, x * scale
    return cent, x, g


def codebooks(cent, x, M):
    """The slices of 16 vectors' residuals."""
    r = x[-16:].double()
    near = torch.cdist(r, cent.double()).argmin(1)
    return (x[-16:] - cent[near]).view(16, M, -1).permute(1, 0, 2).contiguous()


def search(vs, ix, q, k, nprobe):
    """(distances, ids, whether the lists were scanned on the matrix cores)"""
    vs.vs_profile_enable(1)
    vs.vs_profile_read()
    D, I = ix.search(q, k, nprobe)
    torch.cuda.synchronize()
    matrix = vs.vs_profile_read()["scan_first"][1] > 0
    vs.vs_profile_enable(0)
    return D.clone(), I.clone(), matrix


@pytest.mark.parametrize("d,M", [(768, 64), (160, 32), (144, 16)])
@pytest.mark.parametrize("what", ["even", "one sub-quantizer ten times the others", "falling components", "a codeword far out",
                                  "a codeword that is not a number", "an infinite codeword", "crowded lists", "zeros"])
def test_indexes_whose_bounds_tell_little_apart_are_scanned_query_by_query(vs, d, M, what):
    """A batch large enough for the one-hot rows.  Where their common step is too coarse for most sub-quantizers, or most
    vectors lie in a few lists, that scan was up to 3.4 times as slow as the query-major one."""
    scale = torch.ones(d, device="cuda")
    if what.startswith("one sub"):
        scale[3 * (d // M): 4 * (d // M)] = 10
    if what.startswith("falling"):
        scale = (torch.arange(d, device="cuda") + 1.0) ** -0.75
    cent, x, g = clusters(d, d, 256, 150_000, scale, what == "crowded lists")
    cb = codebooks(cent, x, M)
    if what == "a codeword far out":
        cb[5, 2] *= 100
    if "not a number" in what or "infinite" in what:
        cb[0, 1, 0] = float("nan" if "not" in what else "inf")
    if what == "zeros":
        cb[:] = 0
    ix = vs.IVFPQ(d, IP, cent, cb, nbits=4)
    try:
        ix.add(x)
        q = x[torch.randint(0, len(x), (1500,), generator=g, device="cuda")]
        D, I, matrix = search(vs, ix, q, 10, 32)
        assert matrix == (what == "even")
        vs.vs_set_option("matrix_scan", 1)                      # (there it is served all the same)
        D1, I1, matrix = search(vs, ix, q, 10, 32)
        assert matrix and same(D, D1) and same(I, I1)
    finally:
        ix.close()


def both(vs, ix, q, k, nprobe, tell=""):
    """The one-hot scan's results, which are those of the query-major scan."""
    vs.vs_set_option("matrix_scan", -1)
    D0, I0, matrix = search(vs, ix, q, k, nprobe)
    assert not matrix
    vs.vs_set_option("matrix_scan", 1)
    D1, I1, matrix = search(vs, ix, q, k, nprobe)
    assert matrix and same(D0, D1) and same(I0, I1), tell
    return D1, I1


# A wavefront of the tables' kernel takes 2, 4 or 8 queries a pass (64, 32, 16 sub-quantizers), and two to eight passes from
# 4096, 8192 and 16,384 queries on; numbers that leave workgroups, wavefronts and pairs of queries partly empty
@pytest.mark.parametrize("d,M,nq", [(320, 64, 4095), (320, 64, 4097), (768, 64, 8195), (320, 64, 20_011), (160, 32, 8193),
                                    (384, 32, 16_387), (16, 16, 16_385), (144, 16, 32_771), (128, 16, 70_003)])
def test_tables_of_several_passes(vs, d, M, nq):
    cent, x, g = clusters(d + M, d, 24, 3_000)
    ix = vs.IVFPQ(d, IP, cent, codebooks(cent, x, M), nbits=4)
    try:
        ix.add(x)
        q = x[torch.randint(0, len(x), (nq,), generator=g, device="cuda")]
        q = q * (0.5 + torch.rand((nq, 1), generator=g, device="cuda"))
        print("passes", d, M, nq, flush=True)
        both(vs, ix, q, 3, 4)
        assert ix.search_stats(q, 3, 4)[2]["list_major_rescanned"] < nq // 2     # (tables of all queries are right)
    finally:
        ix.close()


# sub-vectors read 16 bytes at a time and one by one, up to the longest that the tables' kernel has the LDS for
@pytest.mark.parametrize("d,M,nq,k,nprobe", [(128, 16, 65, 10, 9), (192, 16, 130, 64, 33), (256, 32, 333, 10, 9),
                                             (384, 32, 17, 100, 64), (512, 64, 130, 1, 9), (2304, 64, 65, 10, 9),
                                             (2496, 64, 17, 10, 33), (2528, 32, 17, 10, 9), (2544, 16, 33, 17, 9)])
def test_lengths_of_sub_vectors(vs, d, M, nq, k, nprobe):
    import test_gpu_mscan
    test_gpu_mscan.test_matrix_scan_equals_query_major(vs, "pq", d, M, 4, IP, 0, nq, k, nprobe)
    cent, x, _ = clusters(d, d, 8, 400)
    ix = vs.IVFPQ(d, IP, cent, codebooks(cent, x, M), nbits=4)
    try:
        ix.add(x)
        both(vs, ix, x[:nq].contiguous(), k, 4)                 # (it is that scan that runs)
    finally:
        ix.close()


@pytest.mark.parametrize("d,M", [(2560, 64), (2560, 32), (2560, 16)])
def test_sub_vectors_without_room_for_their_tables(vs, d, M):
    """... beyond which lists are scanned query by query."""
    cent, x, _ = clusters(d, d, 4, 300)
    ix = vs.IVFPQ(d, IP, cent, codebooks(cent, x, M), nbits=4)
    try:
        ix.add(x)
        vs.vs_set_option("matrix_scan", 1)
        assert not search(vs, ix, x[:50].contiguous(), 5, 2)[2]
    finally:
        ix.close()


@pytest.mark.parametrize("d,M", [(16, 16), (160, 32), (320, 64)])
def test_segments_of_512(vs, d, M):
    """From 32,768 segments on they are 512 codes long."""
    g = torch.Generator(device="cuda").manual_seed(d)
    long = [511, 512, 513, 1023, 1024, 1025, 1537, 2049]
    cent = torch.randn((33_000, d), generator=g, device="cuda")
    cent[: len(long)] *= 3                                      # (the queries' best lists)
    x = torch.cat([cent[l] + 0.4 * torch.randn((n, d), generator=g, device="cuda") for l, n in enumerate(long)] +
                  [cent[len(long):] + 0.1])
    ix = vs.IVFPQ(d, IP, cent, codebooks(cent[:2000], x[:-16], M), nbits=4)
    try:
        ix.set_coarse_metric(0)                                 # (a vector goes to the centroid that it is around)
        ix.add(x)
        assert sorted(ix.list_sizes().tolist())[-4:] > [500] * 4
        q = x[torch.randint(0, sum(long), (5_003,), generator=g, device="cuda")]
        for k in (10, 100):
            both(vs, ix, q, k, 8)
    finally:
        ix.close()


@pytest.mark.parametrize("d,M", [(16, 16), (160, 32)])
def test_pieces_of_a_batch(vs, d, M):
    """More than 65,536 queries are scanned in pieces, whose tables lie in the same place one after the other."""
    cent, x, g = clusters(d, d, 40, 12_000)
    nq, k, nprobe = 131_075, 10, 6
    ix = vs.IVFPQ(d, IP, cent, codebooks(cent, x, M), nbits=4)
    try:
        ix.add(x)
        q = x[torch.randint(0, len(x), (nq,), generator=g, device="cuda")] + 0.1
        both(vs, ix, q, k, nprobe)
        assert ix.search_stats(q, k, nprobe)[2]["list_major_rescanned"] < nq // 4
        vs.vs_set_option("knn_eps_scale", -1.0)                 # (all of every piece are counted)
        assert ix.search_stats(q, k, nprobe)[2]["list_major_rescanned"] == nq
    finally:
        ix.close()


# either side of the lines that vectors visited, probes, pairs per list and list length draw
@pytest.mark.parametrize("d,M,nlist,nq,k,nprobe,matrix", [
    (160, 32, 500, 500, 10, 16, False), (160, 32, 500, 700, 10, 16, True), (160, 32, 500, 1_400, 100, 8, False),
    (160, 32, 500, 2_700, 100, 8, True), (160, 32, 4_000, 5_400, 10, 16, False), (160, 32, 4_000, 11_000, 10, 16, True),
    (16, 16, 500, 700, 10, 16, True), (16, 16, 500, 500, 10, 16, False), (768, 64, 250, 360, 10, 16, True),
    (768, 64, 250, 300, 10, 16, False)])
def test_batches_on_either_side_of_the_lines(vs, d, M, nlist, nq, k, nprobe, matrix):
    cent, x, g = clusters(d + nlist, d, nlist, 500_000)
    ix = vs.IVFPQ(d, IP, cent, codebooks(cent, x, M), nbits=4)
    try:
        ix.add(x)
        q = x[torch.randint(0, len(x), (nq,), generator=g, device="cuda")]
        D, I, was = search(vs, ix, q, k, nprobe)
        assert was == matrix
        vs.vs_set_option("matrix_scan", -1 if matrix else 1)
        D1, I1, _ = search(vs, ix, q, k, nprobe)
        assert same(D, D1) and same(I, I1)
    finally:
        ix.close()
