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
