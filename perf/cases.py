"""The work that users of this library have it do, as cases to time.

A case is one call (or the two calls of a two-stage search) through the public entry points of
paper_2401_08281_amd, on data shaped like the repository's workloads: integer descriptors from a
mixture of Gaussians ("sift"), unit-norm embeddings from such a mixture ("unit"), plain Gaussians
("gauss").  Coarse centroids are database rows, sub-codebooks are residual slices of database rows,
as in the benchmark.  Everything is drawn on the device from the seed.

Paths:
  ivfpq    batched IVF-PQ search of an index that the program keeps (L2 or inner product, 8- or
           4-bit codes, the three ways to evaluate distances), optionally followed by the exact
           re-ranking of its results (refine > 0)
  flat     exact search of a flat index that the program keeps
  flat_once  exact search of rows handed over with the call (nothing kept)
  ivfflat, ivfsq8   the inverted files with raw vectors and with 8-bit scalar codes
  build    create an IVF-PQ index, add all vectors, read codes and assignments back
  train    centroids and codebooks from training vectors
"""
import math

import torch

import paper_2401_08281_amd as vs

L2, IP = 0, 1
MAX_BYTES = 100_000_000 * 96 * 4       # the largest database of the repository's configurations
MAX_PAIRS = 10_000 * 64 * 1526         # (query, code) pairs of its largest search


def listed():
    return [
        # one query of an online service on a million descriptors: launches and latency
        dict(name="ivfpq_one_query", path="ivfpq", data="sift", nb=1_000_000, d=128, nlist=4096, M=16, nbits=8,
             metric=L2, form=0, nq=1, k=10, nprobe=16, refine=0),
        # the ordinary batch on the same index, default evaluation (a table per query and list)
        dict(name="ivfpq_sift", path="ivfpq", data="sift", nb=1_000_000, d=128, nlist=4096, M=16, nbits=8,
             metric=L2, form=0, nq=10_000, k=10, nprobe=16, refine=0),
        # the same index with stored norms (one table per query), many probes for recall
        dict(name="ivfpq_sift_norms", path="ivfpq", data="sift", nb=1_000_000, d=128, nlist=4096, M=16, nbits=8,
             metric=L2, form=1, nq=10_000, k=10, nprobe=64, refine=0),
        # the largest workload of the benchmark: 3.2 GB of codes
        dict(name="ivfpq_deep_100m", path="ivfpq", data="unit", nb=100_000_000, d=96, nlist=65536, M=32, nbits=8,
             metric=L2, form=0, nq=10_000, k=100, nprobe=64, refine=0),
        # text embeddings, inner product, 4-bit codes
        dict(name="ivfpq_embed_ip4", path="ivfpq", data="unit", nb=10_000_000, d=768, nlist=16384, M=64, nbits=4,
             metric=IP, form=0, nq=10_000, k=10, nprobe=32, refine=0),
        # a ragged middling batch in two stages: 100 results of the compressed search, 10 kept exactly
        dict(name="ivfpq_refine", path="ivfpq", data="unit", nb=1_000_003, d=96, nlist=2000, M=32, nbits=8,
             metric=L2, form=0, nq=333, k=100, nprobe=24, refine=10),
        # exact search of a kept index, ground truth for a million descriptors
        dict(name="flat_sift", path="flat", data="sift", nb=1_000_000, d=128, metric=L2, nq=10_000, k=100),
        # exact search without an index, a dimension that fits no tile, inner product
        dict(name="flat_ragged", path="flat_once", data="gauss", nb=200_003, d=100, metric=IP, nq=1_000, k=10),
        # inverted file with the vectors as they are
        dict(name="ivfflat_sift", path="ivfflat", data="sift", nb=1_000_000, d=128, nlist=4096, metric=L2,
             nq=10_000, k=10, nprobe=16),
        # inverted file with scalar codes, inner product
        dict(name="ivfsq8_unit", path="ivfsq8", data="unit", nb=4_000_000, d=96, nlist=8192, metric=IP,
             nq=4_096, k=100, nprobe=32),
        # index construction: assignment, encoding, placement
        dict(name="build_sift", path="build", data="sift", nb=1_000_000, d=128, nlist=4096, M=16, nbits=8, metric=L2),
        # training: the coarse k-means and one k-means per sub-quantizer
        dict(name="train_sift", path="train", data="sift", nb=262_144, d=128, nlist=1024, M=16, nbits=8, metric=L2,
             niter=10),
    ]


def _spread(rng, lo, hi):
    """An integer from lo to hi, even over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (d, M, nbits, data): the shapes of the configurations, and two generic ones without a kernel of their own
PQ_SHAPES = ((32, 8, 8, "gauss"), (128, 16, 8, "sift"), (96, 32, 8, "unit"), (768, 64, 4, "unit"),
             (100, 20, 8, "unit"), (64, 32, 4, "gauss"))


def _index_sizes(rng, d, hi):
    nb = _spread(rng, 10_000, min(hi, MAX_BYTES // (4 * d)))
    nlist = max(16, min(65536, int(math.sqrt(nb) * math.exp(rng.uniform(0.0, math.log(8.0))))))
    return nb, nlist


def _search_sizes(rng, nb, nlist, hi_q=10_000):
    nprobe = min(_spread(rng, 1, 64), nlist)
    nq = _spread(rng, 1, hi_q)
    while nq > 1 and nq * nprobe * (nb / nlist) > MAX_PAIRS:
        nq = (nq + 1) // 2
    return nq, _spread(rng, 1, 100), nprobe


def draw(rng):
    path = rng.choice(("ivfpq", "ivfpq", "ivfpq", "ivfpq", "ivfpq", "ivfpq", "flat", "flat_once", "ivfflat", "ivfsq8",
                       "build", "train"))
    if path == "ivfpq":
        d, M, nbits, data = rng.choice(PQ_SHAPES)
        nb, nlist = _index_sizes(rng, d, 20_000_000)
        nq, k, nprobe = _search_sizes(rng, nb, nlist)
        metric = IP if nbits == 4 and d == 768 else rng.choice((L2, L2, L2, IP))
        own_kernel = nbits == 8 and d != 100
        form = rng.choice((0, 0, 1, 2) if own_kernel else (0, 0, 1)) if metric == L2 else 0
        if form == 2 and nlist * M > 300_000:      # the tables of all lists would not be kept
            form = 0
        refine = 0
        if k >= 20 and nb * d <= 200_000_000 and rng.random() < 0.5:
            refine = k // 5
        return dict(path=path, data=data, nb=nb, d=d, nlist=nlist, M=M, nbits=nbits, metric=metric, form=form, nq=nq,
                    k=k, nprobe=nprobe, refine=refine)
    if path in ("flat", "flat_once"):
        d = rng.choice((32, 96, 128, 256, 768, rng.randint(17, 300)))
        nb = _spread(rng, 1_000, 1_000_000)
        nq = _spread(rng, 1, 10_000)
        most = 1_000_000 * 10_000 * 128 if d % 32 == 0 else 200_000 * 1_000 * 128
        while nq > 1 and nb * nq * d > most:
            nq = (nq + 1) // 2
        return dict(path=path, data=rng.choice(("sift", "unit", "gauss")), nb=nb, d=d, metric=rng.choice((L2, IP)),
                    nq=nq, k=_spread(rng, 1, 100))
    if path in ("ivfflat", "ivfsq8"):
        d = rng.choice((32, 96, 128, rng.randint(17, 200)))
        nb, nlist = _index_sizes(rng, d, 4_000_000)
        nq, k, nprobe = _search_sizes(rng, nb, nlist)
        while nq > 1 and nq * nprobe * (nb / nlist) * d > 10_000 * 16 * 250 * 128 * 4:
            nq = (nq + 1) // 2
        return dict(path=path, data=rng.choice(("sift", "unit")), nb=nb, d=d, nlist=nlist, metric=rng.choice((L2, IP)),
                    nq=nq, k=k, nprobe=nprobe)
    d, M, nbits, data = rng.choice(PQ_SHAPES)
    if path == "build":
        nb = _spread(rng, 10_000, 1_000_000 if d <= 128 else 200_000)
        nlist = max(16, min(8192, int(math.sqrt(nb) * math.exp(rng.uniform(0.0, math.log(8.0))))))
        return dict(path=path, data=data, nb=nb, d=d, nlist=nlist, M=M, nbits=nbits, metric=rng.choice((L2, IP)))
    nb = _spread(rng, 10_000, 262_144 if d <= 128 else 60_000)
    return dict(path=path, data=data, nb=nb, d=d, nlist=_spread(rng, 16, 1024), M=M, nbits=nbits, metric=L2,
                niter=rng.randint(4, 10))


# ---- inputs ---------------------------------------------------------------------------------


class _Source:
    """Database rows and queries of one seed, drawn on the device in pieces."""

    def __init__(self, case, seed):
        self.kind, self.d = case["data"], case["d"]
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        ncomp = {"sift": 1000, "unit": 10_000 if self.d <= 128 else 5_000, "gauss": 1}[self.kind]
        if self.kind == "sift":
            self.centres = torch.rand((ncomp, self.d), generator=self.g, device="cuda") * 255.0
        else:
            self.centres = torch.randn((ncomp, self.d), generator=self.g, device="cuda")

    def rows(self, n):
        v = torch.randn((n, self.d), generator=self.g, device="cuda")
        if self.kind == "gauss":
            return v
        comp = torch.randint(0, self.centres.shape[0], (n,), generator=self.g, device="cuda")
        v *= 20.0 if self.kind == "sift" else 0.3
        v += self.centres[comp]
        if self.kind == "sift":
            return v.clamp_(0.0, 255.0).round_()
        v /= v.norm(dim=1, keepdim=True)
        return v

    def pieces(self, nb):
        step = max(1, min(10_000_000, (4 << 30) // (4 * self.d)))
        for s in range(0, nb, step):
            yield self.rows(min(step, nb - s))

    def pick(self, x, n):
        """n rows of x; all different as long as x has that many."""
        if n > x.shape[0]:
            at = torch.arange(n, device="cuda") % x.shape[0]
        else:
            at = torch.randperm(x.shape[0], generator=self.g, device="cuda")[:n]
        return x[at].contiguous()

    def queries(self, x, n):
        """New rows of the same mixture; for wide embeddings perturbed database rows."""
        if self.d < 512 or self.kind != "unit":
            return self.rows(n)
        v = x[torch.randint(0, x.shape[0], (n,), generator=self.g, device="cuda")]
        v = v + 0.05 * torch.randn((n, self.d), generator=self.g, device="cuda")
        return v / v.norm(dim=1, keepdim=True)

    def codebooks(self, x, cent, M, nbits):
        """Sub-codebook m: the m-th slices of the residuals of 2^nbits rows to their closest centroids."""
        K = 1 << nbits
        rows = self.pick(x, K).double()
        c = cent.double()
        near = ((c * c).sum(1)[None, :] - 2.0 * (rows @ c.T)).argmin(1)
        res = (rows - c[near]).float()
        return res.view(K, M, self.d // M).permute(1, 0, 2).contiguous()


def prepare(case, seed):
    src = _Source(case, seed)
    path, nb, d = case["path"], case["nb"], case["d"]
    st = {"case": case}
    if path in ("flat", "flat_once"):
        x = src.rows(nb)
        st["q"] = src.rows(case["nq"])
        if path == "flat":
            st["ix"] = vs.Flat(d, case["metric"])
            st["ix"].add(x)
        else:
            st["x"] = x
        return st
    if path in ("build", "train"):
        x = src.rows(nb)
        st["x"], st["cent"] = x, src.pick(x, case["nlist"])
        st["cb"] = src.codebooks(x, st["cent"], case["M"], case["nbits"])
        return st
    for i, x in enumerate(src.pieces(nb)):
        if i == 0:
            cent = src.pick(x, case["nlist"])
            if path == "ivfpq":
                ix = vs.IVFPQ(d, case["metric"], cent, src.codebooks(x, cent, case["M"], case["nbits"]), case["nbits"])
                if case["form"]:
                    ix.set_search_type(case["form"])
            elif path == "ivfflat":
                ix = vs.IVFFlat(d, case["metric"], cent)
            else:
                lo, hi = x.amin(0), x.amax(0)
                ix = vs.IVFSQ8(d, case["metric"], cent, lo, ((hi - lo) / 256.0).clamp_min(1e-6))
            st["q"] = src.queries(x, case["nq"])
        ix.add(x)
    if case.get("refine"):
        st["x"] = x
    st["ix"] = ix
    return st


# ---- one pass -------------------------------------------------------------------------------


def run(state):
    case, path = state["case"], state["case"]["path"]
    if path == "ivfpq":
        D, I = state["ix"].search(state["q"], case["k"], case["nprobe"])
        if case["refine"]:
            return (D, I) + tuple(vs.vs_refine(state["x"], state["q"], I, case["refine"], case["metric"]))
        return D, I
    if path in ("ivfflat", "ivfsq8"):
        return state["ix"].search(state["q"], case["k"], case["nprobe"])
    if path == "flat":
        return state["ix"].search(state["q"], case["k"])
    if path == "flat_once":
        return vs.vs_flat_search(state["x"], state["q"], case["k"], case["metric"])
    if path == "build":
        ix = vs.IVFPQ(case["d"], case["metric"], state["cent"], state["cb"], case["nbits"])
        ix.add(state["x"])
        ids, lists = ix.assignments()
        codes = ix.codes()
        ix.close()
        return ids, lists, codes
    cent, cb = state["cent"].clone(), state["cb"].clone()
    objective = vs.vs_ivfpq_train(state["x"], case["metric"], cent, cb, case["nbits"], case["niter"])
    return cent, cb, torch.tensor(objective, dtype=torch.float64)


# ---- what a pass cannot do without ----------------------------------------------------------


def work(case):
    path, nb, d = case["path"], case["nb"], case["d"]
    if path in ("flat", "flat_once"):
        nq, k = case["nq"], case["k"]
        return {"bytes": 4.0 * d * (nb + nq) + 12.0 * nq * k, "flops": 2.0 * nb * nq * d}
    nlist = case["nlist"]
    if path in ("build", "train"):
        M, K = case["M"], 1 << case["nbits"]
        nearest = 2.0 * nb * d * (nlist + K)              # nearest centroid, then nearest codewords
        params = 4.0 * d * (nlist + K)
        if path == "build":
            return {"bytes": 4.0 * nb * d + params + nb * (12.0 + M * case["nbits"] / 8.0), "flops": nearest}
        return {"bytes": 4.0 * nb * d + 2.0 * params, "flops": nearest * case["niter"]}
    nq, k, nprobe = case["nq"], case["k"], case["nprobe"]
    visited = nq * nprobe * (nb / nlist)                  # (query, code) pairs
    read = nb * min(1.0, nq * nprobe / nlist)             # codes of the probed lists, each read once
    size = {"ivfpq": case.get("M", 0) * case.get("nbits", 0) / 8.0 + (4.0 if case.get("form") == 1 else 0.0),
            "ivfflat": 4.0 * d, "ivfsq8": 1.0 * d}[path]
    each = case["M"] if path == "ivfpq" else 2.0 * d      # a table entry added per sub-code; a distance
    bytes_ = read * size + 4.0 * d * (nlist + nq) + 12.0 * nq * k
    flops = 2.0 * nq * nlist * d + visited * each
    if case.get("refine"):
        bytes_ += 4.0 * d * nq * k + 12.0 * nq * case["refine"]
        flops += 2.0 * nq * k * d
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["path"] == "build":
        return "exact"                                    # ids, lists and codes are whole numbers
    # 32-bit sums; an id may differ where two distances agree to within their rounding
    return {"rel": 1e-5, "max": 4e-4, "differ": 2e-3}
