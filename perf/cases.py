"""The work that users of this library have it do, as measurable cases.

A case is either a search over a built index (one query of a live service, a
handful of queries of one request, a query set in one call; with the options
that are used in earnest: bit widths, tenant allowlists, an id-map index with
deleted vectors, TQ+ calibration, large k) or an encode (the rows of one
document as they arrive, and a bulk build).

Corpora are clustered, power-law embeddings as in synth/ (1,000 clusters,
covariance eigenvalues ~ i^-0.8, L2-normalised rows), drawn on the GPU from
the seed; queries are held-out rows of the same mixture.
"""
import functools
import math

import torch

import paper_2607_16973_amd as tq

SEED = 42          # of the rotation: one matrix for all indexes of a program
CLUSTERS = 1000
CHUNK = 65536      # rows generated (and added) at a time


def _search(name, n, nq, k, d=1536, bits=4, tenants=1, filt="none", kind="flat", path="auto"):
    """tenants: T, Zipf(1.1) over random positions; filt: none, one (one
    tenant per query) or tenth (ceil(T/10) tenants per query); kind: flat,
    idmap (uint64 ids, 5% deleted) or plus (TQ+ calibrated)."""
    case = {"op": "search", "d": d, "bits": bits, "n": n, "nq": nq, "k": k, "tenants": tenants,
            "filter": filt, "kind": kind, "path": path}
    return dict(case, name=name) if name else case


def _encode(name, n, d=1536, bits=4):
    case = {"op": "encode", "d": d, "bits": bits, "n": n}
    return dict(case, name=name) if name else case


def listed():
    return [
        # one query of a live service over a small collection: latency only
        _search("one_query_10k", 10_000, 1, 10),
        # one query over the headline corpus: one stream of the whole code store
        _search("one_query_1m", 1_000_000, 1, 10),
        # the sub-queries of one request (query expansion, multi-vector), k = 5 as for RAG prompts
        _search("eight_queries_100k", 100_000, 8, 5),
        # an offline evaluation: the 1,000 held-out queries in one default call
        _search("query_set_999k", 999_000, 1000, 10),
        # a server that gathers requests and asks for the matrix-core path
        _search("gathered_256_1m", 1_000_000, 256, 10, path="mfma"),
        # tenants of a shared index, each query restricted to its own
        _search("own_tenant_1m", 1_000_000, 64, 10, tenants=100, filt="one"),
        # the compact store (2 bits), a request batch
        _search("two_bit_500k", 500_009, 32, 10, bits=2),
        # the precise store (8 bits), a request batch
        _search("eight_bit_250k", 250_000, 16, 10, bits=8),
        # candidates for a reranker: deep lists for a few queries
        _search("deep_list_200k", 200_000, 4, 1000),
        # a live collection with deletions, shorter embeddings
        _search("deletions_120k", 120_037, 24, 10, d=768, kind="idmap"),
        # the chunks of one document, encoded as they arrive
        _encode("encode_document", 257),
        # a bulk build
        _encode("encode_bulk", 100_000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.25:
        d = rng.choice([256, 768, 1024, 1536, 1536])
        return _encode(None, _log_int(rng, 64, 100_000), d, rng.choice([2, 3, 4, 4, 8]))
    d = rng.choice([256, 768, 1024, 1536, 1536, 1536])
    bits = rng.choice([2, 3, 4, 4, 4, 8])
    n = _log_int(rng, 10_000, 999_999)
    # at most the query set's codes read per query and coordinate
    nq = _log_int(rng, 1, max(2, min(1000, int(1000 * 999_000 * 1536 * 4 / (n * d * bits)) // 4)))
    k = rng.choice([1, 5, 10, 10, 20, 100])
    kind = rng.choice(["flat", "flat", "flat", "idmap", "plus"])
    tenants = rng.choice([1, 1, 1, 10, 100, 1000])
    filt = rng.choice(["one", "tenth"]) if tenants > 1 else "none"
    path = "auto"
    if kind == "flat" and bits == 4 and nq > 16 and rng.random() < 0.3:
        path = "mfma"
    return _search(None, n, nq, k, d, bits, tenants, filt, kind, path)


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=None)
def _codebook(d, bits):
    return tq.Codebook(d, bits)


@functools.lru_cache(maxsize=None)
def _rotation(d):
    return tq.Rotation(d, SEED)


class _Mixture:
    """Rows of the power-law mixture, in chunks, from one seed."""

    def __init__(self, d, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        lam = torch.arange(1, d + 1, dtype=torch.float64, device="cuda") ** -0.8
        self.sq = (lam * (d / lam.sum())).sqrt().float()
        self.d = d
        self.centres = torch.randn(CLUSTERS, d, generator=self.g, device="cuda") * self.sq

    def rows(self, n):
        z = torch.randint(CLUSTERS, (n,), generator=self.g, device="cuda")
        x = torch.randn(n, self.d, generator=self.g, device="cuda")
        x.mul_(self.sq * 0.3).add_(self.centres[z])
        return x.div_(x.norm(dim=1, keepdim=True))

    def chunks(self, n):
        for i in range(0, n, CHUNK):
            yield i, self.rows(min(CHUNK, n - i))


def _zipf(T):
    w = torch.arange(1, T + 1, dtype=torch.float64) ** -1.1
    return w / w.sum()


def _allowed(case, g):
    """[nq, T] bool: the tenants that each query may see."""
    T, nq = case["tenants"], case["nq"]
    m = 1 if case["filter"] == "one" else (T + 9) // 10
    pick = torch.rand(nq, T, generator=g, device="cuda").topk(m, dim=1).indices
    return torch.zeros(nq, T, dtype=torch.bool, device="cuda").scatter_(1, pick, True)


def _bitmap(allowed):
    nq, T = allowed.shape
    words = (T + 63) // 64
    b = torch.zeros(nq, words * 64, dtype=torch.int64, device="cuda")
    b[:, :T] = allowed
    sh = torch.arange(64, device="cuda")
    return (b.view(nq, words, 64) << sh).sum(dim=2).contiguous()   # distinct bits: the sum is their OR


def _inputs(case, seed, rows):
    """Feeds the corpus to rows(first slot, X, tenants) and returns what a
    search takes besides the index."""
    mix = _Mixture(case["d"], seed)
    Q = mix.rows(case["nq"])
    cdf = _zipf(case["tenants"]).cumsum(0).float().cuda()
    for i, X in mix.chunks(case["n"]):
        u = torch.rand(X.shape[0], generator=mix.g, device="cuda")
        t = torch.searchsorted(cdf, u).clamp_(max=case["tenants"] - 1).to(torch.int16)
        rows(i, X, t)
    allowed = _allowed(case, mix.g) if case["filter"] != "none" else None
    dead = torch.rand(case["n"], generator=mix.g, device="cuda") < 0.05 if case["kind"] == "idmap" else None
    return Q, allowed, dead


FIRST_ID = 7_000_000_000   # external ids of the id-map index
FIT_ROWS = 10_000          # rows that TQ+ is fitted to


def prepare(case, seed):
    cb, rot = _codebook(case["d"], case["bits"]), _rotation(case["d"])
    if case["op"] == "encode":
        X = torch.empty(case["n"], case["d"], device="cuda")
        for i, x in _Mixture(case["d"], seed).chunks(case["n"]):
            X[i:i + x.shape[0]] = x
        return {"op": "encode", "cb": cb, "rot": rot, "X": X}
    idx = (tq.IdMapIndex if case["kind"] == "idmap" else tq.Index)(cb, rot, case["tenants"])
    idx.reserve(case["n"])

    def rows(i, X, t):
        if case["kind"] == "plus" and i == 0:
            idx.calibrate(X[:FIT_ROWS])
        if case["kind"] == "idmap":
            idx.add(X, range(FIRST_ID + i, FIRST_ID + i + X.shape[0]), t)
        else:
            idx.add(X, t)

    Q, allowed, dead = _inputs(case, seed, rows)
    if dead is not None:
        idx.remove(dead.nonzero().flatten().cpu().numpy() + FIRST_ID)
    return {"op": "search", "idx": idx, "Q": Q, "k": case["k"], "path": case["path"],
            "allow": None if allowed is None else _bitmap(allowed)}


def run(s):
    if s["op"] == "encode":
        return tq.rotate_quantize(s["cb"], s["rot"], s["X"])
    return s["idx"].search(s["Q"], s["k"], allow=s["allow"], path=s["path"])


# -------------------------------------------------------- work, tolerances
def work(case):
    d, n = case["d"], case["n"]
    row = d * case["bits"] / 8 + 4     # codes and scale of a vector
    if case["op"] == "encode":
        return {"bytes": n * (4 * d + row) + 4 * d * d, "flops": 2 * n * d * d}
    nq, k = case["nq"], case["k"]
    seen, scored, extra = n, n * nq, 0
    if case["filter"] != "none":       # vectors that some query may see, and (query, vector) pairs allowed
        T = case["tenants"]
        share = (1 if case["filter"] == "one" else (T + 9) // 10) / T
        seen = n * (1 - (1 - share) ** nq)
        scored, extra = n * nq * share, 2 * n
    if case["kind"] == "idmap":
        seen, scored, extra = seen * 0.95, scored * 0.95, extra + n / 8
    return {"bytes": seen * row + extra + 4 * nq * d + 4 * d * d + 12 * nq * k,
            "flops": 2 * nq * d * d + 2 * scored * d}


def tolerance(case):
    if case["op"] == "encode":
        # codes are whole numbers with one right value; scales are float64 results stored in float32
        return {"rel": 1e-7, "max": 5e-7, "differ": 0.0}
    # scores are sums of d products from float32 rotated queries, by fixed-point or float32 tables: 4e-8 to
    # 1.8e-7 off float64; neighbours of a list may change places where their scores agree to rounding
    return {"rel": 8e-7, "max": 4e-6, "differ": 0.002}


# ------------------------------------------------------------- 64 bits
def _encode64(X, R, bounds, cents, mu=None, kappa=None):
    """(codes, float64 reconstructions, float64 scales) of float64 rows."""
    y = X @ R.T
    nx = X.square().sum(dim=1).sqrt()
    if mu is None:
        codes = torch.searchsorted(bounds, y / nx[:, None], right=True)
        rec = cents[codes]
    else:
        codes = torch.searchsorted(bounds, (y / nx[:, None] - mu) / kappa, right=True)
        rec = mu + kappa * cents[codes]
    return codes, rec, nx / rec.square().sum(dim=1).sqrt()


def _pack(codes, bits):
    n, d = codes.shape
    b = (codes[:, :, None] >> torch.arange(bits, device="cuda")) & 1
    b = b.view(n, d * bits // 8, 8) << torch.arange(8, device="cuda")
    return b.sum(dim=2).to(torch.uint8)


def exact(case, seed):
    """The quantiser's parameters (rotation matrix, codebook tables) are given;
    everything else is computed here in float64."""
    d, bits = case["d"], case["bits"]
    cb = _codebook(d, bits)
    R = torch.from_numpy(_rotation(d).matrix()).cuda().double()
    bounds, cents = torch.from_numpy(cb.bounds).cuda(), torch.from_numpy(cb.cents).cuda()
    STEP = 8192
    if case["op"] == "encode":
        codes, scales = [], []
        for _, X in _Mixture(d, seed).chunks(case["n"]):
            for x in X.split(STEP):
                c, _, s = _encode64(x.double(), R, bounds, cents)
                codes.append(_pack(c, bits))
                scales.append(s)
        return torch.cat(codes), torch.cat(scales)
    # the queries come first in the mixture's stream: the scores need them while the corpus passes by
    Qr = _Mixture(d, seed).rows(case["nq"]).double() @ R.T
    scores, tenants, fit = [], [], []

    def rows(i, X, t):
        if case["kind"] == "plus" and i == 0:
            x = X[:FIT_ROWS].double()
            y = (x @ R.T) / x.square().sum(dim=1, keepdim=True).sqrt()
            fit.append(y.mean(dim=0).float().double())
            fit.append((y.std(dim=0, correction=0) * math.sqrt(d)).float().double())
        for x in X.split(STEP):
            _, rec, s = _encode64(x.double(), R, bounds, cents, *fit)
            scores.append((Qr @ rec.T) * s)
        tenants.append(t)

    _, allowed, dead = _inputs(case, seed, rows)
    all_scores = torch.cat(scores, dim=1)
    del scores[:]
    t = torch.cat(tenants).long()
    ids, best = [], []
    for q in range(case["nq"]):
        s = all_scores[q]
        if allowed is not None:
            s.masked_fill_(~allowed[q][t], -math.inf)
        if dead is not None:
            s.masked_fill_(dead, -math.inf)
        v, i = torch.topk(s, case["k"])
        i = torch.where(v > -math.inf, i + (FIRST_ID if case["kind"] == "idmap" else 0), -1)
        ids.append(i)
        best.append(v)
    return torch.stack(ids), torch.stack(best)
