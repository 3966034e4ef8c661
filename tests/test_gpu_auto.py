"""The default search path: whichever of the single-query scan and the batched
path it takes, ids and scores are the scan's, bit for bit -- over sizes on
both sides of the rule that chooses, with queries whose certificate fails
(the scan answers them within the call), inside a captured graph, and with a
workspace that only the scan fits."""
import numpy as np
import pytest

import synth
from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

import paper_2607_16973_amd as tq  # noqa: E402

_rot = {}


def rotation(d):
    if d not in _rot:
        _rot[d] = tq.Rotation(d, 42)
    return _rot[d]


def corpus(n, d, seed):
    return torch.from_numpy(synth.isotropic_mixture(n, d, seed=seed)).cuda()


def queries(X, nq, seed):
    return torch.from_numpy(synth.isotropic_queries(X.cpu().numpy(), nq, seed=seed)).cuda()


def same(a, b):
    assert torch.equal(a[0], b[0])
    assert torch.equal(a[1], b[1])


@pytest.mark.parametrize("n,nq,k", [(70, 40, 10), (1037, 7, 5), (1037, 33, 100), (20_011, 2, 10), (20_011, 64, 1),
                                    (20_011, 130, 10), (20_011, 300, 256)])
def test_default_equals_scan(n, nq, k):
    d = 256
    X = corpus(n, d, 5)
    idx = tq.Index(tq.Codebook(d, 4), rotation(d))
    idx.add(X)
    Q = queries(X, min(nq, n), 6)
    same(idx.search(Q, k), idx.search(Q, k, path="lut"))


# every width of the batched kernels' feeds: rings of 4 and of 8 chunks, 64
# and 32 table replicas (d = 2048), the shortest vectors, ragged n and tiles
@pytest.mark.parametrize("d,bits,n,nq,k", [
    (256, 2, 20_011, 33, 10), (768, 2, 20_011, 12, 10), (1536, 2, 9_001, 40, 100),
    (128, 3, 20_011, 33, 10), (768, 3, 9_001, 70, 20), (2048, 3, 9_001, 20, 10),
    (128, 4, 20_011, 33, 10), (384, 4, 20_011, 40, 10), (2048, 4, 9_001, 20, 10),
    (64, 8, 20_011, 33, 10), (768, 8, 9_001, 70, 100), (2048, 8, 5_001, 20, 256)])
@pytest.mark.parametrize("plus", [False, True])
def test_widths(d, bits, n, nq, k, plus):
    X = corpus(n, d, 30)
    idx = tq.Index(tq.Codebook(d, bits), rotation(d))
    if plus:
        idx.calibrate(X[:2000])
    idx.add(X)
    Q = queries(X, nq, 31)
    assert idx.workspace_bytes(nq, k) > idx.workspace_bytes(nq, k, path="lut")   # the batched path's
    same(idx.search(Q, k), idx.search(Q, k, path="lut"))


# filtered: tenants allowed per query (0: none for some queries), few and many
# tenants, tiles and wide passes, with and without deletions; the device gate
# leaves the most selective passes to the scan
@pytest.mark.parametrize("bits,d", [(4, 256), (2, 256), (3, 128), (8, 128)])
@pytest.mark.parametrize("T,allowed,nq,k", [(5, 1, 33, 10), (100, 1, 40, 10), (100, 10, 130, 100), (100, 0, 20, 10),
                                            (1000, 1, 150, 10), (4096, 400, 70, 20), (3000, 1, 10, 10)])
@pytest.mark.parametrize("deleted", [False, True])
def test_filtered(bits, d, T, allowed, nq, k, deleted):
    n = 20_011
    X = corpus(n, d, 40)
    g = torch.Generator(device="cuda").manual_seed(41)
    # a third of the rows belongs to one tenant, the others are spread
    ten = torch.where(torch.rand(n, generator=g, device="cuda") < 0.3, 0,
                      torch.randint(T, (n,), generator=g, device="cuda")).to(torch.int16)
    cls = tq.IdMapIndex if deleted else tq.Index
    idx = cls(tq.Codebook(d, bits), rotation(d), T)
    if deleted:
        idx.add(X, range(10 ** 12, 10 ** 12 + n), ten)
        idx.remove([10 ** 12 + i for i in range(0, n, 3)])
        idx.remove(range(10 ** 12 + 640, 10 ** 12 + 1100))   # whole blocks
    else:
        idx.add(X, ten)
    words = (T + 63) // 64
    allow = torch.zeros(nq, words * 64, dtype=torch.bool, device="cuda")
    for q in range(nq):
        if allowed or q % 3:
            allow[q, torch.randint(T, (max(allowed, 1),), generator=g, device="cuda")] = True
    bits64 = (allow.view(nq, words, 64).long() << torch.arange(64, device="cuda")).sum(dim=2).contiguous()
    Q = queries(X, nq, 42)
    for al in (bits64, None):
        same(idx.search(Q, k, allow=al), idx.search(Q, k, allow=al, path="lut"))


@pytest.mark.parametrize("nq", [12, 40, 100])
def test_queries_without_certificate(nq):
    # every score ties: no candidate set can be proven, every query goes to the scan
    d = 256
    X = corpus(1, d, 7).repeat(6000, 1)
    idx = tq.Index(tq.Codebook(d, 4), rotation(d))
    idx.add(X)
    Q = queries(corpus(200, d, 8), nq, 9)
    idx.search(Q, 10, path="mfma")
    assert tq.last_search_fallbacks() == nq
    ids, scores = idx.search(Q, 10)
    same((ids, scores), idx.search(Q, 10, path="lut"))
    assert torch.equal(ids, torch.arange(10, device="cuda").expand(nq, 10))


def test_some_queries_without_certificate():
    # copies of one row tie for the queries near it; the other queries are proven
    d = 256
    X = corpus(8000, d, 10)
    X[1000:5000] = X[0]
    idx = tq.Index(tq.Codebook(d, 4), rotation(d))
    idx.add(X)
    Q = torch.cat([queries(X[6000:], 30, 11), X[:1].repeat(3, 1), queries(X[6000:], 30, 12)])
    idx.search(Q, 10, path="mfma")
    assert 3 <= tq.last_search_fallbacks() < 63
    same(idx.search(Q, 10), idx.search(Q, 10, path="lut"))


def test_captured():
    d, k = 256, 10
    X = corpus(20_011, d, 13)
    idx = tq.Index(tq.Codebook(d, 4), rotation(d))
    idx.add(X)
    Q = queries(X, 40, 14)
    ws = torch.empty(idx.workspace_bytes(40, k), dtype=torch.uint8, device="cuda")
    ids = torch.empty(40, k, dtype=torch.int64, device="cuda")
    scores = torch.empty(40, k, device="cuda")
    idx.search(Q, k, ids=ids, scores=scores, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        idx.search(Q, k, ids=ids, scores=scores, workspace=ws)
    for seed in (15, 16, 17):
        Q.copy_(queries(X, 40, seed))
        want = idx.search(Q, k, path="lut")
        ids.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        same((ids, scores), want)


def test_scan_workspace_is_enough():
    d, k = 256, 10
    X = corpus(20_011, d, 18)
    idx = tq.Index(tq.Codebook(d, 4), rotation(d))
    idx.add(X)
    Q = queries(X, 40, 19)
    small = idx.workspace_bytes(40, k, path="lut")
    assert small < idx.workspace_bytes(40, k)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    same(idx.search(Q, k, workspace=ws), idx.search(Q, k, path="lut"))
    with pytest.raises(tq.TQError):
        idx.search(Q, k, workspace=ws[:small // 2 // 256 * 256])


@pytest.mark.parametrize("kind,k,nq", [("flat", 10, 256), ("flat", 100, 225), ("tenants", 10, 256),
                                       ("deleted", 10, 250), ("plus", 20, 256), ("flat", 10, 487), ("ties", 10, 225)])
def test_wide_passes(kind, k, nq):
    """340,000 vectors and more than 224 queries take a wide pass (and leave a
    rest of 231 for another one); the ids and scores are the scan's."""
    print("wide %s k=%d nq=%d" % (kind, k, nq), flush=True)
    d, n, T = 256, 340_007, 10
    g = torch.Generator(device="cuda").manual_seed(nq)
    cb, rot = tq.Codebook(d, 4), tq.Rotation(d, 42)
    c = torch.randn(500, d, generator=g, device="cuda")
    X = torch.randn(n, d, generator=g, device="cuda") * 0.5 + c[torch.randint(500, (n,), generator=g, device="cuda")]
    Q = torch.randn(nq, d, generator=g, device="cuda") * 0.5 + c[torch.randint(500, (nq,), generator=g, device="cuda")]
    if kind == "ties":      # more equal scores than any list holds: every query goes back to the scan
        X = X[:1].expand(n, d).contiguous()
    ten = torch.randint(T, (n,), generator=g, device="cuda").to(torch.int16)
    idx = (tq.IdMapIndex if kind == "deleted" else tq.Index)(cb, rot, T)
    if kind == "plus":
        idx.calibrate(X[:5000])
    if kind == "deleted":
        idx.add(X, range(n), ten)
        idx.remove(np.arange(0, n, 7))
    else:
        idx.add(X, ten)
    allow = torch.randint(1, 1 << T, (nq, 1), generator=g, device="cuda") if kind == "tenants" else None
    a_i, a_s = idx.search(Q, k, allow=allow)
    b_i, b_s = idx.search(Q, k, allow=allow, path="lut")
    assert torch.equal(a_i, b_i) and torch.equal(a_s, b_s)


@pytest.mark.parametrize("bits,d,n,nq", [(4, 1536, 5000, 33), (4, 1536, 5000, 224), (2, 512, 4100, 257), (3, 128, 9001, 300),
                                         (8, 640, 3001, 95), (8, 128, 700, 65)])
@pytest.mark.parametrize("filt", [False, True])
def test_groups_of_tiles(bits, d, n, nq, filt):
    """More than one tile of 32 queries, whole and ragged, up to more than the
    8 tiles of a group; the ids and scores are the scan's."""
    print("groups b=%d d=%d n=%d nq=%d filt=%d" % (bits, d, n, nq, filt), flush=True)
    T = 70
    g = torch.Generator(device="cuda").manual_seed(n + nq)
    cb, rot = tq.Codebook(d, bits), tq.Rotation(d, 42)
    X = torch.randn(n, d, generator=g, device="cuda")
    Q = torch.randn(nq, d, generator=g, device="cuda")
    idx = tq.Index(cb, rot, T)
    idx.add(X, torch.randint(T, (n,), generator=g, device="cuda").to(torch.int16))
    allow = torch.randint(-(1 << 60), 1 << 60, (nq, 2), generator=g, device="cuda") if filt else None
    for k in (1, 10, 100):
        a_i, a_s = idx.search(Q, k, allow=allow)
        b_i, b_s = idx.search(Q, k, allow=allow, path="lut")
        assert torch.equal(a_i, b_i) and torch.equal(a_s, b_s), k


def test_eight_bit_close_candidates():
    """Clusters so tight that more than 64 candidates of a query lie within
    the error of its tenth best, many with equal stored scores."""
    print("8-bit close candidates", flush=True)
    d, n, nq = 768, 60_000, 256
    g = torch.Generator(device="cuda").manual_seed(8)
    c = torch.randn(40, d, generator=g, device="cuda")
    near = lambda m: torch.randn(m, d, generator=g, device="cuda") * 0.08 + c[torch.randint(40, (m,), generator=g, device="cuda")]
    idx = tq.Index(tq.Codebook(d, 8), rotation(d))
    idx.add(near(n))
    Q = near(nq)
    for k in (1, 5, 10, 64, 65):
        same(idx.search(Q, k), idx.search(Q, k, path="lut"))
