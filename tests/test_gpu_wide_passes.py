"""Wide passes (one pass over the code store for up to 256 queries) at sizes
that take them: from 333,334 vectors on for more than 224 queries, 1,000,000
for more than 160.  Against the oracle's brute force over the whole corpus and
the single-query scan's lists."""
import numpy as np
import pytest

import oracle
import synth
from tests.conftest import gpu_available
from tests.parity import assert_codes_equal, check_topk, oracle_tables

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

import paper_2607_16973_amd as tq  # noqa: E402

D = 256


def rows(n, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n, d, generator=g, device="cuda")


def is_wide(monkeypatch, idx, nq, k):
    """Wide passes take up to 1,024 workgroups: their lists are in the workspace
    for 1,024 and not for 1,025, which is the same size otherwise."""
    size = []
    for grid in (1024, 1025):
        monkeypatch.setenv("TQ_SCAN_GRID", str(grid))
        size.append(idx.workspace_bytes(nq, k))
    monkeypatch.delenv("TQ_SCAN_GRID")
    return abs(size[0] / size[1] - 1) > 0.01


@pytest.mark.parametrize("n,k", [(1_000_000, 100), (1_600_000, 100), (1_850_000, 256), (1_600_000, 20), (2_200_000, 100),
                                 (7_500_000, 10)])
def test_candidates_fit(monkeypatch, n, k):
    """The largest corpora that wide passes take: a query's candidates fit the
    final selection, so that hardly any goes back to the scan."""
    print("wide candidates n=%d k=%d" % (n, k), flush=True)
    idx = tq.Index(tq.Codebook(D, 4), tq.Rotation(D, 42))
    idx.reserve(n)
    for i in range(0, n, 400_000):
        idx.add(rows(min(400_000, n - i), D, 100 + i))
    Q = rows(256, D, 3)
    assert is_wide(monkeypatch, idx, 256, k) and not is_wide(monkeypatch, idx, 160, k)
    ids, scores = idx.search(Q, k, path="mfma")
    assert tq.last_search_fallbacks() <= 2
    want = idx.search(Q[:8].contiguous(), k, path="lut")
    assert torch.equal(ids[:8], want[0]) and torch.equal(scores[:8], want[1])


class Corpus:
    """334,011 clustered rows (the last block is partial), coded by the library;
    a sample of the codes is the oracle's."""

    def __init__(self, d):
        self.n, self.d = 334_011, d
        g = torch.Generator(device="cuda").manual_seed(d)
        c = torch.randn(500, d, generator=g, device="cuda")
        near = lambda m: torch.randn(m, d, generator=g, device="cuda") * 0.5 + c[torch.randint(500, (m,), generator=g, device="cuda")]
        X, self.Q = near(self.n), near(256)
        self.cb, self.rot = tq.Codebook(d, 4), tq.Rotation(d, 42)
        self.packed, self.scales_d = tq.rotate_quantize(self.cb, self.rot, X)
        R32, tables = self.rot.matrix(), oracle_tables(self.cb)
        sample = slice(0, self.n, 1000)
        want, _, _ = oracle.encode(X[sample].cpu().numpy(), R32, tables)
        assert_codes_equal(self.packed[sample].cpu().numpy(), want, 4)
        self.cents = tables.cents
        self.codes = oracle.unpack_codes(self.packed.cpu().numpy(), d, 4)
        self.scales = self.scales_d.cpu().numpy()
        Q = self.Q.cpu().numpy()
        self.qrot = oracle.rotate_queries(R32, Q)
        self.qn = np.linalg.norm(Q.astype(np.float64), axis=1)
        self.scores = oracle.score_all(self.codes, self.scales, self.cents, self.qrot)

    def index(self, tenants=None, T=1):
        idx = tq.Index(self.cb, self.rot, T)
        idx.add_codes(self.packed, self.scales_d, tenants)
        return idx

    def check(self, idx, nq, k, path, tenants=None, bm=None):
        Q = self.Q[:nq].contiguous()
        allow = None if bm is None else torch.from_numpy(bm.view(np.int64)).cuda()
        ids, scores = idx.search(Q, k, allow=allow, path=path)
        lut = idx.search(Q, k, allow=allow, path="lut")
        assert torch.equal(ids, lut[0]) and torch.equal(scores, lut[1])
        masks = None if bm is None else [oracle.allowed_mask(tenants, bm[b]) for b in range(nq)]
        ref_i, ref_s = oracle.topk_from_scores(self.scores[:nq], k, tenants=tenants, allow=bm)
        check_topk(ids.cpu().numpy(), scores.cpu().numpy(), self.codes, self.scales, self.cents, self.qrot[:nq],
                   self.qn[:nq], k, ref_i, ref_s, allowed=masks)


@pytest.fixture(scope="module", params=[256, 384])
def corpus(request):
    """d = 384: 12 chunks a vector, not whole rings of 8."""
    print("wide corpus d=%d" % request.param, flush=True)
    return Corpus(request.param)


@pytest.mark.parametrize("nq,k", [(225, 10), (256, 1), (256, 100)])
def test_against_the_oracle(monkeypatch, corpus, nq, k):
    print("wide oracle d=%d nq=%d k=%d" % (corpus.d, nq, k), flush=True)
    idx = corpus.index()
    assert is_wide(monkeypatch, idx, nq, k)
    corpus.check(idx, nq, k, "auto")
    if corpus.d % 256 == 0:
        corpus.check(idx, nq, k, "mfma")
        assert tq.last_search_fallbacks() <= nq // 8


@pytest.mark.parametrize("mode", ["selective", "broad"])
def test_tenants_against_the_oracle(monkeypatch, corpus, mode):
    print("wide oracle d=%d tenants, %s" % (corpus.d, mode), flush=True)
    T, nq, k = 100, 240, 10
    tenants = synth.zipf_tenants(corpus.n, T, seed=44)
    bm = synth.allowlist_bitmap(synth.allowlists(nq, T, mode, seed=45), T)
    idx = corpus.index(torch.from_numpy(tenants.view(np.int16)).cuda(), T)
    assert is_wide(monkeypatch, idx, nq, k)
    corpus.check(idx, nq, k, "auto", tenants, bm)


def test_selective_pass_is_left_to_the_scan():
    """1,000 tenants of 2,400 neighbouring vectors, 161 queries of one each: by
    the device's rule the scan takes 161 x 9 us and 10 ns for each of 6,300
    blocks, 1.5 ms, and the pass 2 ms for its 1.8 GB.  The pass's kernels leave
    (the 67 MB of pilot scores are not written), the lists are the scan's."""
    print("wide pass left to the scan", flush=True)
    d, n, nq, k, T = 1536, 2_400_000, 161, 10, 1000
    g = torch.Generator(device="cuda").manual_seed(11)
    idx = tq.Index(tq.Codebook(d, 4), tq.Rotation(d, 42), T)
    idx.reserve(n)
    ten = (torch.arange(n, device="cuda") // (n // T)).to(torch.int16)
    for i in range(0, n, 600_000):
        codes = torch.randint(256, (600_000, d // 2), generator=g, device="cuda", dtype=torch.uint8)
        idx.add_codes(codes, torch.rand(600_000, generator=g, device="cuda") + 0.5, ten[i:i + 600_000].contiguous())
    Q = rows(nq, d, 12)
    one = torch.zeros(nq, 16, dtype=torch.int64, device="cuda")
    t = torch.randint(T, (nq,), generator=g, device="cuda")
    one[torch.arange(nq, device="cuda"), t >> 6] = torch.ones_like(t) << (t & 63)
    ws = torch.empty(idx.workspace_bytes(nq, k), dtype=torch.uint8, device="cuda")
    for allow, left in ((one, True), (torch.full_like(one, -1), False)):
        ws.fill_(0xAB)
        ids, scores = idx.search(Q, k, allow=allow, workspace=ws)
        assert ((ws != 0xAB).sum().item() < 24e6) == left
        want = idx.search(Q[:40].contiguous(), k, allow=allow[:40].contiguous(), path="lut")
        assert torch.equal(ids[:40], want[0]) and torch.equal(scores[:40], want[1])
