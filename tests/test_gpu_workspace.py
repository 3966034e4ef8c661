"""Workspaces that are not the size the call would ask for: made for more
queries, or for another path."""
import pytest

from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu
if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

import paper_2607_16973_amd as tq  # noqa: E402

D, N, K = 256, 340_007, 10   # from 333,334 vectors on 256 queries are a wide pass


def rows(n, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n, d, generator=g, device="cuda")


@pytest.fixture(scope="module")
def index():
    idx = tq.Index(tq.Codebook(D, 4), tq.Rotation(D, 42))
    idx.add(rows(N, D, 1))
    return idx


@pytest.mark.parametrize("made_for", [256, 1000])
@pytest.mark.parametrize("path", ["auto", "mfma"])
def test_workspace_made_for_more_queries(index, made_for, path):
    """One workspace for the largest batch serves every smaller one, on the
    batched path (which writes past the room of the scan)."""
    ws = torch.empty(index.workspace_bytes(made_for, K, path=path), dtype=torch.uint8, device="cuda")
    Q = rows(256, D, 2)
    for nq in (4, 33, 64, 65, 96, 97, 128, 160, 161, 224, 225, 256):
        print("workspace for %d, %d queries, %s" % (made_for, nq, path), flush=True)
        q = Q[:nq].contiguous()
        lut = index.workspace_bytes(nq, K, path="lut")
        ws.fill_(0xAB)
        ids, scores = index.search(q, K, path=path, workspace=ws)
        assert (ws[lut:] != 0xAB).any()
        want = index.search(q, K, path="lut")
        assert torch.equal(ids, want[0]) and torch.equal(scores, want[1])


@pytest.mark.parametrize("plus", [False, True])
def test_smallest_workspaces(plus):
    """Every size from the scan's up is taken, results do not depend on it,
    and nothing past its end is written."""
    d, n, nq, k = 256, 60_013, 200, 10
    X = rows(n, d, 3)
    idx = tq.Index(tq.Codebook(d, 4), tq.Rotation(d, 42))
    if plus:
        idx.calibrate(X[:2000])
    idx.add(X)
    Q = rows(nq, d, 4)
    want = idx.search(Q, k, path="lut")
    lo, hi = idx.workspace_bytes(nq, k, path="lut"), idx.workspace_bytes(nq, k)
    buf = torch.empty(hi + 4096, dtype=torch.uint8, device="cuda")
    for i in range(17):
        size = lo + (hi - lo) * i // 16
        print("workspace of %d bytes" % size, flush=True)
        buf.fill_(0xAB)
        ids, scores = idx.search(Q, k, workspace=buf[:size])
        assert torch.equal(ids, want[0]) and torch.equal(scores, want[1])
        assert (buf[size:] == 0xAB).all()


def take_memory(leave):
    """Tensors that hold all of the GPU's memory but about `leave` bytes."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    for _ in range(20):
        free = torch.cuda.mem_get_info()[0]
        if free < leave + (16 << 20):
            break
        held.append(torch.empty(free - leave, dtype=torch.uint8, device="cuda"))
    return held


def big_index(n=14_000_000, d=128):
    """Codes as they come: a tile's scores alone take 0.9 GB."""
    idx = tq.Index(tq.Codebook(d, 4), tq.Rotation(d, 42), 4)
    g = torch.Generator(device="cuda").manual_seed(5)
    codes = torch.randint(256, (n, d // 2), generator=g, device="cuda", dtype=torch.uint8)
    idx.add_codes(codes, torch.rand(n, generator=g, device="cuda") + 0.5)
    return idx


def test_search_where_the_batched_workspace_does_not_fit():
    """100 MiB left on the GPU: the default search of four queries takes the
    scan's workspace instead of failing, in the library and in the binding."""
    print("little memory left", flush=True)
    idx = big_index()
    Q = rows(4, 128, 6)
    assert idx.workspace_bytes(4, K) > 800 << 20
    want = idx.search(Q, K, path="lut")
    held = take_memory(100 << 20)
    try:
        for search in (idx.search_alloc, idx.search):
            print(search.__name__, flush=True)
            ids, scores = search(Q, K)
            assert torch.equal(ids, want[0]) and torch.equal(scores, want[1])
    finally:
        del held
        torch.cuda.empty_cache()


def test_workspace_kept_is_that_of_the_scan_where_the_scan_runs(index):
    """Slot allowlists, and tenant allowlists of few queries, never take the
    batched path: the workspace that the index keeps is the scan's."""
    idx = tq.Index(tq.Codebook(D, 4), tq.Rotation(D, 42))
    idx.add(rows(200_000, D, 7))
    Q = rows(40, D, 8)
    slots = torch.full((40, (200_000 + 63) // 64), -1, dtype=torch.int64, device="cuda")
    idx.search(Q, K, slot_allow=slots)
    assert idx._ws.numel() == idx.workspace_bytes(40, K, path="lut") < idx.workspace_bytes(40, K)
    idx._ws = None
    few = tq.AUTO_FILTERED_QUERIES - 1
    allow = torch.ones(40, 1, dtype=torch.int64, device="cuda")
    idx.search(Q[:few].contiguous(), K, allow=allow[:few].contiguous())
    assert idx._ws.numel() == idx.workspace_bytes(few, K, path="lut") < idx.workspace_bytes(few, K)
    idx.search(Q, K, allow=allow)
    assert idx._ws.numel() == idx.workspace_bytes(40, K)


def test_encode_where_the_workspace_of_large_chunks_does_not_fit():
    """40,000 rows at d = 1536 take 410 MB in chunks of 32,768; with 300 MiB
    left they are encoded in smaller ones, to the same codes."""
    print("encode with little memory left", flush=True)
    d, n = 1536, 40_000
    cb, rot = tq.Codebook(d, 4), tq.Rotation(d, 42)
    X = rows(n, d, 9)
    want = tq.rotate_quantize(cb, rot, X)
    got = tuple(torch.empty_like(t) for t in want)
    idx = tq.Index(cb, rot)
    idx.reserve(n)
    held = take_memory(300 << 20)
    try:
        tq.rotate_quantize(cb, rot, X, codes=got[0], scales=got[1])
        idx.add(X)
        torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert torch.equal(idx.export()[0], want[0])
