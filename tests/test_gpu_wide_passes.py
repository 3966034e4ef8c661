"""Wide passes (one pass over the code store for up to 256 queries) at sizes
that take them: from 333,334 vectors on for more than 224 queries, 1,000,000
for more than 160."""
import pytest

from tests.conftest import gpu_available

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
