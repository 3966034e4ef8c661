"""The default search of several queries where stored scores leave the float16
range or exact ones the float32 range: ids and scores are the scan's, bit for
bit."""
import numpy as np
import pytest

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


def rows(n, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(n, d, generator=g, device="cuda")
    return x / x.norm(dim=1, keepdim=True)


def same(a, b):
    assert torch.equal(a[0], b[0])
    assert torch.equal(a[1], b[1])


def check(idx, Q, k, allow=None):
    assert idx.workspace_bytes(Q.shape[0], k) > idx.workspace_bytes(Q.shape[0], k, path="lut")
    same(idx.search(Q, k, allow=allow), idx.search(Q, k, allow=allow, path="lut"))


# The constant term of a calibrated score is C / (s_max ||kappa q'||) in the
# stored scores: past 65,504 for these kappa (but 1e-3 and 0).  100 vectors:
# all of them are candidates; 20,011: they are selected.
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("n,k", [(100, 10), (100, 100), (5, 10), (20_011, 10)])
@pytest.mark.parametrize("kappa", [1e-3, 1e-8, 1e-30, 0.0])
def test_narrow_calibration(bits, n, k, kappa):
    print("narrow calibration b=%d n=%d k=%d kappa=%g" % (bits, n, k, kappa), flush=True)
    d = 256
    idx = tq.Index(tq.Codebook(d, bits), rotation(d))
    mu = np.random.default_rng(5).standard_normal(d).astype(np.float32) / 16
    idx.set_calibration(mu, np.full(d, kappa, np.float32))
    idx.add(rows(n, d, 1))
    check(idx, rows(8, d, 2), k)


def test_calibration_fitted_to_near_copies():
    print("calibration fitted to near copies", flush=True)
    d = 256
    x = rows(1, d, 3) + 1e-7 * rows(50, d, 4)
    idx = tq.Index(tq.Codebook(d, 4), rotation(d))
    idx.calibrate(x)
    idx.add(x)
    Q = rows(16, d, 5)
    check(idx, Q, 10)
    ids, scores = idx.search(Q, 10)
    assert (ids >= 0).all() and torch.isfinite(scores).all()


@pytest.mark.parametrize("bits", [4, 8])
def test_narrow_calibration_small_tenants(bits):
    """About 20 vectors for a query: every admitted one is a candidate."""
    print("narrow calibration, small tenants b=%d" % bits, flush=True)
    d, n, T, nq = 256, 20_011, 1000, 40
    idx = tq.Index(tq.Codebook(d, bits), rotation(d), T)
    mu = np.random.default_rng(6).standard_normal(d).astype(np.float32) / 16
    idx.set_calibration(mu, np.full(d, 1e-8, np.float32))
    g = torch.Generator(device="cuda").manual_seed(7)
    idx.add(rows(n, d, 8), torch.randint(T, (n,), generator=g, device="cuda").to(torch.int16))
    words = (T + 63) // 64
    t = torch.randint(T, (nq,), generator=g, device="cuda")
    allow = torch.zeros(nq, words, dtype=torch.int64, device="cuda")
    allow[torch.arange(nq, device="cuda"), t >> 6] = torch.ones_like(t) << (t & 63)
    check(idx, rows(nq, d, 9), 10, allow=allow)


# Scores that are subnormal (rounded to multiples of 2^-149, many equal), tiny
# queries on tiny scales, and s_max ||q'|| above the largest float32.
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("n", [100, 20_011])
@pytest.mark.parametrize("s,q", [(1e-43, 1.0), (3e-45, 1.0), (1e-11, 1e-32), (1e-30, 1.0), (1.0, 1e-36), (100.0, 1e37),
                                 (1e30, 1e7), (0.0, 1.0)])
def test_scales_and_queries(bits, n, s, q):
    print("magnitudes b=%d n=%d s=%g q=%g" % (bits, n, s, q), flush=True)
    d = 256
    cb = tq.Codebook(d, bits)
    codes, scales = tq.rotate_quantize(cb, rotation(d), rows(n, d, 11))
    idx = tq.Index(cb, rotation(d))
    idx.add_codes(codes, scales * s)
    check(idx, rows(40, d, 12) * q, 10)
