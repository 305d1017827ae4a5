"""nuq_quantize under finite norms that the caller supplies, over vectors that hold infinite coordinates and NaNs: an infinite
coordinate takes the top level, a NaN level 1 beside coordinates that all lie below twice the first level and the top
level elsewhere, and no other coordinate is touched by it."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("n", [300, 512, 2048, 8192, 20000])
@pytest.mark.parametrize("s", [1, 3, 14])
@pytest.mark.parametrize("route", ["first", "two", "any"])
@pytest.mark.parametrize("norm", [1.0, 1e-30])
def test_nan_and_infinity(g, n, s, route, norm):
    nuq, d = g.nuq, 3 * n + 17
    rng = np.random.default_rng(n + s)
    top = {"first": 0.9 * 2.0 ** -s, "two": 1.9 * 2.0 ** -s, "any": 1.0}[route]
    v = (rng.uniform(0.4, 1.0, d) * top * norm * rng.choice([-1.0, 1.0], d)).astype(np.float32)
    at = rng.permutation(d - 4)[:24].reshape(3, 8)
    if route == "any":
        v[::4] = np.copysign(np.float32(norm), v[::4])         # every group of four holds one at the norm
        at = at - at % 4 + 1
    v[at[0]], v[at[1]] = np.nan, -np.nan
    v.view(np.uint32)[at[0][:4]] = 0x7FA00001                  # signaling
    if route == "any":
        v[at[2]] = np.inf
    v.view(np.uint32)[at[2][:4]] |= 0x80000000
    norms = np.full(oracle.num_buckets(d, n), norm, dtype=np.float32)
    q = torch.full((d,), 0x7F, dtype=torch.uint8, device=g.DEV)
    nuq.nuq_quantize(torch.from_numpy(v).to(g.DEV), n, s, n, torch.from_numpy(norms).to(g.DEV), q)
    want = oracle.quantize(v, n, s, n, norms)
    isnan = np.isnan(v)
    want[isnan] = np.where(np.signbit(v[isnan]), 0x80, 0) | (s + 1 if route == "any" else 1)
    np.testing.assert_array_equal(q.cpu().numpy(), want)
    if route == "any":
        assert (want[at[2]] & 0x7F).min() >= 1 and (want[np.isinf(v)] & 0x7F == s + 1).all()
    assert nuq.nuq_last_error_flags() == 0
