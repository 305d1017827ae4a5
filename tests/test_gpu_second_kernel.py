"""Offsets and gather of the encoder's strings, bit for bit against the oracle, on both sides of the lines where the launch
takes another shape: buckets per workgroup (4, 16, 64), groups per workgroup (one, two, more, the most), sums over all units
or per chunk of them, for one worker and for several whose strings differ."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("n,nb", [(16, 1), (16, 15), (16, 65), (16, 64 * 1023), (16, 64 * 1023 + 1), (16, 16 * 8192),
                                  (16, 16 * 8192 + 1), (16, 64 * 32767), (16, 64 * 32767 + 1), (600, 3), (600, 16383),
                                  (600, 16384), (600, 4 * 8192), (600, 4 * 8192 + 1), (600, 64 * 1023),
                                  (600, 64 * 1023 + 1), (2049, 5), (2049, 8192), (2049, 8193),
                                  (2049, 16384)])
def test_offsets_and_gather(g, n, nb):
    nuq, s = g.nuq, 3
    rng = np.random.default_rng(nb + n)
    d = nb * n - min(3, n - 1)
    q = np.zeros(d, dtype=np.uint8)
    at = rng.integers(0, d, size=min(d, max(2 * nb, 8)))       # some buckets empty, most strings of one to three words
    q[at] = rng.integers(1, s + 2, size=at.size) | (rng.integers(0, 2, size=at.size) << 7)
    first = slice(0, min(n, d))
    q[first] = 1                                               # and one long one, before all the others
    m = g.alloc_message(d, n, s, 0)
    nuq.nuq_encode(torch.from_numpy(q).to(g.DEV), n, s, 0, m.bit_off, m.words, None, g.workspace(d, n, s))
    assert nuq.nuq_last_error_flags() == 0
    bo, words, _ = oracle.encode(q, n, s, 0)
    assert np.array_equal(g.u64(m.bit_off), bo)
    assert np.array_equal(g.u32(m.words)[: words.size], words)


@pytest.mark.parametrize("n,nb,K", [
    (2, 30_001, 5),             # direct sums, 64 buckets per workgroup
    (2, 140_001, 3),            # sums per chunk
    (2, 64 * 1536 + 1, 32),     # three groups per one-wave workgroup, direct sums
    (2, 64 * 4097, 32),         # eight, sums per chunk
    (600, 4 * 8192 + 5, 4),     # units of four buckets, sums per chunk
    (1025, 16 * 1025, 32),      # two groups of 16 buckets per workgroup, units of four
    (2049, 9_001, 2),           # units of one bucket, sums per chunk
])
def test_several_workers(g, n, nb, K):
    nuq, s = g.nuq, 3
    rng = np.random.default_rng(nb + n)
    d = nb * n - 1

    def gradient(k):                                           # every third worker has the same one, with other draws
        v = np.zeros(d, dtype=np.float32)
        at = rng.integers(0, d, size=nb * (k + 1) // 2)
        v[at] = rng.choice([-1.0, 1.0], at.size)
        v[: 2 * n] = 1.0
        return v, oracle.bucket_norms(v, n).astype(np.float32)

    grads = [gradient(k) for k in range(min(K, 3))]
    vts = [torch.from_numpy(v).to(g.DEV) for v, _ in grads]
    seeds = [int(x) for x in rng.integers(0, 2 ** 62, K)]

    def reference(k):
        v, norms = grads[k % 3]
        return oracle.encode(oracle.quantize(v, n, s, seeds[k], norms), n, s, 0)[:2]

    with ThreadPoolExecutor(max_workers=8) as pool:
        want = list(pool.map(reference, range(K)))
    assert len({int(bo[-1]) for bo, _ in want}) >= min(K, 3)
    new = lambda size, dt, fill: torch.full((size,), fill, dtype=dt, device=g.DEV)
    msgs = [nuq.Message(new(nb, torch.float32, -1.0), new(nb + 1, torch.int64, -1), new(w.size + 8, torch.int32, 0),
                        new(1, torch.int32, 0)) for _, w in want]
    ws = torch.empty(nuq.nuq_encode_workspace_bytes(K, d, n, s), dtype=torch.uint8, device=g.DEV)
    nuq.nuq_quantize_encode_batch([vts[k % 3] for k in range(K)], n, s, seeds, 0, msgs, ws)
    assert nuq.nuq_last_error_flags() == 0
    for k, (m, (bo, words)) in enumerate(zip(msgs, want)):
        assert np.array_equal(m.norms.cpu().numpy(), grads[k % 3][1])
        assert np.array_equal(g.u64(m.bit_off), bo)
        assert np.array_equal(g.u32(m.words)[: words.size], words)
        assert not g.u32(m.words)[words.size:].any()
