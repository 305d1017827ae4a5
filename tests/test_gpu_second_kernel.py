"""Offsets and gather of the encoder's strings, bit for bit against the oracle, on both sides of every line where the launch
takes another shape: buckets per workgroup (4, 16, 64), groups per workgroup, sums over all units or per chunk of them."""
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
                                  (600, 16384), (600, 4 * 8192), (600, 4 * 8192 + 1), (2049, 5), (2049, 8192), (2049, 8193),
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
