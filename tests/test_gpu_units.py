"""ENCODE where a workgroup holds several buckets: strings back to back in the staging area, buckets whose nonzeros fit the index
list beside buckets whose do not, messages that end inside a unit."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def coded(g, q, n, s, S, words_cap=None):
    m = g.alloc_message(q.size, n, s, S)
    m.words.fill_(0x5A5A5A5A)
    words = m.words if words_cap is None else m.words[:words_cap]
    g.nuq.nuq_encode(torch.from_numpy(q).to(g.DEV), n, s, S, m.bit_off, words, m.sync, g.workspace(q.size, n, s))
    return m


def crafted(rng, n, counts, tail, s):
    q = np.zeros(len(counts) * n - tail, dtype=np.uint8)
    for b, c in enumerate(counts):
        size = min(n, q.size - b * n)
        at = rng.choice(size, size=min(c, size), replace=False)
        q[b * n + at] = (rng.integers(1, s + 2, at.size) | (rng.integers(0, 2, at.size) << 7)).astype(np.uint8)
    return q


@pytest.mark.parametrize("s", [3, 8])
@pytest.mark.parametrize("n,S", [(3, 64), (257, 64), (320, 128), (511, 256), (512, 64), (1024, 128), (1025, 64), (2048, 256),
                                 (5000, 64), (14400, 64), (16384, 128)])
def test_list_edges(g, n, S, s):
    """One nonzero fewer than the list holds, as many, one more, in buckets side by side; the last unit partly filled."""
    rng = np.random.default_rng(n + s)
    cap = g.nuq.nuq_encode_shape(1, 1, 33 * n, n, s, S)[1]
    counts = [n // 4, cap - 1, cap, min(n, cap + 1), 0, n, cap, n // 4, min(n, cap + 1), 1, n // 3] * 3
    q = crafted(rng, n, counts, 1 if n > 1 else 0, s)
    m = coded(g, q, n, s, S)
    assert g.nuq.nuq_last_error_flags() == 0
    bo, words, sync = oracle.encode(q, n, s, S)
    np.testing.assert_array_equal(g.u64(m.bit_off), bo)
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    assert (g.u32(m.words)[words.size:] == 0x5A5A5A5A).all()
    np.testing.assert_array_equal(g.u32(m.sync)[: sync.size], sync)


def test_list_edges_of_half_a_wave(g):
    """Half a wave keeps 24 records per thread: 768 nonzeros of a bucket's 1000 (from 5120 buckets of sparse levels)."""
    n, s, S = 1000, 3, 256
    rng = np.random.default_rng(5)
    counts = [40] * 5124
    assert g.nuq.nuq_encode_shape(1, 1, len(counts) * n - 3, n, s, S)[:2] == (32, 768)
    counts[7:12] = counts[5118:5123] = [767, 768, 769, 1000, 768]
    q = crafted(rng, n, counts, 3, s)
    m = coded(g, q, n, s, S)
    bo, words, sync = oracle.encode(q, n, s, S)
    np.testing.assert_array_equal(g.u64(m.bit_off), bo)
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    np.testing.assert_array_equal(g.u32(m.sync)[: sync.size], sync)


@pytest.mark.parametrize("n,nb", [(40, 333), (512, 19), (512, 1100), (1000, 70), (2000, 9), (5000, 7), (8192, 40)])
def test_message_that_ends_inside_a_unit(g, n, nb):
    """A bucket's words are written if all of them fit, nothing behind the message's end is, offsets are complete."""
    s, S = 3, 256
    rng = np.random.default_rng(n)
    q = crafted(rng, n, rng.integers(0, n // 3, nb).tolist(), 0, s)
    bo, words, _ = oracle.encode(q, n, s, S)
    end = (bo[1:] + np.uint64(31)) // np.uint64(32)
    for b in (0, nb // 3, nb - 1):
        cut = max(int(end[b]) - 1, 0)                       # one word short of bucket b
        m = coded(g, q, n, s, S, cut)
        fit = int(end[:b].max(initial=0)) if end[b] else 0
        assert g.nuq.nuq_last_error_flags() == (g.nuq.FLAG_CAPACITY if int(end[-1]) > cut else 0)
        np.testing.assert_array_equal(g.u64(m.bit_off), bo)
        np.testing.assert_array_equal(g.u32(m.words)[:fit], words[:fit])
        assert (g.u32(m.words)[fit:] == 0x5A5A5A5A).all()
