"""ENCODE from crafted level|sign bytes at the edges of the coding phase, bit for bit against the oracle: one to sixteen
rows per thread, the byte format on both sides of s = 7, gaps on both sides of the table's range, more records per thread
than are kept in registers, exactly as many nonzeros as the index list holds and one more, bit strings on both sides of the
buffer's size."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("s", [3, 7, 8, 14])
@pytest.mark.parametrize("n,S", [(512, 128), (512, 64), (500, 256), (60, 64), (64, 0), (1, 0), (17, 64), (2048, 64),
                                 (1000, 128), (1021, 1024), (2049, 256), (8192, 256), (5000, 64), (16384, 128),
                                 (20001, 512), (32768, 1024)])
def test_crafted_bytes(g, n, S, s):
    nuq = g.nuq
    rng = np.random.default_rng(n * 16 + s)
    cap = nuq.nuq_encode_shape(1, 1, 10 * n, n, s, S)[1]                                   # indices the list holds
    counts = [n, min(n, cap), min(n, cap + 1), max(n // 4, 1), max(n // 15, 1), max(n // 40, 1), 1, 0, n // 2, n]
    d = len(counts) * n - min(5, n - 1)
    q = np.zeros(d, dtype=np.uint8)
    for b, c in enumerate(counts):
        lo, hi = b * n, min(d, (b + 1) * n)
        at = rng.choice(hi - lo, size=min(c, hi - lo), replace=False)
        lev = rng.integers(1, s + 2, size=at.size) if b % 3 else np.where(rng.random(at.size) < 0.9, 1, s + 1)
        q[lo + at] = (lev | (rng.integers(0, 2, size=at.size) << 7)).astype(np.uint8)
    if n >= 64:                                    # gaps of 15, 16, 31, 32, 33 and the largest there is
        q[6 * n:7 * n] = 0
        at = np.cumsum([1, 15, 16])
        q[6 * n + at] = 1
        if n >= 256:
            q[6 * n + at[-1] + np.cumsum([31, 32, 33])] = s + 1
        q[7 * n - 1] = 0x81
    m = g.alloc_message(d, n, s, S)
    nuq.nuq_encode(torch.from_numpy(q).to(g.DEV), n, s, S, m.bit_off, m.words, m.sync if nuq.nuq_num_sync(n, S) else None,
                   g.workspace(d, n, s))
    assert nuq.nuq_last_error_flags() == 0
    bo, words, sync = oracle.encode(q, n, s, S)
    np.testing.assert_array_equal(g.u64(m.bit_off), bo)
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    assert not g.u32(m.words)[words.size:].any()
    if sync.size:
        np.testing.assert_array_equal(g.u32(m.sync)[: sync.size], sync)


@pytest.mark.parametrize("s,density", [(1, 0.04), (3, 0.04), (7, 0.04), (7, 0.9), (8, 0.3), (14, 0.9)])
@pytest.mark.parametrize("n,S", [(500, 128), (512, 128), (2048, 256), (1000, 64), (8192, 256), (20001, 512)])
def test_levels_above_the_top(g, n, S, s, density):
    """A level index above s + 1 is the caller's error, but not one that turns into another valid message: the level is coded
    modulo 16 (1 for a multiple of 16), no other record changes, and the decoder refuses a level it does not have."""
    nuq = g.nuq
    rng = np.random.default_rng(n + 100 * s)
    d = 4 * n - 7
    q = np.where(rng.random(d) < density, rng.integers(1, s + 2, d), 0)
    bad = (q > 0) & (rng.random(d) < 0.2)
    bad[rng.permutation(np.flatnonzero(q))[:24]] = True
    q[bad] = rng.integers(s + 2, 128, np.count_nonzero(bad))
    q[np.flatnonzero(bad)[:8]] = [9, 15, 16, 17, 64, 65, 112, 127]
    coded = np.where((q > 0) & (q % 16 == 0), 1, q % 16)
    sign = np.where(q > 0, rng.integers(0, 2, d) << 7, 0)
    m = g.alloc_message(d, n, 14, S)
    nuq.nuq_encode(torch.from_numpy((q | sign).astype(np.uint8)).to(g.DEV), n, s, S, m.bit_off, m.words, m.sync,
                   g.workspace(d, n, s))
    assert nuq.nuq_last_error_flags() == 0
    bo, words, sync = oracle.encode((coded | sign).astype(np.uint8), n, 14, S)
    np.testing.assert_array_equal(g.u64(m.bit_off), bo)
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    np.testing.assert_array_equal(g.u32(m.sync)[: sync.size], sync)
    m.norms.fill_(1.0)
    out = torch.empty(d, dtype=torch.float32, device=g.DEV)
    nuq.nuq_decode_accumulate([m], d, n, s, S, 1.0, False, out)
    assert nuq.nuq_last_error_flags() == (nuq.FLAG_MALFORMED if (coded > s + 1).any() else 0)


@pytest.mark.parametrize("n,S", [(3000, 0), (3000, 64), (8192, 256), (16384, 128), (20000, 512), (32768, 1024)])
def test_strings_of_one_window_and_of_two(g, n, S):
    """Buckets without a zero, a string of exactly the words that are put together at once, a word more, and the longest."""
    nuq, s = g.nuq, 14
    rng = np.random.default_rng(n)
    _, listed, _, cap = nuq.nuq_encode_shape(1, 1, 6 * n, n, s, S)
    assert listed < n
    x = (32 * cap - 3 * n) // 6                                # records of 9 bits (level 15), the others take 3 (level 1)
    d = 6 * n
    q = np.ones(d, dtype=np.uint8)
    for b, c in enumerate((x, x + 1, n, x + 6, x - 6, x)):
        q[b * n + rng.permutation(n)[:c]] = 15
    q |= (rng.integers(0, 2, d) << 7).astype(np.uint8)
    m = g.alloc_message(d, n, s, S)
    nuq.nuq_encode(torch.from_numpy(q).to(g.DEV), n, s, S, m.bit_off, m.words, m.sync if S else None, g.workspace(d, n, s))
    assert nuq.nuq_last_error_flags() == 0
    bo, words, sync = oracle.encode(q, n, s, S)
    lens = (bo[1:].astype(np.int64) - (bo[:-1].astype(np.int64) + 31) // 32 * 32 + 31) // 32
    assert lens[0] == cap and lens[1] == cap + 1 and lens[2] > cap
    np.testing.assert_array_equal(g.u64(m.bit_off), bo)
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    if S:
        np.testing.assert_array_equal(g.u32(m.sync)[: sync.size], sync)


@pytest.mark.parametrize("s", [1, 3])
@pytest.mark.parametrize("n,S", [(64, 64), (200, 0), (300, 64), (512, 128), (1000, 256), (1024, 0), (2000, 64), (2049, 512),
                                 (3000, 0), (8192, 256), (16384, 128), (20001, 512), (32768, 1024)])
def test_strings_longer_than_slots(g, n, S, s):
    """Levels above s + 1 can make a string longer than any of levels up to it: of exactly a slot's words it is coded like any
    other, a word longer it is refused.  The bucket is one word of ones, the flag is raised, decoders refuse it, and no other
    bucket changes, in the same workgroup or not."""
    nuq = g.nuq
    rng = np.random.default_rng(n + s)
    slot = ((n * (5 if s == 1 else 8) + 31) // 32 + 3) & ~3
    x = (32 * slot - 3 * n) // 6                            # records of 9 bits (level 15), the others take 3 (level 1)

    def full(high):
        b = np.ones(n, dtype=np.uint8)
        b[rng.permutation(n)[:high]] = 15
        return b | (rng.integers(0, 2, n) << 7).astype(np.uint8)

    def ordinary():
        return np.where(rng.random(n) < 0.2, rng.integers(1, s + 2, n) | (rng.integers(0, 2, n) << 7), 0).astype(np.uint8)
    every_other = np.where(np.arange(n) % 2 == 0, 15, 0).astype(np.uint8)
    buckets = [ordinary(), full(x + 1), ordinary(), full(x), np.zeros(n, dtype=np.uint8), full(n), full(n), every_other, ordinary(),
               ordinary()] + ([ordinary() for _ in range(9)] + [full(x + 1), ordinary()[: n // 2]])
    q = np.concatenate(buckets)
    d = q.size
    bit_off, words, sync, kept = [0], [], [], []
    for b in buckets:
        bo, w, sy = oracle.encode(b, n, 14, S)
        kept.append(w.size <= slot)
        bits, w, sy = (int(bo[1]), w, sy) if kept[-1] else (32, np.array([0xFFFFFFFF], dtype=np.uint32), np.zeros_like(sy))
        bit_off.append(32 * sum(v.size for v in words) + bits)
        words.append(w)
        sync.append(sy)
    assert kept[:7] == [True, False, True, True, True, False, False] and not kept[-2] and words[3].size == slot
    m = g.alloc_message(d, n, 14, S)
    nuq.nuq_encode(torch.from_numpy(q).to(g.DEV), n, s, S, m.bit_off, m.words, m.sync if S else None, g.workspace(d, n, s))
    assert nuq.nuq_last_error_flags() == nuq.FLAG_MALFORMED
    words = np.concatenate(words)
    np.testing.assert_array_equal(g.u64(m.bit_off), np.array(bit_off, dtype=np.uint64))
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    assert not g.u32(m.words)[words.size:].any()
    if S:
        np.testing.assert_array_equal(g.u32(m.sync), np.concatenate(sync))
    m.norms.fill_(1.0)
    legal = np.concatenate([np.full(b.size, k and (b & 127).max() <= s + 1) for k, b in zip(kept, buckets)])
    level = (q & 127).astype(np.int64)
    want = np.where(level > 0, np.ldexp(1.0, level - 1 - s), 0.0) * np.where(q >> 7, -1.0, 1.0)
    out = torch.empty(d, dtype=torch.float32, device=g.DEV)
    for msgs in ([m], [m, m]):
        nuq.nuq_decode_accumulate(msgs, d, n, s, S, 1.0 / len(msgs), False, out)
        assert nuq.nuq_last_error_flags() == nuq.FLAG_MALFORMED
        np.testing.assert_array_equal(out.cpu().numpy()[legal], want[legal].astype(np.float32))


@pytest.mark.parametrize("s", [6, 7, 8, 14])
@pytest.mark.parametrize("n,nb,S", [(17, 40, 0), (64, 19, 64), (200, 21, 64), (256, 33, 128), (300, 18, 64), (400, 19, 256),
                                    (512, 21, 64), (600, 9, 128), (600, 5200, 128), (768, 5200, 256), (1000, 7, 64),
                                    (1000, 5200, 256), (1024, 6, 1024), (2000, 7, 64)])
def test_longest_strings(g, n, nb, S, s):
    """Several buckets per workgroup, strings up to the longest there are: no zero and the top level (longer than the bytes they
    are made from, where levels need seven bits), every other coordinate, as many nonzeros as the list holds at the longest
    level code, beside ordinary and empty buckets and in a unit that is not full."""
    nuq = g.nuq
    rng = np.random.default_rng(n + nb + s)
    d = nb * n - n // 3
    _, listed, buffer, _ = nuq.nuq_encode_shape(1, 1, d, n, s, S)
    q = np.zeros(nb * n, dtype=np.uint8)
    top = min(s + 1, 15)
    for b in list(range(min(nb, 40))) + list(range(max(nb - 7, 0), nb)):
        at = [np.arange(n), np.flatnonzero(rng.random(n) < 0.2), np.arange(0, n, 2), np.arange(n),
              np.sort(rng.choice(n, min(listed, n), replace=False)), np.arange(0)][b % 6]
        lev = rng.integers(1, s + 2, at.size) if b % 6 == 1 else np.full(at.size, top)
        q[b * n + at] = lev
    q = np.where(q, q | (rng.integers(0, 2, q.size) << 7), 0).astype(np.uint8)[:d]
    m = g.alloc_message(d, n, s, S)
    nuq.nuq_encode(torch.from_numpy(q).to(g.DEV), n, s, S, m.bit_off, m.words, m.sync if S else None, g.workspace(d, n, s))
    assert nuq.nuq_last_error_flags() == 0
    bo, words, sync = oracle.encode(q, n, s, S)
    first = int(bo[1] + 31) // 32
    assert first == (n * (9 if s >= 7 else 8) + 31) // 32
    if listed == n:
        assert buffer >= first and (s < 7 or 32 * buffer > 8 * n)
    np.testing.assert_array_equal(g.u64(m.bit_off), bo)
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    assert not g.u32(m.words)[words.size:].any()
    if sync.size:
        np.testing.assert_array_equal(g.u32(m.sync)[: sync.size], sync)
