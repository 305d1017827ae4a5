"""DECODE of crafted level|sign bytes at the edges of the record parser, bit for bit against exact sums: gaps on both sides
of every code length, all level codes, runs of every length modulo a word, norms that are zero, infinite or no number, odd
tile ends, and parameters that are updated in place (full tiles, ragged ones, unaligned ones)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def _bytes(rng, d, n, s, sparse):
    """One worker's bytes: gaps drawn around the powers of two below 2^15, levels uniform."""
    q = np.zeros(d, dtype=np.uint8)
    edges = np.array([1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 127, 128, 255, 256, 511, 512, 1023, 4095, 16383])
    at = -1
    while True:
        at += int(rng.choice(edges[edges < n][: len(edges) if sparse else 9])) if n > 1 else 1
        if at >= d:
            break
        q[at] = rng.integers(1, s + 2) | (int(rng.integers(0, 2)) << 7)
    return q


def _message(g, q, n, s, S, norms):
    nuq, d = g.nuq, q.size
    m = g.alloc_message(d, n, s, S)
    nuq.nuq_encode(torch.from_numpy(q).to(g.DEV), n, s, S, m.bit_off, m.words, m.sync if nuq.nuq_num_sync(n, S) else None,
                   g.workspace(d, n, s))
    m.norms.copy_(torch.from_numpy(norms))
    return m


def _value(q, n, s, norms):
    lev = (q & 0x7f).astype(np.int64)
    v = np.repeat(norms.astype(np.float64), n)[: q.size]
    with np.errstate(invalid="ignore"):
        v = np.where(lev > 0, np.ldexp(v, lev - 1 - s), 0.0)
    return np.where(q & 0x80, -v, v)


@pytest.mark.parametrize("s", [1, 3, 7, 14])
@pytest.mark.parametrize("n,S,K", [(8192, 256, 8), (8192, 256, 1), (512, 128, 4), (512, 128, 1), (1000, 128, 3), (16384, 128, 4),
                                   (4096, 256, 2), (20001, 512, 5), (17, 64, 2), (512, 0, 3), (8192, 64, 8), (2048, 0, 1)])
def test_crafted_records(g, n, S, K, s):
    nuq = g.nuq
    rng = np.random.default_rng(n + 64 * s + K)
    d = max(3 * n + n // 3, 9000)
    nb = -(-d // n)
    qs = [_bytes(rng, d, n, s, sparse=k % 2 == 1) for k in range(K)]
    norms = [np.exp2(rng.uniform(-3, 3, nb)).astype(np.float32) for _ in range(K)]
    norms[0][0] = 0.0
    msgs = [_message(g, q, n, s, S, v) for q, v in zip(qs, norms)]
    want = sum(_value(q, n, s, v) for q, v in zip(qs, norms))          # exact in fp64: spans far below 2^29
    out = torch.full((d,), 7.0, device=g.DEV)
    nuq.nuq_decode_accumulate(msgs, d, n, s, S, 0.5, False, out)
    assert nuq.nuq_last_error_flags() == 0
    np.testing.assert_array_equal(out.cpu().numpy(), (0.5 * want).astype(np.float32))
    # added to what is there, at an aligned and at an odd address
    for shift in (0, 1):
        flat = torch.arange(d + 1, dtype=torch.float32, device=g.DEV)
        prior = flat[shift:shift + d].cpu().numpy()
        nuq.nuq_decode_accumulate(msgs, d, n, s, S, 0.5, True, flat[shift:shift + d])
        np.testing.assert_array_equal(flat[shift:shift + d].cpu().numpy(), (0.5 * want).astype(np.float32) + prior)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, -2.0, 2.0 ** -149])
@pytest.mark.parametrize("n,S,K", [(8192, 256, 2), (512, 128, 1)])
def test_unusual_norms(g, n, S, K, bad):
    """A received norm is taken as its magnitude (the sign is the record's), whatever it is."""
    nuq = g.nuq
    rng = np.random.default_rng(5)
    d, s = 3 * n, 3
    qs = [_bytes(rng, d, n, s, sparse=True) for _ in range(K)]
    norms = [np.ones(3, dtype=np.float32) for _ in range(K)]
    norms[0][1] = bad
    msgs = [_message(g, q, n, s, S, v) for q, v in zip(qs, norms)]
    out = torch.empty(d, device=g.DEV)
    nuq.nuq_decode_accumulate(msgs, d, n, s, S, 1.0, False, out)
    want = sum(_value(q, n, s, np.abs(v)) for q, v in zip(qs, norms)).astype(np.float32)
    np.testing.assert_array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("n,S,K,d,shift", [(8192, 256, 8, 8192 * 3 + 5, 0), (512, 128, 4, 512 * 40 + 7, 0), (512, 128, 4, 512 * 40, 1),
                                           (16384, 256, 4, 16384 * 2 + 3000, 0), (1000, 128, 3, 9001, 0)])
def test_momentum_tiles(g, n, S, K, d, shift):
    nuq = g.nuq
    rng = np.random.default_rng(d)
    s, nb = 3, -(-d // n)
    qs = [_bytes(rng, d, n, s, sparse=False) for _ in range(K)]
    norms = [np.exp2(rng.uniform(-3, 3, nb)).astype(np.float32) for _ in range(K)]
    msgs = [_message(g, q, n, s, S, v) for q, v in zip(qs, norms)]
    scale = float(np.float32(1.0 / K))
    gd = (scale * sum(_value(q, n, s, v) for q, v in zip(qs, norms))).astype(np.float32).astype(np.float64)
    w0, y0 = rng.standard_normal((2, d)).astype(np.float32)
    w, y = (torch.empty(d + shift, device=g.DEV)[shift:].copy_(torch.from_numpy(a)) for a in (w0, y0))
    alpha, mu, l = 0.25, 0.5, 1.0
    nuq.nuq_decode_momentum_step(msgs, d, n, s, S, scale, alpha, mu, l, w, y)
    yl = w0.astype(np.float64) - l * alpha * gd
    want = (w0.astype(np.float64) - alpha * gd) + mu * (yl - y0.astype(np.float64))
    np.testing.assert_allclose(w.cpu().numpy(), want, rtol=2.0 ** -23, atol=2.0 ** -30)      # one rounding to fp32
    np.testing.assert_allclose(y.cpu().numpy(), yl, rtol=2.0 ** -23, atol=2.0 ** -30)


def _dense_bytes(rng, d, n, s, density):
    """Bytes whose share of nonzeros differs from bucket to bucket around `density`, a bucket in four full, one empty."""
    nb = -(-d // n)
    share = np.clip(density * 2.0 ** rng.uniform(-1, 1, nb), 0, 1)
    share[::4], share[1::8] = 1.0, 0.0
    level = rng.integers(1, s + 2, d).astype(np.uint8) | (rng.integers(0, 2, d).astype(np.uint8) << 7)
    return np.where(rng.random(d) < np.repeat(share, n)[:d], level, 0).astype(np.uint8)


@pytest.mark.parametrize("density", [0.02, 0.25, 0.7])
@pytest.mark.parametrize("n,S,K,s", [(8192, 256, 8, 3), (512, 128, 4, 3), (512, 256, 4, 7), (512, 512, 2, 14), (256, 256, 4, 3),
                                     (256, 64, 3, 5), (1000, 256, 8, 3), (1024, 512, 3, 2), (16384, 512, 4, 7), (20000, 1024, 2, 14),
                                     (64, 64, 2, 3)])
def test_pieces_of_every_length(g, n, S, K, s, density):
    """Pieces of less than a row of words to many rows, one to eight lanes loading a row, in messages that end with their last
    word (the last piece's row would leave the message): the average, and the same through Huffman-coded levels."""
    nuq = g.nuq
    rng = np.random.default_rng(n + 7 * S + K)
    d = 9 * n + n // 2 + 1
    nb = -(-d // n)
    qs = [_dense_bytes(rng, d, n, s, density) for _ in range(K)]
    norms = [np.exp2(rng.uniform(-3, 3, nb)).astype(np.float32) for _ in range(K)]
    want = (0.5 * sum(_value(q, n, s, v) for q, v in zip(qs, norms))).astype(np.float32)      # the sum is exact in fp64

    def cut(m):        # the message's words alone, the next thing in memory something else
        used = (int(m.bit_off[-1].item()) + 31) // 32
        return nuq.Message(m.norms, m.bit_off, m.words[:used].clone(), m.sync)

    msgs = [cut(_message(g, q, n, s, S, v)) for q, v in zip(qs, norms)]
    out = torch.full((d,), 7.0, device=g.DEV)
    nuq.nuq_decode_accumulate(msgs, d, n, s, S, 0.5, False, out)
    assert nuq.nuq_last_error_flags() == 0
    np.testing.assert_array_equal(out.cpu().numpy(), want)

    nsync = nuq.nuq_huffman_num_sync(n, S)
    if not nsync or -(-min(n, 2048) // S) > 64 // (max(1, 2048 // n) * K):
        return                                     # no index, or more pieces in a tile than lanes: not taken
    for code_s, hist in ((s, [1 << (s + 1 - j) for j in range(s + 2)]), (s, [1] * (s + 2))):     # "0" for level 0, and not
        lengths = nuq.nuq_huffman_lengths(hist, code_s)
        hm = []
        for q, v in zip(qs, norms):
            m = nuq.Message(torch.from_numpy(v).to(g.DEV), torch.empty(nb + 1, dtype=torch.int64, device=g.DEV),
                            torch.zeros(nuq.nuq_huffman_max_words(d, n), dtype=torch.int32, device=g.DEV),
                            torch.empty(max(1, nb * nsync), dtype=torch.int32, device=g.DEV))
            ws = torch.empty(nuq.nuq_encode_huffman_workspace_bytes(d, n), dtype=torch.uint8, device=g.DEV)
            nuq.nuq_encode_huffman(torch.from_numpy(q).to(g.DEV), n, s, S, lengths, m.bit_off, m.words, m.sync, ws)
            hm.append(cut(m))
        out.fill_(7.0)
        nuq.nuq_decode_accumulate_huffman(hm, d, n, s, S, lengths, 0.5, False, out)
        assert nuq.nuq_last_error_flags() == 0
        np.testing.assert_array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n,S,s,d", [(511, 64, 3, 511 * 9 + 1), (512, 64, 3, 512 * 70), (513, 512, 3, 513 * 70 + 2), (1000, 256, 7, 1), (1000, 256, 7, 40_003),
                                     (2047, 1024, 14, 2047 * 40 + 5), (2049, 128, 3, 2049 * 30 + 2048), (4098, 256, 5, 4098 * 9 + 3),
                                     (8192, 256, 3, 8192 * 700 + 77), (20001, 64, 3, 20001 * 3 + 2049), (32768, 1024, 1, 32768 * 5 + 4),
                                     (8192, 256, 1, 8192 * 1024 - 1), (8192, 256, 1, 8192 * 1024 + 77)])
def test_one_message(g, n, S, s, d, shift):
    """A single message written out: blocks per workgroup from one to the most that fit, odd bucket sizes (blocks that begin and
    end inside a float4 group), a last bucket that ends inside a block and leaves others empty, an odd output address."""
    nuq = g.nuq
    rng = np.random.default_rng(d + n)
    nb = -(-d // n)
    q = _dense_bytes(rng, d, n, s, 0.1)
    norms = np.exp2(rng.uniform(-140, 100, nb)).astype(np.float32)
    msg = _message(g, q, n, s, S, norms)
    flat = torch.full((d + 9,), 7.0, device=g.DEV)
    nuq.nuq_decode_accumulate([msg], d, n, s, S, 0.3, False, flat[shift + 4:shift + 4 + d])
    assert nuq.nuq_last_error_flags() == 0
    got = flat.cpu().numpy()
    want = (np.float64(np.float32(0.3)) * _value(q, n, s, norms)).astype(np.float32)
    np.testing.assert_array_equal(got[shift + 4:shift + 4 + d].view(np.uint32), want.view(np.uint32))
    assert (got[:shift + 4] == 7.0).all() and (got[shift + 4 + d:] == 7.0).all()


@pytest.mark.parametrize("update", ["write", "add", "momentum"])
@pytest.mark.parametrize("n,S,K,d", [(1000, 256, 2, 9000), (1000, 256, 2, 8009), (1001, 128, 3, 6006), (512, 512, 4, 512 * 17), (512, 256, 2, 512 * 16 + 259),
                                     (256, 256, 2, 256 * 33 + 2), (2048, 512, 2, 2048 * 5 + 6), (1024, 512, 4, 1024 * 9), (20000, 256, 4, 40_004),
                                     (4100, 256, 2, 8200), (512, 512, 4, 512 * 2050 + 2), (512, 256, 2, 512 * 2052 + 258)])
def test_tiles_that_are_not_full(g, n, S, K, d, update):
    """Tiles of 2048 and of 4096 coordinates that small buckets do not fill, of few or of no float4 groups, and both tile sizes'
    lines: the result of each way of applying a tile."""
    nuq = g.nuq
    rng = np.random.default_rng(n + d)
    s, nb = 3, -(-d // n)
    qs = [_dense_bytes(rng, d, n, s, 0.2) for _ in range(K)]
    norms = [np.exp2(rng.uniform(-3, 3, nb)).astype(np.float32) for _ in range(K)]
    msgs = [_message(g, q, n, s, S, v) for q, v in zip(qs, norms)]
    r = (0.5 * sum(_value(q, n, s, v) for q, v in zip(qs, norms))).astype(np.float32)
    w0, y0 = rng.standard_normal((2, d + 8)).astype(np.float32)
    w, y = torch.from_numpy(w0.copy()).to(g.DEV), torch.from_numpy(y0.copy()).to(g.DEV)
    if update == "momentum":
        nuq.nuq_decode_momentum_step(msgs, d, n, s, S, 0.5, 0.25, 0.5, 1.0, w[:d], y[:d])
        g64 = r.astype(np.float64)
        yl = w0[:d].astype(np.float64) - 0.25 * g64
        want = (w0[:d].astype(np.float64) - 0.25 * g64) + 0.5 * (yl - y0[:d].astype(np.float64))
        np.testing.assert_allclose(y.cpu().numpy()[:d], yl, rtol=2.0 ** -23, atol=2.0 ** -30)      # one rounding to fp32
        np.testing.assert_allclose(w.cpu().numpy()[:d], want, rtol=2.0 ** -23, atol=2.0 ** -30)
    else:
        nuq.nuq_decode_accumulate(msgs, d, n, s, S, 0.5, update == "add", w[:d])
        np.testing.assert_array_equal(w.cpu().numpy()[:d], r + w0[:d] if update == "add" else r)
    np.testing.assert_array_equal(w.cpu().numpy()[d:], w0[d:])
    np.testing.assert_array_equal(y.cpu().numpy()[d:], y0[d:])
    assert nuq.nuq_last_error_flags() == 0


@pytest.mark.parametrize("update", ["write", "add", "momentum"])
@pytest.mark.parametrize("n,K,d", [(1, 1, 203), (1, 3, 1000), (1, 16, 67), (3, 5, 2005), (8, 4, 4100), (8, 16, 4104), (33, 8, 9002), (100, 16, 3000)])
def test_tiles_of_few_groups(g, n, K, d, update):
    """Tiles of a few coordinates up to a few float4 groups per lane (so many workers, or so small buckets, that a tile's bit
    strings are its limit): none, one or both halves of the output stage."""
    nuq = g.nuq
    rng = np.random.default_rng(n + d)
    s, S, nb = 3, 64, -(-d // n)
    qs = [_dense_bytes(rng, d, n, s, 0.5) for _ in range(K)]
    norms = [np.exp2(rng.uniform(-3, 3, nb)).astype(np.float32) for _ in range(K)]
    msgs = [_message(g, q, n, s, S, v) for q, v in zip(qs, norms)]
    r = (0.5 * sum(_value(q, n, s, v) for q, v in zip(qs, norms))).astype(np.float32)
    w0, y0 = rng.standard_normal((2, d + 8)).astype(np.float32)
    w, y = torch.from_numpy(w0.copy()).to(g.DEV), torch.from_numpy(y0.copy()).to(g.DEV)
    if update == "momentum":
        nuq.nuq_decode_momentum_step(msgs, d, n, s, S, 0.5, 0.25, 0.5, 1.0, w[:d], y[:d])
        yl = w0[:d].astype(np.float64) - 0.25 * r.astype(np.float64)
        np.testing.assert_allclose(y.cpu().numpy()[:d], yl, rtol=2.0 ** -23, atol=2.0 ** -30)      # one rounding to fp32
        np.testing.assert_allclose(w.cpu().numpy()[:d], yl + 0.5 * (yl - y0[:d].astype(np.float64)), rtol=2.0 ** -23, atol=2.0 ** -30)
    else:
        nuq.nuq_decode_accumulate(msgs, d, n, s, S, 0.5, update == "add", w[:d])
        np.testing.assert_array_equal(w.cpu().numpy()[:d], r + w0[:d] if update == "add" else r)
    np.testing.assert_array_equal(w.cpu().numpy()[d:], w0[d:])
    np.testing.assert_array_equal(y.cpu().numpy()[d:], y0[d:])
    assert nuq.nuq_last_error_flags() == 0


@pytest.mark.parametrize("n,S,s,d", [(8192, 256, 3, (1 << 21) - 1), (8192, 256, 3, 1 << 21), (8192, 256, 4, 1 << 21), (8193, 256, 4, 1 << 21),
                                     (1000, 256, 2, 3_000_001), (512, 256, 2, 3_000_001), (4096, 64, 5, (1 << 22) - 1),
                                     (4096, 64, 5, 1 << 22), (513, 128, 7, 1_000_003), (700, 128, 7, 1_000_003), (2049, 256, 7, 1_000_003),
                                     (3000, 256, 7, 1_000_003), (600, 1024, 7, 1_000_003), (8192, 256, 1, (1 << 26) - 1),
                                     (8192, 256, 1, 1 << 26), (513, 128, 1, (1 << 26) + 5)])
def test_one_message_written_and_added(g, n, S, s, d):
    """Both sides of every line between the two decoders of a single written message: what it writes is what a zero vector holds
    after the message was added to it, which always takes the scattering decoder."""
    nuq = g.nuq
    gen = torch.Generator(device=g.DEV).manual_seed(n + s)
    q = torch.randint(1, s + 2, (d,), generator=gen, device=g.DEV, dtype=torch.uint8)
    q |= torch.randint(0, 2, (d,), generator=gen, device=g.DEV, dtype=torch.uint8) << 7
    q *= torch.rand(d, generator=gen, device=g.DEV) < 0.1
    nb = -(-d // n)
    m = nuq.Message(torch.rand(nb, generator=gen, device=g.DEV), torch.empty(nb + 1, dtype=torch.int64, device=g.DEV),
                    torch.zeros(d // 8 + 2 * nb + 64, dtype=torch.int32, device=g.DEV),
                    torch.empty(nb * nuq.nuq_num_sync(n, S), dtype=torch.int32, device=g.DEV))
    nuq.nuq_encode(q, n, s, S, m.bit_off, m.words, m.sync, g.workspace(d, n, s))
    written, added = torch.full((d,), 7.0, device=g.DEV), torch.zeros(d, device=g.DEV)
    nuq.nuq_decode_accumulate([m], d, n, s, S, 0.3, False, written)
    nuq.nuq_decode_accumulate([m], d, n, s, S, 0.3, True, added)
    assert nuq.nuq_last_error_flags() == 0
    assert torch.equal(written, added) and int((written != 0).sum()) == int((q != 0).sum())


@pytest.mark.parametrize("n,S,K,s,d", [(512, 128, 4, 7, 512 * 7300 + 100), (8192, 256, 8, 10, 8192 * 280 + 5), (1000, 256, 6, 10, 1000 * 1400),
                                       (4096, 256, 4, 14, 4096 * 1200), (2048, 128, 4, 10, 2048 * 1900)])
@pytest.mark.parametrize("update", [False, True])
def test_pieces_row_by_row_and_from_global_memory(g, n, S, K, s, d, update):
    """Pieces longer than a row on a full chip (row by row) and bucket range by bucket range (a wave per CU: from global memory)."""
    nuq = g.nuq
    gen = torch.Generator(device=g.DEV).manual_seed(d)
    B, nsync = nuq.nuq_num_buckets(d, n), nuq.nuq_num_sync(n, S)
    ws = torch.empty(nuq.nuq_encode_workspace_bytes(1, d, n, s), dtype=torch.uint8, device=g.DEV)
    msgs = []
    for k in range(K):
        v = torch.randn(d, generator=gen, device=g.DEV) * torch.rand(d, generator=gen, device=g.DEV) ** 4
        m = nuq.Message(torch.empty(B, device=g.DEV), torch.empty(B + 1, dtype=torch.int64, device=g.DEV),
                        torch.empty(nuq.nuq_max_words(d, n, s), dtype=torch.int32, device=g.DEV),
                        torch.empty(B * nsync, dtype=torch.int32, device=g.DEV))
        nuq.nuq_quantize_encode(v, n, s, k, S, m.norms, m.bit_off, m.words, m.sync, ws)
        msgs.append(m)
    assert float(msgs[0].bit_off[-1]) / 32 / (B * nsync) > 13              # words per piece
    prior = torch.randn(d, generator=gen, device=g.DEV)
    out, parts = prior.clone(), prior.clone()
    nuq.nuq_decode_accumulate(msgs, d, n, s, S, 1.0 / K, update, out)
    step = max(1, 200 * 2048 // n)
    for b in range(0, B, step):
        e = min(B, b + step)
        some = [nuq.Message(m.norms[b:e], m.bit_off[b:e + 1], m.words, m.sync[b * nsync:e * nsync]) for m in msgs]
        lo, hi = b * n, min(d, e * n)
        nuq.nuq_decode_accumulate(some, hi - lo, n, s, S, 1.0 / K, update, parts[lo:hi])
    assert torch.equal(out, parts)
    assert nuq.nuq_last_error_flags() == 0
