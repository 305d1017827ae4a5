"""The fused encoder and the fixed-width pack on both sides of every line between two team shapes: bucket sizes that fill every
row of a team or leave some empty, a last bucket of a few coordinates, gradients at an odd address."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

SIZES = [3, 4, 60, 255, 256, 257, 512, 513, 700, 1024, 1025, 2048, 2049, 4093, 4096, 4097, 8192, 8193, 16384, 16385, 24576, 24577, 32768]


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def _vector(n, tail, s):
    rng = np.random.default_rng(n + tail + s)
    v = rng.standard_normal(3 * n + tail).astype(np.float32)
    v[: n // 2] *= 2.0 ** -100                       # half a bucket far below the rest
    v[n: 2 * n] *= np.float32(2.0 ** -130)           # a bucket whose norm takes the fp64 way
    return v


@pytest.mark.parametrize("tail,shift", [(0, 0), (1, 1), (3, 0), (5, 1)])
@pytest.mark.parametrize("n", SIZES)
def test_messages(g, n, tail, shift):
    for s in (3, 7):
        v_np = _vector(n, tail, s)
        d, S = v_np.size, 64 if n >= 64 else 0
        v = torch.empty(d + shift, device=g.DEV)[shift:].copy_(torch.from_numpy(v_np))
        m = g.fused_encode(v, n, s, 5, S)
        g.check_norms(v_np, n, m.norms.cpu().numpy())
        g.check_message_against_oracle(v_np, n, s, 5, S, m)
        assert g.nuq.nuq_last_error_flags() == 0


@pytest.mark.parametrize("n", SIZES)
def test_packed_and_maximum_norm(g, n):
    nuq, s, tail = g.nuq, 3, 2
    v_np = _vector(n, tail, s)
    d = v_np.size
    v = torch.from_numpy(v_np).to(g.DEV)
    B, levels = nuq.nuq_num_buckets(d, n), np.array([j / 4 for j in range(5)], dtype=np.float32)
    norms = torch.empty(B, device=g.DEV)
    for b in (4, 8):
        packed = torch.zeros(nuq.nuq_fixed_words(d, n, b), dtype=torch.int32, device=g.DEV)
        nuq.nuq_quantize_pack_fixed_batch([v], n, s, b, [5], [norms], [packed])
        want = oracle.pack_fixed(oracle.quantize(v_np, n, s, 5, norms.cpu().numpy()), n, s, b)
        np.testing.assert_array_equal(g.u32(packed), want)
        nuq.nuq_quantize_pack_fixed_table_batch([v], n, levels.tolist(), nuq.NORM_LINF, b, [5], [norms], [packed])
        np.testing.assert_array_equal(norms.cpu().numpy(), oracle.bucket_norms_linf(v_np, n))
        want = oracle.pack_fixed(oracle.quantize_table(v_np, n, levels, 5, norms.cpu().numpy()), n, s, b)
        np.testing.assert_array_equal(g.u32(packed), want)
    S = 64 if n >= 64 else 0
    m = g.alloc_message(d, n, s, S)
    nuq.nuq_quantize_encode_table_batch([v], n, levels.tolist(), nuq.NORM_LINF, [5], S, [m], g.workspace(d, n, s))
    bo, words, sync = oracle.encode(oracle.quantize_table(v_np, n, levels, 5, m.norms.cpu().numpy()), n, s, S)
    np.testing.assert_array_equal(g.u64(m.bit_off), bo)
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    if sync.size:
        np.testing.assert_array_equal(g.u32(m.sync)[: sync.size], sync)


def _many_buckets(nb, n):
    """nb buckets, the last of five coordinates: zero ones, tiny ones (the norm's fp64 way), others of all magnitudes."""
    rng = np.random.default_rng(nb + n)
    d = (nb - 1) * n + 5
    scale = np.exp2(rng.uniform(-10, 10, nb))
    scale[::7], scale[1::11] = 0.0, 2.0 ** -130
    return (rng.standard_normal(d) * np.repeat(scale, n)[:d]).astype(np.float32)


# (coding, s or levels, bucket, buckets of all workers from which a team has half the threads)
UNIFORM7, UNIFORM3 = [j / 8 for j in range(9)], [j / 4 for j in range(5)]
LINES = [("erc", 3, 513, 5120), ("erc", 7, 600, 5120), ("erc", 5, 832, 5120), ("erc", 3, 833, 5120), ("erc", 3, 1024, 5120),
         ("erc", 3, 2049, 2048), ("erc", 6, 2049, 4096), ("erc", 3, 4096, 2048), ("erc", 3, 16385, 257), ("erc", 7, 20000, 257),
         ("erc", 14, 24577, 257), ("erc", 3, 32768, 257), ("linf", UNIFORM3, 700, 5120), ("linf", UNIFORM7, 2050, 8192),
         ("l2", UNIFORM7, 3000, 2048), ("linf", UNIFORM3, 16390, 257), ("huffman", 3, 600, 5120), ("huffman", 7, 1023, 8192),
         ("huffman", 3, 3000, 4096), ("huffman", 7, 16385, 1024), ("huffman", 3, 24576, 1024), ("pack", UNIFORM3, 520, 8192),
         ("pack", UNIFORM3, 700, 32768), ("pack", UNIFORM7, 4096, 8192)]


@pytest.mark.parametrize("coding,code,n,line", LINES)
def test_messages_of_both_shapes(g, coding, code, n, line):
    """One gradient by itself, in a batch just below the line and in one at it: the same bits, norms included (a norm is a sum of
    fp32 partial sums, in an order that the shapes share), and the norm of nuq_bucket_norms."""
    nuq = g.nuq
    s = code if isinstance(code, int) else len(code) - 2
    nb = -(-line // 32)
    at = -(-line // nb)                                      # workers at the line; one fewer: below it
    assert nb * (at - 1) < line <= nb * at <= 32 * nb
    v_np, S = _many_buckets(nb, n), 256
    d = v_np.size
    v = torch.empty(d + 1, device=g.DEV)[1:].copy_(torch.from_numpy(v_np))
    kind = nuq.NORM_LINF if coding in ("linf", "pack") else nuq.NORM_L2
    lengths = nuq.nuq_huffman_lengths([1 << (s + 1 - j) for j in range(s + 2)], s)
    zeros = lambda size, dt: torch.zeros(size, dtype=dt, device=g.DEV)
    if coding == "huffman":
        sizes = (nuq.nuq_huffman_max_words(d, n), nb * nuq.nuq_huffman_num_sync(n, S),
                 nuq.nuq_encode_huffman_batch_workspace_bytes(at, d, n, s))
    else:
        sizes = nuq.nuq_max_words(d, n, s), nb * nuq.nuq_num_sync(n, S), nuq.nuq_encode_workspace_bytes(at, d, n, s)
    ws = zeros(sizes[2], torch.uint8)

    def first(K):
        ms = [nuq.Message(torch.full((nb,), -1.0, device=g.DEV), zeros(nb + 1, torch.int64), zeros(sizes[0], torch.int32),
                          zeros(max(1, sizes[1]), torch.int32)) for _ in range(K)]
        vs, seeds = [v] * K, [5] * K
        if coding == "erc":
            nuq.nuq_quantize_encode_batch(vs, n, s, seeds, S, ms, ws)
        elif coding == "huffman":
            nuq.nuq_quantize_encode_huffman_batch(vs, n, s, seeds, S, lengths, ms, ws)
        elif coding == "pack":
            out = [zeros(2 * nuq.nuq_fixed_words(d, n, 8), torch.int32) for _ in range(K)]
            for b in (5, 8):
                nuq.nuq_quantize_pack_fixed_table_batch(vs, n, code, kind, b, seeds, [m.norms for m in ms], out)
                ms = [nuq.Message(m.norms, m.bit_off, o.clone(), m.sync) for m, o in zip(ms, out)]
        else:
            nuq.nuq_quantize_encode_table_batch(vs, n, code, kind, seeds, S, ms, ws)
        for m in ms[1:]:                                     # every worker's message is the same
            assert all(torch.equal(a, b) for a, b in zip((m.norms, m.bit_off, m.words, m.sync),
                                                         (ms[0].norms, ms[0].bit_off, ms[0].words, ms[0].sync)))
        return ms[0]

    norms = torch.empty(nb, device=g.DEV)
    (nuq.nuq_bucket_norms_linf if kind == nuq.NORM_LINF else nuq.nuq_bucket_norms)(v, n, norms)
    alone = first(1)
    assert torch.equal(alone.norms, norms)
    for K in (at - 1, at):
        m = first(K)
        assert torch.equal(m.norms, norms)
        assert torch.equal(m.bit_off, alone.bit_off) and torch.equal(m.words, alone.words) and torch.equal(m.sync, alone.sync)
    assert nuq.nuq_last_error_flags() == 0


@pytest.mark.parametrize("n,line", [(513, 8192), (640, 8192), (832, 32768), (1000, 5120), (2049, 2048), (16385, 257)])
def test_single_vectors_of_both_shapes(g, n, line):
    """Norms, quantizers, the coders and the pack of given bytes: a vector at the line and its beginning, below the line."""
    nuq, s, S = g.nuq, 3, 256
    v = torch.from_numpy(_many_buckets(line, n)).to(g.DEV)
    lengths, levels = [1, 2, 3, 4, 4], UNIFORM3

    def run(v):
        d = v.numel()
        nb, e = nuq.nuq_num_buckets(d, n), lambda size, dt: torch.zeros(size, dtype=dt, device=g.DEV)
        n2, ninf, q, qt = e(nb, torch.float32), e(nb, torch.float32), e(d, torch.uint8), e(d, torch.uint8)
        nuq.nuq_bucket_norms(v, n, n2)
        nuq.nuq_bucket_norms_linf(v, n, ninf)
        nuq.nuq_quantize(v, n, s, 5, n2, q)
        nuq.nuq_quantize_table(v, n, levels, 5, ninf, qt)
        packed = e(nuq.nuq_fixed_words(d, n, 4), torch.int32)
        nuq.nuq_pack_fixed(q, n, s, 4, packed)
        bo, words, sync = e(nb + 1, torch.int64), e(nuq.nuq_max_words(d, n, s), torch.int32), e(nb * nuq.nuq_num_sync(n, S), torch.int32)
        nuq.nuq_encode(q, n, s, S, bo, words, sync, g.workspace(d, n, s))
        hbo, hwords = e(nb + 1, torch.int64), e(nuq.nuq_huffman_max_words(d, n), torch.int32)
        hsync = e(nb * nuq.nuq_huffman_num_sync(n, S), torch.int32)
        nuq.nuq_encode_huffman(q, n, s, S, lengths, hbo, hwords, hsync,
                               e(nuq.nuq_encode_huffman_workspace_bytes(d, n), torch.uint8))
        return [n2, ninf, q, qt, packed, bo, sync, hbo, hsync], [(bo, words), (hbo, hwords)]

    (whole, strings), (start, start_strings) = run(v), run(v[: (line - 1) * n])
    for a, b in zip(whole, start):
        assert torch.equal(a[: b.numel()], b)
    for (_, a), (bo, b) in zip(strings, start_strings):
        used = int(bo[-1].item()) // 32                      # the last word is shared with the next bucket's padding
        assert torch.equal(a[:used], b[:used])
    assert nuq.nuq_last_error_flags() == 0
