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
