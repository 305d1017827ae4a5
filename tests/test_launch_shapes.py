"""Launch shapes, asked of the library (no GPU): the LDS lists of the ERC encoders hold what buckets have, their buffers the longest
string of what is listed; the decoder's tiles."""
import numpy as np
import pytest

import oracle
import paper_1908_06077_amd as nuq


def erc_bits(x):
    return 1 if x == 1 else erc_bits(x.bit_length() - 1) + x.bit_length()


@pytest.mark.parametrize("n", [1, 3, 17, 64, 200, 256, 257, 300, 350, 400, 450, 512, 513, 600, 768, 769, 1000, 1024, 1025, 1500, 2048])
def test_longest_string_of_a_listed_bucket(n):
    """Every record at the longest level code, gaps spread so that their codes are longest: pairs first (ERC(2) takes 3 bits for two
    coordinates), what is left over single."""
    for mode in (0, 1):
        for s in range(1, 15):
            for nb in (1, 20_000):
                _, listed, buffer, whole = nuq.nuq_encode_shape(mode, 1, nb * n, n, s, 64)
                level = 7 if mode == 1 else max(erc_bits(j) for j in range(1, s + 2))
                slot = (n * (2 + max(erc_bits(j) for j in range(1, s + 2))) + 31) // 32
                pairs = min(listed, n - listed)
                longest = (listed * (1 + level) + 3 * pairs + (listed - pairs) + 31) // 32
                assert buffer >= min(longest, slot) and whole >= slot


@pytest.mark.parametrize("law", ["gauss", "heavy"])
@pytest.mark.parametrize("n,levels", [(260, range(1, 15)), (300, range(1, 15)), (350, range(1, 15)), (400, range(1, 6)),
                                      (450, range(1, 6)), (500, range(1, 5)), (512, range(1, 5)), (768, range(1, 15)), (780, range(1, 15)),
                                      (832, range(1, 15)), (1000, range(1, 15))])
def test_lists_hold_what_buckets_have(n, levels, law):
    rng = np.random.default_rng(n)
    rows = 200
    v = rng.standard_normal((rows, n))
    if law == "heavy":
        v = v / np.sqrt(rng.chisquare(3, v.shape) / 3.0)
    v = v.astype(np.float32).ravel()
    norms = oracle.bucket_norms(v, n).astype(np.float32)
    for s in levels:
        nonzeros = np.count_nonzero(oracle.quantize(v, n, s, 1, norms).reshape(rows, n), axis=1)
        for mode in (0, 1):
            for S in (64, 128, 512):
                listed = nuq.nuq_encode_shape(mode, 4, 4_000_000, n, s, S)[1]
                assert np.mean(nonzeros <= listed) > 0.97, (s, mode, S, listed, nonzeros.mean())


@pytest.mark.parametrize("n", [12288, 12289, 14336, 15000, 16000, 16384, 20000])
def test_lists_of_large_buckets(n):
    """A quarter of the bucket where nonzeros are anyone's guess (bytes) or five workgroups leave room for it, little less
    elsewhere."""
    for s in range(1, 15):
        for S in (0, 64, 256):
            assert nuq.nuq_encode_shape(1, 1, 9 * n, n, s, S)[1] == n // 4
            listed, buffer = nuq.nuq_encode_shape(0, 1, 9 * n, n, s, S)[1:3]
            assert listed == n // 4 or (n > 15000 and n // 4 - 290 < listed < n // 4)
            index = max(256, nuq.nuq_num_sync(n, S)) - (-n // 2048) + 2
            words = ((n + 1023) // 1024) * 256 + (listed + 1) // 2 + buffer + index + 64 + 512
            assert n <= 12288 or n > 16384 or 5 * (-(-4 * words // 1280)) <= 128                   # of 128 pieces of 1280 bytes


def test_decode_tiles():
    """Large buckets: 4096 coordinates where pieces may hold more than 128 records (64 in large messages), which no piece of fewer
    coordinates does, and the lanes are at most half full; level tables, whose density nothing is known of, in any case."""
    for n in (4096, 8192, 20000, 32768):
        for s in range(1, 15):
            for d, most in ((65_537, 128), (1 << 24, 64)):
                for K in (1, 2, 4, 8):
                    for S in (64, 128, 256, 512, 1024):
                        dense = S * min(1.0, 0.8 * 2 ** s / n ** 0.5) > most
                        few = K * 2048 // S <= 32
                        for update in (0, 1, 2):
                            assert nuq.nuq_decode_tile(K, d, n, s, S, False, update) == (4096 if few and dense else 2048)
                        assert nuq.nuq_decode_tile(K, d, n, s, S, True) == (4096 if few else 2048)
    assert nuq.nuq_decode_tile(4, 1 << 24, 512, 3, 512) == 4096 and nuq.nuq_decode_tile(4, 1 << 24, 512, 3, 512, update=2) == 2048
    assert nuq.nuq_decode_tile(4, 1 << 18, 512, 3, 512) == 2048 and nuq.nuq_decode_tile(1, 1 << 24, 1000, 3, 512) == 2048
    assert nuq.nuq_decode_tile(4, 1 << 24, 8192, 3, 0) == 2048 and nuq.nuq_decode_tile(0, 1 << 24, 8192, 3, 256) == 0
