"""Fixed-width coding at 4 and 8 bits, where pack and unpack go between registers and memory without an LDS phase: sizes
at the edges of that route, against the oracle as in test_gpu_fixed.py (packed words bit-exact, averages within the bar)."""
import numpy as np
import pytest
import torch

import test_gpu_fixed as fixed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("d,n,s,b,K,kind", [
    (5_001, 1000, 3, 4, 3, "mixed"),      # a wave's rows cross buckets; last float4 group cut
    (2_600, 600, 3, 4, 2, "mixed"),       # odd number of rows: the last row has no partner
    (45_001, 20_000, 6, 4, 5, "gauss"),   # five rows of a 1024-thread team
    (64, 8, 2, 4, 1, "mixed"),            # one word per bucket
    (7, 8, 2, 4, 2, "edges"),             # less than a word
    (900, 300, 5, 8, 4, "mixed"),
    (4_099, 4, 14, 8, 1, "mixed"),        # one word per bucket; too many tables for LDS: the other kernel
    (12_345, 512, 6, 4, 8, "mixed"),      # tables exactly fill their LDS
    (12_345, 512, 6, 4, 9, "mixed"),      # ... and one worker more: the other kernel
    (70_001, 8192, 3, 4, 12, "gauss"),    # more workers than words in flight at once
    (70_001, 4096, 14, 8, 17, "gauss"),
    (8_192 * 3 + 513, 8192, 3, 4, 2, "gauss"),   # the last wave holds one coordinate of its second row
    (33_000, 32768, 14, 8, 2, "mixed"),
    (12_289, 8192, 6, 8, 1, "gauss"),     # one and two workers: all words of a wave requested at once
    (4_096 * 2 + 769, 512, 6, 8, 2, "mixed"),
    (30_001, 1000, 9, 8, 2, "mixed"),
    (30_001, 1000, 9, 8, 1, "edges"),
    (1_022, 1022, 3, 4, 2, "mixed"),      # buckets that are not whole words: the other kernel unpacks
])
def test_sizes_at_the_edges(g, d, n, s, b, K, kind):
    fixed.test_pack_fused_pack_and_unpack_average(g, d, n, s, b, K, kind)


@pytest.mark.parametrize("n", [64, 512, 2048, 8192, 20000])
def test_levels_above_the_top(g, n):
    """Level indices from 8 up do not fit four bits (the caller's error): bit 3 is OR-ed with the sign, as it is at the widths
    that go through LDS."""
    nuq, d = g.nuq, 2 * n + 40
    rng = np.random.default_rng(n)
    q = rng.integers(0, 16, d)
    q |= np.where(q > 0, rng.integers(0, 2, d) << 7, 0)
    packed = torch.full((nuq.nuq_fixed_words(d, n, 4),), -1, dtype=torch.int32, device=g.DEV)
    nuq.nuq_pack_fixed(torch.from_numpy(q.astype(np.uint8)).to(g.DEV), n, 3, 4, packed)
    codes = np.zeros(3 * n, dtype=np.uint32)
    codes[:d] = ((q >> 4) & 8) | (q & 15)
    want = (codes.reshape(-1, 8) << np.arange(28, -1, -4, dtype=np.uint32)).sum(axis=1, dtype=np.uint32)
    np.testing.assert_array_equal(g.u32(packed), want)
