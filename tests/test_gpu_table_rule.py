"""The level-table quantizer's fp32 rule where it can go wrong, bit for bit against the oracle's real-number rule:
coordinates planted on, one unit above and one unit below their own rounding threshold (the rule must notice that it
cannot tell and hand them to the fp64 rule), coordinates on the levels themselves, buckets whose bins reach the subnormals
(fp64 rule throughout), and level tables whose lowest bins are tiny.  One size per shape of thread team, with short last
buckets."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


CASES = [
    # (d, bucket, kind, s, p, norm)
    (3_001, 512, "uniform", 3, 0.0, 1.0),
    (3_001, 300, "exp", 7, 0.3, 3e-7),
    (9_001, 2048, "exp", 14, 0.05, 2.5),
    (9_001, 1000, "uniform", 14, 0.0, 7e33),
    (30_001, 8192, "uniform", 3, 0.0, 0.37),
    (30_001, 8192, "exp", 14, 0.01, 1e-20),
    (40_001, 16384, "exp", 1, 0.9, 1.0),
    (70_001, 32768, "uniform", 6, 0.0, 1e-3),
    (9_001, 2048, "uniform", 3, 0.0, 1e-36),
    (3_001, 512, "exp", 4, 0.3, 1e-40),
]


def planted(d, n, kind, s, p, norm):
    """Levels, seed, coordinates on or beside their own rounding threshold or on a level, norms (the maximum of each bucket)."""
    lev = workloads.level_table(kind, s, p) if kind == "uniform" else [0.0] + [float(np.float32(p ** (s + 1 - j))) for j in range(1, s + 2)]
    rng = np.random.default_rng(d + n + s)
    seed, B = int(rng.integers(1 << 60)), oracle.num_buckets(d, n)
    N = np.float32(norm)
    u = oracle.rng_fill(seed, d, n).astype(np.float64)
    e = np.array(lev, dtype=np.float32).astype(np.float64) * float(N)
    j = rng.integers(0, s + 1, d)
    tie = (e[j] + u * (e[j + 1] - e[j]) * 2.0 ** -24).astype(np.float32)
    v = np.where(rng.random(d) < 0.1, e[j].astype(np.float32), tie)
    ulp = rng.integers(-1, 2, d)
    v = np.where(ulp > 0, np.nextafter(v, np.float32(np.inf)), np.where(ulp < 0, np.nextafter(v, np.float32(0)), v))
    v = (np.minimum(v, N) * rng.choice([-1.0, 1.0], d)).astype(np.float32)
    v[::n] = N                                        # the maximum norm of every bucket is N
    norms_np = np.full(B, N, dtype=np.float32)
    return lev, seed, v, norms_np


@pytest.mark.parametrize("d,n,kind,s,p,norm", CASES)
def test_planted_near_ties(g, d, n, kind, s, p, norm):
    nuq = g.nuq
    lev, seed, v, norms_np = planted(d, n, kind, s, p, norm)
    B = norms_np.size
    want = oracle.quantize_table(v, n, lev, seed, norms_np)
    vt = torch.from_numpy(v).to(g.DEV)
    q = torch.full((d,), 0x7F, dtype=torch.uint8, device=g.DEV)
    nuq.nuq_quantize_table(vt, n, lev, seed, torch.from_numpy(norms_np).to(g.DEV), q)
    np.testing.assert_array_equal(q.cpu().numpy(), want)
    # the fused front (its rows are decided in registers, the doubtful ones again from memory), as fixed-width codes
    b = 5
    norms = torch.empty(B, dtype=torch.float32, device=g.DEV)
    packed = torch.full((nuq.nuq_fixed_words(d, n, b),), -1, dtype=torch.int32, device=g.DEV)
    nuq.nuq_quantize_pack_fixed_table_batch([vt], n, lev, nuq.NORM_LINF, b, [seed], [norms], [packed])
    np.testing.assert_array_equal(norms.cpu().numpy(), norms_np)
    np.testing.assert_array_equal(g.u32(packed), oracle.pack_fixed(want, n, s, b))
    assert nuq.nuq_last_error_flags() == 0


@pytest.mark.parametrize("d,n,kind,s,p,norm", CASES)
def test_planted_near_ties_where_a_row_is_put_twice(g, d, n, kind, s, p, norm):
    """The fused kernels that hand a row's bytes on before they know that it is decided again: fixed width at 4 bits (codes in
    registers) and at 8 (words in memory), and the bit strings (bytes in the coding phase's format)."""
    nuq = g.nuq
    lev, seed, v, norms_np = planted(d, n, kind, s, p, norm)
    want = oracle.quantize_table(v, n, lev, seed, norms_np)
    vt = torch.from_numpy(v).to(g.DEV)
    for b in (4, 8):
        if s + 2 > 1 << (b - 1):
            continue
        norms = torch.empty(norms_np.size, dtype=torch.float32, device=g.DEV)
        packed = torch.full((nuq.nuq_fixed_words(d, n, b),), -1, dtype=torch.int32, device=g.DEV)
        nuq.nuq_quantize_pack_fixed_table_batch([vt], n, lev, nuq.NORM_LINF, b, [seed], [norms], [packed])
        np.testing.assert_array_equal(norms.cpu().numpy(), norms_np)
        np.testing.assert_array_equal(g.u32(packed), oracle.pack_fixed(want, n, s, b))
    S = 128
    m = g.alloc_message(d, n, s, S)
    nuq.nuq_quantize_encode_table_batch([vt], n, lev, nuq.NORM_LINF, [seed], S, [m], g.workspace(d, n, s))
    bo, words, sync = oracle.encode(want, n, s, S)
    np.testing.assert_array_equal(m.norms.cpu().numpy(), norms_np)
    np.testing.assert_array_equal(g.u64(m.bit_off), bo)
    np.testing.assert_array_equal(g.u32(m.words)[: words.size], words)
    np.testing.assert_array_equal(g.u32(m.sync)[: sync.size], sync)
    assert nuq.nuq_last_error_flags() == 0


@pytest.mark.parametrize("n", [300, 512, 2048, 8192, 20000])
@pytest.mark.parametrize("kind,s", [("uniform", 3), ("exp", 7), ("uniform", 14)])
@pytest.mark.parametrize("scale", [0.01, 0.5])
def test_infinite_and_nan_coordinates_under_a_finite_norm(g, n, kind, s, scale):
    """A norm that the caller supplies need not see what the vector holds: an infinite coordinate takes the top level, a
    NaN level 0.  Beside coordinates that all lie in the first bin and beside ones that do not."""
    nuq, d = g.nuq, 3 * n + 17
    lev = workloads.level_table(kind, s, 0.3)
    rng = np.random.default_rng(n + s)
    v = (rng.uniform(-1.0, 1.0, d) * scale * lev[1]).astype(np.float32)
    if scale > 0.1:
        v[::5] = rng.uniform(-1.0, 1.0, v[::5].size)
    at = rng.permutation(d)[:48].reshape(6, 8)
    for a, x in zip(at, (np.inf, -np.inf, np.nan, -np.nan, 0.0, 1.0)):
        v[a] = x
    v.view(np.uint32)[at[2][:4]] = 0x7FA00001                  # signaling
    norms = np.ones(oracle.num_buckets(d, n), dtype=np.float32)
    q = torch.full((d,), 0x7F, dtype=torch.uint8, device=g.DEV)
    nuq.nuq_quantize_table(torch.from_numpy(v).to(g.DEV), n, lev, n, torch.from_numpy(norms).to(g.DEV), q)
    want = oracle.quantize_table(v, n, lev, n, norms)
    assert want[at[0]].min() == s + 1 and not want[at[2]].any()
    np.testing.assert_array_equal(q.cpu().numpy(), want)
    assert nuq.nuq_last_error_flags() == 0


@pytest.mark.parametrize("n", [60, 512, 2048, 8192, 32768])
@pytest.mark.parametrize("kind,s", [("uniform", 3), ("exp", 7)])
def test_dead_buckets_beside_live_ones(g, n, kind, s):
    """Buckets of zeros, and buckets whose norm is infinite or NaN, among buckets with planted near-ties (four to a wave where
    buckets are small)."""
    nuq, B = g.nuq, 23
    d = B * n - n // 3
    lev, seed, v, norms_np = planted(d, n, kind, s, 0.3, 0.7)
    for b in (0, 3, 5, 8, 9, 10, 11, 13, 22):
        v[b * n:(b + 1) * n] = 0.0
        norms_np[b] = 0.0
    vt = torch.from_numpy(v).to(g.DEV)
    want = oracle.quantize_table(v, n, lev, seed, norms_np)
    norms = torch.empty(B, dtype=torch.float32, device=g.DEV)
    packed = torch.full((nuq.nuq_fixed_words(d, n, 5),), -1, dtype=torch.int32, device=g.DEV)
    nuq.nuq_quantize_pack_fixed_table_batch([vt], n, lev, nuq.NORM_LINF, 5, [seed], [norms], [packed])
    np.testing.assert_array_equal(norms.cpu().numpy(), norms_np)
    np.testing.assert_array_equal(g.u32(packed), oracle.pack_fixed(want, n, s, 5))
    assert nuq.nuq_last_error_flags() == 0
    norms_np[[2, 12]], norms_np[14] = np.inf, np.nan
    for b in (2, 12, 14):
        want[b * n:(b + 1) * n] = 0
    q = torch.full((d,), 0x7F, dtype=torch.uint8, device=g.DEV)
    nuq.nuq_quantize_table(vt, n, lev, seed, torch.from_numpy(norms_np).to(g.DEV), q)
    np.testing.assert_array_equal(q.cpu().numpy(), want)


@pytest.mark.parametrize("n", [1000, 2048, 8192])
@pytest.mark.parametrize("s", [1, 2, 3, 4, 5, 6, 7, 8, 11, 12, 13, 14])
def test_rows_that_end_at_every_level(g, s, n):
    """Rows (a wave's 256 coordinates) whose largest coordinate is on, just above or just below each level in turn: both ways of
    leaving out the levels that no coordinate of a row reaches, in the standalone quantizer and in the pack, either norm."""
    nuq = g.nuq
    rng = np.random.default_rng(s + n)
    d = 5 * n + 3
    for kind in ("uniform", "exp"):
        lev = [0.0] + [float(np.float32(j / (s + 1) if kind == "uniform" else 0.4 ** (s + 1 - j))) for j in range(1, s + 2)]
        table = np.array(lev, dtype=np.float32)
        top = np.repeat(table[rng.integers(1, s + 2, -(-d // 256))], 256)[:d]
        v = (top * rng.random(d)).astype(np.float32)
        v[::256] = np.nextafter(top[::256], np.where(rng.random(v[::256].size) < 0.5, 0, 2).astype(np.float32))
        v[128::256] = np.where(rng.random(v[128::256].size) < 0.5, top[128::256], v[128::256])
        v = np.minimum(v, np.float32(1.0)) * rng.choice([-1.0, 1.0], d).astype(np.float32)
        v[::n] = 1.0
        vt = torch.from_numpy(v).to(g.DEV)
        B = nuq.nuq_num_buckets(d, n)
        norms, q = torch.empty(B, device=g.DEV), torch.empty(d, dtype=torch.uint8, device=g.DEV)
        for norm in (nuq.NORM_LINF, nuq.NORM_L2):
            packed = torch.zeros(nuq.nuq_fixed_words(d, n, 8), dtype=torch.int32, device=g.DEV)
            nuq.nuq_quantize_pack_fixed_table_batch([vt], n, lev, norm, 8, [5], [norms], [packed])
            want = oracle.quantize_table(v, n, table, 5, norms.cpu().numpy())
            np.testing.assert_array_equal(g.u32(packed), oracle.pack_fixed(want, n, s, 8))
            nuq.nuq_quantize_table(vt, n, lev, 5, norms, q)
            np.testing.assert_array_equal(q.cpu().numpy(), want)
    assert nuq.nuq_last_error_flags() == 0
