"""The launching calls through C++ (_nuq_calls) and through the checks and ctypes calls behind it: same results on any stream,
same errors, and the same objects accepted."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


class _Declines:
    def __getattr__(self, name):
        return lambda *a: None


def _step(g, d=40_003, K=3, n=1000, s=3, S=128, bucket_type=int):
    """One of every call on fixed inputs; all that they write."""
    nuq = g.nuq
    n = bucket_type(n)
    gen = torch.Generator(device=g.DEV).manual_seed(1)
    vs = [torch.randn(d, generator=gen, device=g.DEV) for _ in range(K)]
    seeds = [-1, 2 ** 70 + 5, 7][:K]
    B, empty = nuq.nuq_num_buckets(d, int(n)), lambda *sh, dt=torch.float32: torch.zeros(*sh, dtype=dt, device=g.DEV)
    ws = empty(max(nuq.nuq_encode_workspace_bytes(K, d, int(n), 14),
                   nuq.nuq_encode_huffman_batch_workspace_bytes(K, d, int(n), s)), dt=torch.uint8)
    outs = []

    def message(words, nsync):
        return nuq.Message(empty(B), empty(B + 1, dt=torch.int64), empty(words, dt=torch.int32),
                           empty(max(1, B * nsync), dt=torch.int32))

    def keep(*ts):
        outs.extend(t.clone() for t in ts)
    ms = [message(nuq.nuq_max_words(d, int(n), s), nuq.nuq_num_sync(int(n), S)) for _ in range(K)]
    out = empty(d)
    nuq.nuq_quantize_encode_batch(vs, n, s, seeds, S, ms, ws)
    nuq.nuq_decode_accumulate(ms, d, n, s, S, 1.0 / K, False, out)
    keep(out, *[t for m in ms for t in (m.norms, m.bit_off, m.words, m.sync)])
    nuq.nuq_decode_accumulate(ms, d, n, s, S, -1, True, out)                  # an int for a float
    w, yl = vs[0].clone(), vs[1].clone()
    nuq.nuq_decode_momentum_step(ms, d, n, s, S, 1.0 / K, 0.1, 0.9, 0.5, w, yl)
    keep(out, w, yl)
    lev = [0.0, 0.2, 0.4, 0.7, 1.0]
    nuq.nuq_quantize_encode_table_batch(vs, n, lev, nuq.NORM_LINF, seeds, S, ms, ws)
    nuq.nuq_decode_accumulate_table(ms, d, n, tuple(lev), S, 1.0 / K, False, out)
    keep(out, *[m.words for m in ms])
    norms = [empty(B) for _ in range(K)]
    packed = [empty(nuq.nuq_fixed_words(d, int(n), 4), dt=torch.int32) for _ in range(K)]
    nuq.nuq_quantize_pack_fixed_batch(vs, n, s, 4, seeds, norms, packed)
    nuq.nuq_unpack_accumulate_fixed(norms, packed, d, n, s, 4, 1.0 / K, False, out)
    keep(out, *packed)
    nuq.nuq_quantize_pack_fixed_table_batch(vs, n, lev, nuq.NORM_L2, 4, seeds, norms, packed)
    nuq.nuq_unpack_accumulate_fixed_table(norms, packed, d, n, lev, 4, 1.0 / K, False, out)
    keep(out, *packed)
    hm = [message(nuq.nuq_huffman_max_words(d, int(n)), nuq.nuq_huffman_num_sync(int(n), S)) for _ in range(K)]
    lengths = nuq.nuq_huffman_lengths([900, 80, 30, 8, 2], s)
    nuq.nuq_quantize_encode_huffman_batch(vs, n, s, seeds, S, lengths, hm, ws)
    nuq.nuq_decode_accumulate_huffman(hm, d, n, s, S, lengths, 1.0 / K, False, out)
    keep(out, *[m.words for m in hm])
    total, total_sq = empty(d, dt=torch.float64), empty(d, dt=torch.float64)
    nuq.nuq_moments_accumulate(out, total, total_sq)
    keep(total, total_sq)
    return outs


def test_same_results_as_the_general_way(g, monkeypatch):
    from paper_1908_06077_amd import binding
    fast = _step(g)
    with torch.cuda.stream(torch.cuda.Stream()):
        side = _step(g)
    torch.cuda.synchronize()
    odd = _step(g, bucket_type=np.int64)              # declined in C++, taken by ctypes
    monkeypatch.setattr(binding, "_calls", _Declines())
    slow = _step(g)
    for a, b, c, e in zip(fast, side, odd, slow):
        assert torch.equal(a, e) and torch.equal(b, e) and torch.equal(c, e)
    assert g.nuq.nuq_last_error_flags() == 0


def test_plain_calls_do_not_reach_the_general_way(g, monkeypatch):
    from paper_1908_06077_amd import binding

    class Refuses:
        def __getattr__(self, name):
            real = getattr(real_lib, name)
            if name.endswith("_batch") or "accumulate" in name or "momentum" in name:
                raise AssertionError(name)
            return real
    real_lib = binding._lib
    monkeypatch.setattr(binding, "_lib", Refuses())
    _step(g)


def test_the_same_errors(g):
    nuq = g.nuq
    d, n, s, S, K = 5000, 512, 3, 128, 2
    v = torch.randn(d, device=g.DEV)
    ws = torch.empty(nuq.nuq_encode_workspace_bytes(K, d, n, s), dtype=torch.uint8, device=g.DEV)
    ms = [g.alloc_message(d, n, s, S) for _ in range(K)]
    call = lambda **kw: nuq.nuq_quantize_encode_batch(**{**dict(vs=[v, v], bucket=n, s=s, seeds=[1, 2], sync_stride=S, messages=ms,
                                                               workspace=ws), **kw})
    call()
    call(vs=(torch.nn.Parameter(v, requires_grad=False), v))
    for error, kw in [(ValueError, dict(vs=[v, v[:-1]])), (ValueError, dict(vs=[v, v.double()])), (ValueError, dict(vs=[v, v.cpu()])),
                      (ValueError, dict(vs=[v, torch.randn(2 * d, device=g.DEV)[::2]])), (ValueError, dict(seeds=[1])),
                      (ValueError, dict(messages=ms[:1])), (nuq.NuqError, dict(s=15)), (nuq.NuqError, dict(sync_stride=100)),
                      (nuq.NuqError, dict(workspace=ws[:16])), (IndexError, dict(vs=[], seeds=[], messages=[])),
                      (ValueError, dict(messages=[ms[0], nuq.Message(ms[1].norms[:-1], ms[1].bit_off, ms[1].words, ms[1].sync)])),
                      (ValueError, dict(messages=[ms[0], nuq.Message(ms[1].norms, ms[1].bit_off, ms[1].words, None)])),
                      (nuq.NuqError, dict(vs=[v] * 33, seeds=[0] * 33, messages=ms[:1] * 33))]:
        with pytest.raises(error):
            call(**kw)
    out = torch.empty(d, device=g.DEV)
    with pytest.raises(ValueError):
        nuq.nuq_decode_accumulate(ms, d, n, s, S, 1.0, False, out[:-1])
    with pytest.raises(nuq.NuqError):
        nuq.nuq_decode_accumulate(ms, d, n, 0, S, 1.0, False, out)
    with pytest.raises(Exception):                    # a batched tensor has no address
        torch.vmap(lambda x: nuq.nuq_moments_accumulate(x, out.double(), out.double()) or x)(torch.randn(2, d, device=g.DEV))
    torch.cuda.synchronize()
    assert g.nuq.nuq_last_error_flags() == 0
