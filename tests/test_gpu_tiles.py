"""DECODE of large buckets on both sides of the line between tiles of 2048 and of 4096 coordinates, written, added and with the
momentum rule, against the oracle; short last buckets that end inside a tile."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("K", [2, 4])
@pytest.mark.parametrize("n,s,S,tile", [(8192, 3, 256, 2048), (8192, 5, 256, 2048), (8192, 6, 256, 4096), (4096, 3, 512, 2048),
                                        (4096, 7, 128, 2048), (4096, 7, 256, 4096), (5000, 14, 256, 4096), (20000, 7, 128, 2048),
                                        (16384, 7, 256, 4096), (16384, 5, 512, 2048), (16384, 6, 512, 4096), (5000, 2, 1024, 2048)])
def test_parts_of_large_buckets(g, n, s, S, tile, K):
    nuq, d = g.nuq, 3 * n + 2049
    assert nuq.nuq_decode_tile(K, d, n, s, S) == tile
    vs = [torch.randn(d, device=g.DEV, generator=torch.Generator(device=g.DEV).manual_seed(9 * n + k)) for k in range(K)]
    msgs = [g.fused_encode(v, n, s, 70 + k, S) for k, v in enumerate(vs)]
    host = [(m.norms.cpu().numpy(), g.u64(m.bit_off), g.u32(m.words)) for m in msgs]
    out = torch.full((d,), 7.0, device=g.DEV)
    nuq.nuq_decode_accumulate(msgs, d, n, s, S, 1.0 / K, False, out)
    g.check_average(host, d, n, s, 1.0 / K, out.cpu().numpy())
    prior = torch.randn(d, device=g.DEV, generator=torch.Generator(device=g.DEV).manual_seed(5))
    acc = prior.clone()
    nuq.nuq_decode_accumulate(msgs, d, n, s, S, 1.0 / K, True, acc)
    assert torch.equal(acc, prior + out)
    w, yl = prior.clone(), prior.flip(0).clone()
    w2, yl2 = w.clone(), yl.clone()
    nuq.nuq_decode_momentum_step(msgs, d, n, s, S, 1.0 / K, 0.1, 0.9, 1.0, w, yl)
    nuq.nuq_momentum_step(w2, yl2, out, 0.1, 0.9, 1.0)
    assert torch.equal(w, w2) and torch.equal(yl, yl2)
    assert nuq.nuq_last_error_flags() == 0
