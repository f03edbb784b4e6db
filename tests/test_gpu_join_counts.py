"""The counts of finished workgroups that KVCache hands to the joined calls: what they hold when a call begins."""
import pytest
import torch

from paper_2506_04642_amd import synth
from parity_util import to_dev

pytestmark = pytest.mark.gpu

BF16 = 1
CHAN = 0


@pytest.fixture(scope="module")
def kv():
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding

    return binding


def config(kv, g=4):
    return kv.make_config(1, 2, 2 * g, 2, 128, 2048, 32, 32, 32, BF16, CHAN, [4], [4])


def fill(cache, T=1000):
    k, v = synth.make_kv(1, 2, T, 2, 128, BF16)
    cache.append(0, to_dev(k, BF16), to_dev(v, BF16))
    return to_dev(synth.make_q(2, 2, cache.cfg.n_q_heads, 128, BF16), BF16)


def plain(kv, cache, q):
    """Attention through the call without counts."""
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda:0")
    kv.kv_decode_attn(cache.handle, 0, q.data_ptr(), out.data_ptr(), cache.workspace.data_ptr(), cache.ws_bytes, cache._stream())
    return out


def test_cache_made_while_a_stream_is_capturing(kv):
    """Nothing that is recorded then has run when the cache is first used: its counts would be what the memory held before."""
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cache = kv.KVCache(config(kv), zero=False)
    if cache._counts is not None:
        cache._counts.view(torch.int32).fill_(1)  # what the memory may hold
    q = fill(cache)
    want = plain(kv, cache, q)
    for _ in range(2):
        out = torch.full_like(want, float("nan"))
        assert torch.equal(cache.attend(0, q, out), want)
