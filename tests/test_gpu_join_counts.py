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
        cache._counts.view(torch.int32).fill_(1 << 20)  # what the memory may hold
    q = fill(cache)
    want = plain(kv, cache, q)
    for _ in range(2):
        out = torch.full_like(want, float("nan"))
        assert torch.equal(cache.attend(0, q, out), want)


@pytest.mark.parametrize("g", [1, 4, 8])
@pytest.mark.parametrize("call,left", [(1, 1), (1, 3), (1, 1000), (4, 0), (3, 2)])
def test_what_overlapping_calls_have_left(kv, g, call, left):
    """Counts that are not zero, as two calls at once on the same counts can leave them: the next call starts over.  A cache's n-th
    call counts down to -n * 2^20; what its workgroups, or another call's in between, leave is there or just beside."""
    cache = kv.KVCache(config(kv, g))
    q = fill(cache, 1000 if g <= 4 else 600)
    want = plain(kv, cache, q)
    for _ in range(call):
        assert torch.equal(cache.attend(0, q), want)
    for _ in range(3):
        cache._counts.view(torch.int64).fill_(left - call * (1 << 20))
        for _ in range(2):
            out = torch.full_like(want, float("nan"))
            assert torch.equal(cache.attend(0, q, out), want)
            assert not bool(cache._counts.view(torch.int64)[:-8:8].any())


def test_recorded_step_after_overlapping_calls(kv):
    """The step that ends by making its lengths the current ones has one count more; a replay wants the counts zeroed."""
    T, steps = 600, 6
    k, v = synth.make_kv(3, 2, T + steps, 2, 128, BF16)
    kd, vd = to_dev(k, BF16), to_dev(v, BF16)
    caches = [kv.KVCache(config(kv)) for _ in range(2)]
    got = []
    for spoil, cache in enumerate(caches):
        q = fill(cache, 1)
        cache.append(0, kd[:, 1:T], vd[:, 1:T])
        cache.lengths_to_device()
        out = torch.empty((steps, 2, 8, 128), dtype=torch.float32, device="cuda:0")
        for i in range(steps):
            if spoil and i:
                cache._counts.view(torch.int64).fill_(5 - i * (1 << 20))
            cache.step_dev(0, kd[:, T + i], vd[:, T + i], q, out[i])
        got.append(out)
    assert torch.equal(got[0], got[1])
    assert torch.equal(caches[0].dev_lengths, caches[1].dev_lengths)
    assert not bool(caches[1]._counts.view(torch.int64)[::8].any())
    want = caches[0].attend(0, q)
    torch.cuda.synchronize()
    graph, out = torch.cuda.CUDAGraph(), torch.empty_like(want)
    with torch.cuda.graph(graph):
        caches[0].attend(0, q, out)
    for _ in range(3):
        caches[0]._counts.fill_(1)
        caches[0].zero_counts()
        out.fill_(float("nan"))
        graph.replay()
        assert torch.equal(out, want) and torch.equal(caches[0].attend(0, q), want)
