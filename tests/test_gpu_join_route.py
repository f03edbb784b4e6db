"""Which calls join their splits inside the split launch.  With counts that are preset to a small number no workgroup takes itself
for the last, so an output that is NaN before the call stays NaN exactly if the split kernel was to join (every
kernel ends as ever; the counts are zeroed afterwards).  Both sides of each limit, with the split counts exactly there."""
import numpy as np
import pytest
import torch

from paper_2506_04642_amd import synth
from parity_util import make_pair, to_dev

pytestmark = pytest.mark.gpu

F16, BF16 = 0, 1
CHAN, CROSS, NONE = 0, 1, 2
TOL = 2e-3 / 40  # unit-scale values: the oracle tests' measured errors are below 1e-5


@pytest.fixture(scope="module")
def kv():
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding

    return binding


def joins(cache, call):
    """call(out) is made on spoiled counts: was its output left to the split kernel?  Then again on zeros: its output."""
    shape = (cache.cfg.batch, cache.cfg.n_q_heads, 128)
    out = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda:0")
    cache._counts.view(torch.int64).fill_(1 << 20)
    call(out)
    left = bool(torch.isnan(out).all())
    assert left or not bool(torch.isnan(out).any())
    counted = bool((cache._counts.view(torch.int64) != 1 << 20).any())
    assert left == counted
    cache._counts.zero_()
    return left


@pytest.mark.parametrize("bits,G,g,Hkv,mode,dtype,most", [(4, 32, 4, 2, CHAN, BF16, 34), (2, 64, 1, 3, CHAN, F16, 34), (8, 128, 3, 2, NONE, BF16, 34),
                                                          (4, 32, 5, 1, CHAN, F16, 8), (2, 128, 8, 2, NONE, BF16, 8), (16, 32, 4, 2, CHAN, BF16, 8),
                                                          (16, 64, 8, 1, CHAN, F16, 8), (4, 32, 4, 4, CROSS, BF16, 0)])
def test_limits(kv, oracle, bits, G, g, Hkv, mode, dtype, most):
    B = 2
    for ns in (1, 2, 8, 9, 34, 35):
        T = (ns - 1) * G + 5  # as many pieces of work as splits: blocks, and the raw tokens
        gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=36 * G, G=G, Gc=G, dtype=dtype, mode=mode, k_bits=(bits,))
        k, v = synth.make_kv(1, B, T, Hkv, 128, dtype)
        gpu.append(0, to_dev(k, dtype), to_dev(v, dtype))
        orc.append(0, k, v)
        q = synth.make_q(2, B, Hkv * g, 128, dtype)
        qd = to_dev(q, dtype)
        kv.kv_set_decode_splits(gpu.handle, ns)
        assert kv.kv_decode_splits(gpu.handle, 0) == ns
        assert joins(gpu, lambda out: gpu.attend(0, qd, out)) == (1 < ns <= most), ns
        got = gpu.attend(0, qd)
        plain = torch.empty_like(got)
        kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), plain.data_ptr(), gpu.workspace.data_ptr(), gpu.ws_bytes, gpu._stream())
        assert torch.equal(got, plain)
        assert float(np.max(np.abs(got.cpu().numpy().astype(np.float64) - orc.attend(0, q)))) <= TOL, ns


def filled(kv, lengths, *, bits=4, g=4, Hkv=2, T_max=4128, pool=0):
    cache = kv.KVCache(kv.make_config(1, len(lengths), Hkv * g, Hkv, 128, T_max, 32, 32, 32, BF16, CHAN, [bits], [bits], pool_blocks=pool))
    for b, n in enumerate(lengths):
        if n:
            k, v = synth.make_kv_torch(10 + b, 1, n, Hkv, 128, BF16, "cuda:0")
            cache.append_seq(0, b, k[0], v[0])
    return cache, synth.make_q_torch(3, len(lengths), Hkv * g, 128, BF16, "cuda:0")


@pytest.mark.parametrize("short,want", [(300, True), (0, False)])
def test_splits_by_length(kv, short, want):
    """One long sequence among 39 short ones: splits by its length, joined unless a sequence has no workgroup to write its zeros."""
    lengths = [300] * 40
    lengths[7], lengths[23] = 8000, short
    cache, q = filled(kv, lengths, Hkv=4, T_max=8224)
    assert 16 < kv.kv_decode_splits(cache.handle, 0) <= 34  # (one count for all: 1024 workgroups / 160 units at most)
    assert joins(cache, lambda out: cache.attend(0, q, out)) == want
    got, plain = cache.attend(0, q), torch.empty_like(q, dtype=torch.float32)
    kv.kv_decode_attn(cache.handle, 0, q.data_ptr(), plain.data_ptr(), cache.workspace.data_ptr(), cache.ws_bytes, cache._stream())
    assert torch.equal(got, plain) and bool(got[7].any()) and bool(got[23].any()) == want


@pytest.mark.parametrize("bits", [4, 16])
def test_raw_tokens_only_are_one_split(kv, bits):
    cache, q = filled(kv, [5, 9, 31, 1, 2, 3], bits=bits)
    assert not joins(cache, lambda out: cache.attend(0, q, out))


def test_automatic_plans(kv):
    """One sequence of 8205 tokens and 8 kv heads: the chunks in 33 splits at most, one launch.  The vector-ALU kernels: never."""
    cache, q = filled(kv, [8205], Hkv=8, T_max=8224)
    assert 8 < kv.kv_decode_splits(cache.handle, 0) <= 34
    assert joins(cache, lambda out: cache.attend(0, q, out))
    kv.kv_set_decode_path(cache.handle, 1)
    assert not joins(cache, lambda out: cache.attend(0, q, out))


@pytest.mark.parametrize("g", [4, 8])
def test_steps(kv, g):
    """The one-call step and the recorded one; a step that completes a block stores it first and is joined as well."""
    cache, q = filled(kv, [637, 637], g=g)
    k, v = synth.make_kv_torch(9, 2, 4, 2, 128, BF16, "cuda:0")
    for i in range(3):  # raw tokens 30, 31, none
        assert joins(cache, lambda out: cache.append_attend(0, k[:, i], v[:, i], q, out))
    cache.lengths_to_device()
    assert joins(cache, lambda out: cache.step_dev(0, k[:, 3], v[:, 3], q, out))
