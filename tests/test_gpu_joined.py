"""Decode attention in one launch (the last workgroup of a unit joins the partial results of its splits) against the two
launches of the plain call, bit for bit: split counts around the forms' limits, one to eight query heads per kv head,
the packed widths and 16-bit layers, paged blocks, sequences of different lengths, and the same counts used call after call."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2506_04642_amd import synth
from parity_util import append_both, make_pair, to_dev

F16, BF16 = 0, 1
CHAN, CROSS, NONE = 0, 1, 2
TOL = 2e-3 / 40  # unit-scale values: the oracle tests' measured errors are below 1e-5


@pytest.fixture(scope="module")
def kv():
    from paper_2506_04642_amd import binding

    return binding


def both(kv, gpu, q):
    """The joined call (twice, on the same counts) and the plain one: equal, and the counts are zero again."""
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda:0")
    ws = torch.full_like(gpu.workspace, 0xFF)  # (NaN wherever nothing has been stored)
    kv.kv_decode_attn(gpu.handle, 0, q.data_ptr(), out.data_ptr(), ws.data_ptr(), gpu.ws_bytes, gpu._stream())
    for _ in range(2):
        gpu.workspace.fill_(0xFF)
        got = gpu.attend(0, q)
        assert torch.equal(got, out)
        assert not bool(gpu._counts.any())
    return out.cpu().numpy().astype(np.float64)


@pytest.mark.gpu
@pytest.mark.parametrize("bits,G,g,Hkv,mode,dtype", [(4, 32, 4, 2, CHAN, BF16), (2, 64, 1, 3, CHAN, F16), (8, 128, 7, 2, NONE, BF16),
                                                     (4, 32, 8, 1, CHAN, F16), (16, 32, 4, 2, CHAN, BF16), (16, 32, 8, 1, CHAN, F16),
                                                     (4, 32, 4, 4, CROSS, BF16)])
def test_split_counts(kv, oracle, bits, G, g, Hkv, mode, dtype):
    B, T = 2, 40 * G + 5  # (a forced split holds a whole number of blocks)
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=41 * G, G=G, Gc=G, dtype=dtype, mode=mode, k_bits=(bits,))
    k, v = synth.make_kv(1, B, T, Hkv, 128, dtype)
    append_both(gpu, orc, 0, k, v, dtype)
    q = synth.make_q(2, B, Hkv * g, 128, dtype)
    want = orc.attend(0, q)
    for ns in (0, 1, 2, 3, 7, 8, 9, 14, 21, 34, 41):
        kv.kv_set_decode_splits(gpu.handle, ns)
        got = both(kv, gpu, to_dev(q, dtype))
        assert float(np.max(np.abs(got - want))) <= TOL, ns


@pytest.mark.gpu
@pytest.mark.parametrize("bits,dtype", [(4, BF16), (8, F16), (16, BF16)])
@pytest.mark.parametrize("lengths", [[1, 40, 700, 33, 4100, 64], [0, 3000, 32, 0, 31, 2000], [5, 9, 31, 1, 2, 3]])
def test_lengths(kv, oracle, bits, dtype, lengths):
    """Splits by length, sequences without a token (whose zeros no workgroup of the split kernel writes), raw tokens only."""
    Hkv, g = 2, 4
    gpu, orc = make_pair(kv, oracle, B=len(lengths), Hq=Hkv * g, Hkv=Hkv, T_max=4128, dtype=dtype, mode=CHAN, k_bits=(bits,))
    for b, n in enumerate(lengths):
        if n:
            k, v = synth.make_kv(10 + b, 1, n, Hkv, 128, dtype)
            gpu.append_seq(0, b, to_dev(k[0], dtype), to_dev(v[0], dtype))
            orc.append_seq(0, b, k[0], v[0])
    q = synth.make_q(3, len(lengths), Hkv * g, 128, dtype)
    got = both(kv, gpu, to_dev(q, dtype))
    assert float(np.max(np.abs(got - orc.attend(0, q)))) <= TOL
    for b, n in enumerate(lengths):
        if n == 0:
            assert not got[b].any()


@pytest.mark.gpu
def test_paged_step_and_graph(kv, oracle):
    """The one-call step, paged blocks, and a recorded call: replays on the same counts."""
    B, Hkv, g, G, T = 3, 2, 4, 64, 1000
    cfg = kv.make_config(1, B, Hkv * g, Hkv, 128, 2048, G, G, G, BF16, CHAN, [4], [4], pool_blocks=3 * 32)
    gpu = kv.KVCache(cfg)
    table = torch.randperm(96, dtype=torch.int32).view(B, 32).to("cuda:0")
    gpu.set_block_table(table)
    k, v = synth.make_kv(5, B, T + 70, Hkv, 128, BF16)
    kd, vd = to_dev(k, BF16), to_dev(v, BF16)
    gpu.append(0, kd[:, :T], vd[:, :T])
    q = to_dev(synth.make_q(6, B, Hkv * g, 128, BF16), BF16)
    for i in range(70):
        one = gpu.append_attend(0, kd[:, T + i], vd[:, T + i], q)
        if i % 9 == 0:
            assert np.array_equal(both(kv, gpu, q), one.cpu().numpy().astype(np.float64))
    want = gpu.attend(0, q)
    out = torch.empty_like(want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gpu.attend(0, q, out)
    for _ in range(5):
        out.fill_(float("nan"))
        graph.replay()
        assert torch.equal(out, want) and torch.equal(gpu.attend(0, q), want)
    assert not bool(gpu._counts.any())


@pytest.mark.gpu
def test_recorded_step_makes_its_lengths_current(kv, oracle):
    """kv_decode_step_dev with counts: every step finds the lengths that the one before left, as without counts."""
    B, Hkv, g, T, steps = 2, 3, 4, 600, 40
    cfg = kv.make_config(1, B, Hkv * g, Hkv, 128, 1024, 32, 32, 32, BF16, CHAN, [4], [4])
    k, v = synth.make_kv(7, B, T + steps, Hkv, 128, BF16)
    kd, vd = to_dev(k, BF16), to_dev(v, BF16)
    q = to_dev(synth.make_q(8, B, Hkv * g, 128, BF16), BF16)
    outs, caches = [], [kv.KVCache(cfg), kv.KVCache(cfg)]
    for n, c in enumerate(caches):
        c.append(0, kd[:, :T], vd[:, :T])
        c.lengths_to_device()
        got = torch.empty((steps, B, Hkv * g, 128), dtype=torch.float32, device="cuda:0")
        for i in range(steps):
            kn, vn = kd[:, T + i], vd[:, T + i]
            if n == 0:
                c.step_dev(0, kn, vn, q, got[i])
            else:
                kv.kv_decode_step_dev(c.handle, 0, kn.data_ptr(), vn.data_ptr(), kn.stride(0), kn.stride(1), q.data_ptr(),
                                      got[i].data_ptr(), c.workspace.data_ptr(), c.ws_bytes, c._stream())
        outs.append(got)
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(caches[0].dev_lengths, caches[1].dev_lengths)
    assert not bool(caches[0]._counts.any())


@pytest.mark.gpu
def test_counts_are_zero_for_every_stream(kv):
    """A new cache's counts are zeroed on the stream that makes it; the first call may be on another one that does not wait.
    (With zero=True the layers' own zeros have to be waited for in any case.)"""
    cfg = kv.make_config(1, 2, 4, 1, 128, 1024, 32, 32, 32, BF16, CHAN, [4], [4])
    k, v = synth.make_kv_torch(1, 2, 900, 1, 128, BF16, "cuda:0")
    q = synth.make_q_torch(2, 2, 4, 128, BF16, "cuda:0")
    got, want = (torch.full((2, 4, 128), float("nan"), dtype=torch.float32, device="cuda:0") for _ in range(2))
    side = torch.cuda.Stream()
    x = torch.ones((4096, 4096), device="cuda:0")
    torch.cuda.synchronize()
    for _ in range(20):
        x = torch.mm(x, x)
    gpu = kv.KVCache(cfg, zero=False)
    assert torch.cuda.current_stream().query()
    for _ in range(20):
        x = torch.mm(x, x)
    with torch.cuda.stream(side):  # (does not wait for the products)
        gpu.append(0, k, v)
        gpu.attend(0, q, got)
        kv.kv_decode_attn(gpu.handle, 0, q.data_ptr(), want.data_ptr(), gpu.workspace.data_ptr(), gpu.ws_bytes, gpu._stream())
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert not bool(gpu._counts.any())


def test_arguments(kv):
    cfg = kv.make_config(1, 3, 8, 2, 128, 256, 32, 32, 32, BF16, CHAN, [4], [4])
    assert kv.kv_join_counts_bytes(cfg) == (3 * 2 + 1) * 64
    assert kv._lib.kv_join_counts_bytes(ctypes.byref(cfg), None) == kv.KV_E_NULL
    h = kv.kv_cache_create(cfg, [0x100000])
    try:
        K, V, Q, O, W, C = 0x300000, 0x400000, 0x500000, 0x600000, 0x700000, 0x800000  # never dereferenced
        lib = kv._lib
        assert lib.kv_decode_attn_joined(h, 0, Q, O, W, 1 << 20, C + 4, None) == kv.KV_E_ALIGN
        assert lib.kv_decode_attn_joined(h, 0, Q, O, W, 1 << 20, C, None) == kv.KV_E_EMPTY
        assert lib.kv_decode_attn_joined(h, 0, Q, None, W, 1 << 20, C, None) == kv.KV_E_NULL
        assert lib.kv_append_decode_attn_joined(h, 0, K, V, 256, 128, Q, O, W, 1 << 20, C + 32, None) == kv.KV_E_ALIGN
        assert lib.kv_decode_step_dev_joined(h, 0, K, V, 256, 128, Q, O, W, 1 << 20, C, None) == kv.KV_E_BAD_CONFIG
        assert kv.kv_cache_len(h, 0) == (0, 0)
    finally:
        kv.kv_cache_destroy(h)
