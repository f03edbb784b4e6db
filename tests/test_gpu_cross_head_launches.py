"""Mean over the kv heads: how its launches are dealt out.  Decode with eight kv heads as one workgroup of eight waves (long
launches at 4 bits) and as pairs of four, with split counts that leave the last workgroups of a launch without a whole
group of pairs, against the oracle or the vector-ALU kernels; and the mean plane of a bulk append (parts of 32 tokens of a block,
rows from the residual buffer, rotated keys) byte for byte against the oracle."""
import numpy as np
import pytest
import torch

from paper_2506_04642_amd import synth
from parity_util import check_bytes, make_pair, to_dev

pytestmark = pytest.mark.gpu

F16, BF16 = 0, 1
CROSS = 1
TOL = 2e-3 / 40  # unit-scale values: the oracle tests' measured errors are below 1e-5


@pytest.fixture(scope="module")
def kv():
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding

    return binding


@pytest.mark.parametrize("bits,G,Hkv,g,B", [(4, 32, 8, 4, 3), (2, 64, 8, 2, 5), (8, 128, 16, 1, 3), (4, 32, 12, 4, 2), (2, 32, 8, 8, 3)])
def test_split_counts(kv, oracle, bits, G, Hkv, g, B):
    T = 11 * max(G, 64) + 7
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=12 * max(G, 64), G=G, Gc=G, dtype=BF16, mode=CROSS, k_bits=(bits,))
    k, v = synth.make_kv(1, B, T, Hkv, 128, BF16)
    gpu.append(0, to_dev(k, BF16), to_dev(v, BF16))
    orc.append(0, k, v)
    q = synth.make_q(2, B, Hkv * g, 128, BF16)
    want = orc.attend(0, q)
    for ns in (0, 1, 2, 3, 5, 8, 11):
        kv.kv_set_decode_splits(gpu.handle, ns)
        got = gpu.attend(0, to_dev(q, BF16)).cpu().numpy().astype(np.float64)
        assert float(np.max(np.abs(got - want))) <= TOL, ns


@pytest.mark.parametrize("bits,Hkv,g", [(4, 1, 4), (2, 2, 8), (8, 3, 2)])
def test_split_counts_with_the_means_apart(kv, oracle, bits, Hkv, g):
    """Head counts that are no multiple of four: the merge adds the value mean plane's share, by forms that change at 8 and 36 splits."""
    B, G, T = 2, 32, 40 * 64 + 7
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=41 * 64, G=G, Gc=G, dtype=BF16, mode=CROSS, k_bits=(bits,))
    k, v = synth.make_kv(4, B, T, Hkv, 128, BF16)
    gpu.append(0, to_dev(k, BF16), to_dev(v, BF16))
    orc.append(0, k, v)
    q = synth.make_q(5, B, Hkv * g, 128, BF16)
    want = orc.attend(0, q)
    out = torch.empty((B, Hkv * g, 128), dtype=torch.float32, device="cuda:0")
    qd = to_dev(q, BF16)
    for ns in (1, 2, 7, 8, 9, 27, 41):
        kv.kv_set_decode_splits(gpu.handle, ns)
        # (a forced count may want more than the automatic ones)
        ws = torch.full((kv.kv_decode_workspace_need(gpu.handle, 0),), 0xFF, dtype=torch.uint8, device="cuda:0")
        kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), gpu._stream())
        assert float(np.max(np.abs(out.cpu().numpy().astype(np.float64) - want))) <= TOL, ns


@pytest.mark.parametrize("G,T", [(32, 12224), (32, 12352), (128, 12416)])
def test_either_side_of_the_long_launches(kv, G, T):
    """16 sequences, 8 kv heads, 4 bits: up to 24576 chunks of 64 tokens pairs of four waves, beyond that eight."""
    B, Hkv, g = 16, 8, 2
    cache = kv.KVCache(kv.make_config(1, B, Hkv * g, Hkv, 128, 12544, G, G, G, BF16, CROSS, [4], [4]))
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    for t in range(0, T, 4096):
        n = min(4096, T - t)
        k = torch.randn((B, n, Hkv, 128), generator=gen, device="cuda:0").to(torch.bfloat16)
        v = torch.randn((B, n, Hkv, 128), generator=gen, device="cuda:0").to(torch.bfloat16)
        cache.append(0, k, v)
    q = torch.randn((B, Hkv * g, 128), generator=gen, device="cuda:0").to(torch.bfloat16)
    got = cache.attend(0, q)
    kv.kv_set_decode_path(cache.handle, 1)
    assert float((got - cache.attend(0, q)).abs().max()) <= TOL


@pytest.mark.parametrize("pairing", [0, 1, 2])
@pytest.mark.parametrize("G,Hkv,dtype", [(32, 3, F16), (64, 8, BF16), (128, 5, BF16), (128, 4, F16)])
def test_mean_plane(kv, oracle, pairing, G, Hkv, dtype):
    """A raw buffer of two blocks: the second call's first block is made of rows that waited and rows that are new."""
    B, R, first, second = 2, 2 * G, G + 13, 3 * G
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv, Hkv=Hkv, T_max=6 * G, G=G, Gc=G, R=R, dtype=dtype, mode=CROSS, k_bits=(4,))
    k, v = synth.make_kv(3, B, first + second, Hkv, 128, dtype)
    cos, sin = synth.rope_tables(range(first + second), 128)
    for t0, t1 in ((0, first), (first, first + second)):
        kd, vd = to_dev(k[:, t0:t1], dtype), to_dev(v[:, t0:t1], dtype)
        if pairing == 0:
            gpu.append(0, kd, vd)
            orc.append(0, k[:, t0:t1], v[:, t0:t1])
        else:
            pairing_id = kv.KV_ROPE_HALF if pairing == 1 else kv.KV_ROPE_INTERLEAVED
            gpu.append_rope(0, kd, vd, torch.from_numpy(cos[t0:t1]).to("cuda:0"), torch.from_numpy(sin[t0:t1]).to("cuda:0"), pairing_id)
            orc.append(0, k[:, t0:t1], v[:, t0:t1], rope_tables=(cos[t0:t1], sin[t0:t1], pairing_id))
    check_bytes(gpu, orc, 0)
