"""Long appends in blocks of 32 tokens: from 40960 items (blocks x units x 2) on another instance stores the records plainly, at 8 bits and
at 4 bits without a mean on fewer workgroups.  A call on each side of the line against one call per sequence, all of which
are below it: the same bytes."""
import pytest
import torch

pytestmark = pytest.mark.gpu

F16, BF16 = 0, 1
CHAN, CROSS, NONE = 0, 1, 2
ITEMS, H = 40960, 8


@pytest.mark.parametrize("bits,B,mode,dtype,Gc", [(8, 8, CHAN, BF16, 32), (8, 9, NONE, F16, 64), (8, 7, CHAN, F16, 128), (8, 8, CROSS, BF16, 32),
                                                  (4, 8, NONE, BF16, 32), (4, 8, CHAN, F16, 128), (2, 9, CHAN, BF16, 64)])
def test_same_bytes_on_both_sides(bits, B, mode, dtype, Gc):
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding as kv

    need = -(-ITEMS // (2 * B * H))  # blocks of a sequence
    half = torch.bfloat16 if dtype == BF16 else torch.float16
    gen = torch.Generator(device="cuda:0").manual_seed(bits * B)
    T = need * 32 + 13
    k, v = (torch.randn((B, T, H, 128), generator=gen, device="cuda:0").to(half) for _ in range(2))
    cfg = kv.make_config(1, B, H, H, 128, (need + 1) * 32, 32, Gc, 32, dtype, mode, [bits], [bits])
    whole, apart = kv.KVCache(cfg), kv.KVCache(cfg)
    for blocks, tail in ((need, 13), (need, 0), (need - 1, 31)):
        n = blocks * 32 + tail
        for cache in (whole, apart):
            kv.kv_cache_reset(cache.handle)
            cache.layers[0].zero_()
        whole.append(0, k[:, :n], v[:, :n])
        for b in range(B):
            apart.append_seq(0, b, k[b, :n], v[b, :n])
        assert torch.equal(whole.layers[0], apart.layers[0]), n
