"""Large launches fetch a layer's records past the caches, small ones do not (another instance of the split kernel; kv_decode_past_caches
says which).  With the split count fixed a sequence's output does not depend on the others: a launch of all sequences, on the one
side of the limit, against launches of one sequence at a time, on the other side."""
import pytest
import torch

pytestmark = pytest.mark.gpu

F16, BF16 = 0, 1
CHAN, CROSS = 0, 1


@pytest.mark.parametrize("bits,G,B,T,g,mode,dtype,paged", [(4, 32, 8, 4005, 4, CHAN, BF16, False), (8, 64, 3, 8070, 8, CHAN, F16, False),
                                                           (8, 128, 3, 8322, 4, CHAN, BF16, True), (2, 32, 45, 4001, 4, CHAN, F16, False),
                                                           (4, 64, 8, 6043, 4, CROSS, BF16, False), (16, 32, 4, 4101, 4, CHAN, BF16, True)])
def test_same_output_on_both_sides(bits, G, B, T, g, mode, dtype, paged):
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding as kv

    H, half = 8, torch.bfloat16 if dtype == BF16 else torch.float16
    blocks = -(-T // G)
    gen = torch.Generator(device="cuda:0").manual_seed(bits * G)
    k, v = (torch.randn((B, T, H, 128), generator=gen, device="cuda:0").to(half) for _ in range(2))
    q = torch.randn((B, H * g, 128), generator=gen, device="cuda:0").to(half)

    def cache(n):
        c = kv.KVCache(kv.make_config(1, n, H * g, H, 128, blocks * G, G, G, G, dtype, mode, [bits], [bits], **({"pool_blocks": n * blocks} if paged else {})))
        if paged:
            c.set_block_table(torch.randperm(n * blocks, generator=gen, device="cuda:0").to(torch.int32).view(n, blocks))
        return c

    whole = cache(B)
    whole.append(0, k, v)
    kv.kv_set_decode_splits(whole.handle, 3)
    assert kv.kv_decode_past_caches(whole.handle, 0)
    got = whole.attend(0, q)
    assert torch.isfinite(got).all()
    for b in sorted({0, B // 2, B - 1}):
        one = cache(1)
        one.append(0, k[b:b + 1], v[b:b + 1])
        kv.kv_set_decode_splits(one.handle, 3)
        assert not kv.kv_decode_past_caches(one.handle, 0)
        assert torch.equal(got[b:b + 1], one.attend(0, q[b:b + 1])), b
