"""The value projection's three tiles: a call on either side of each tile's limit of (32 tokens x one head) items, with a ragged last
workgroup and a raw tail, stores the bytes that calls of the small tile store (whose values the other tests compare with the oracle)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BF16 = 1


@pytest.mark.parametrize("dtype,H,groups,kdim", [(1, 8, 64, 64), (1, 8, 65, 320), (0, 8, 256, 64), (1, 8, 257, 192), (1, 3, 171, 64), (0, 3, 682, 64),
                                                 (1, 3, 683, 128), (0, 1, 513, 64), (1, 1, 2049, 64)])
@pytest.mark.parametrize("batch", [1, 2])
def test_same_bytes_as_the_small_tile(dtype, H, groups, kdim, batch):
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding as kv

    per = -(-groups // batch)  # groups of 32 tokens per sequence; 9 tokens more stay raw
    T = 32 * per + 9
    half = torch.bfloat16 if dtype == BF16 else torch.float16
    gen = torch.Generator(device="cuda:0").manual_seed(groups)
    k = torch.randn((batch, T, H, 128), generator=gen, device="cuda:0").to(half)
    x = torch.randn((batch, T, kdim), generator=gen, device="cuda:0").to(half)
    w = (torch.randn((H * 128, kdim), generator=gen, device="cuda:0") / kdim ** 0.5).to(half)
    images = []
    for step in (T, 32 * max(1, 256 // (H * batch))):  # one call; calls of at most 256 items
        c = kv.KVCache(kv.make_config(1, batch, H, H, 128, 32 * (per + 1), 32, 32, 32, dtype, 0, [4], [4]))
        for t in range(0, T, step):
            c.append_compressv(0, k[:, t:t + step], x[:, t:t + step], w)
        images.append(c.layers[0].cpu().numpy())
    assert np.array_equal(images[0], images[1])
