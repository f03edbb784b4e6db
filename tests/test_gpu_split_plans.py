"""Decode launches whose splits are not one count for all: sequences of very different lengths get splits by
their length, and the raw tokens get splits of their own where the device holds them.  Attention against the
oracle (binary64) on both kinds of launch, over the edges of the plan: sequences without tokens, with raw tokens
only, batches beyond one wavefront's count of sequences, group sizes, head counts, 16-bit layers, paged blocks."""
import numpy as np
import pytest

from paper_2506_04642_amd import synth
from parity_util import make_pair, to_dev

pytestmark = pytest.mark.gpu

F16, BF16 = 0, 1
CHAN, NONE = 0, 2
TOL = 2e-3 / 40  # unit-scale values: the oracle tests' measured errors are below 1e-5


@pytest.fixture(scope="module")
def kv():
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding

    return binding


def fill(gpu, orc, lengths, Hkv, dtype, seed):
    for b, n in enumerate(lengths):
        if n:
            k, v = synth.make_kv(seed + b, 1, n, Hkv, 128, dtype)
            gpu.append_seq(0, b, to_dev(k[0], dtype), to_dev(v[0], dtype))
            orc.append_seq(0, b, k[0], v[0])


def check(kv, gpu, orc, B, Hq, dtype, seed):
    import torch

    q = synth.make_q(seed, B, Hq, 128, dtype)
    got = gpu.attend(0, to_dev(q, dtype))
    torch.cuda.synchronize()
    got = got.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got))
    assert float(np.max(np.abs(got - orc.attend(0, q)))) <= TOL
    return q, got


def even_splits(kv, B, T, Hkv, g, G, Gc, R, dtype, mode, bits):
    """Split count of sequences that all have T tokens (whole raw buffers): the plan with one count for all."""
    import torch

    assert T % R == 0
    cache = kv.KVCache(kv.make_config(1, B, Hkv * g, Hkv, 128, T, G, Gc, R, dtype, mode, [bits], [bits]), zero=False)
    row = torch.zeros((1, T, Hkv, 128), dtype=torch.bfloat16 if dtype else torch.float16, device="cuda:0").expand(B, T, Hkv, 128)
    cache.append(0, row, row)
    return kv.kv_decode_splits(cache.handle, 0)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("bits,G,Gc,R,Hkv,g,mode", [(4, 32, 32, 32, 2, 4, CHAN), (2, 64, 64, 64, 3, 8, CHAN), (8, 128, 128, 128, 2, 1, NONE),
                                                    (4, 64, 32, 128, 3, 3, CHAN), (16, 32, 32, 64, 2, 5, CHAN)])
@pytest.mark.parametrize("lengths", [[24000, 9000] + [37 * b % 200 for b in range(46)],
                                     [5 * b % 130 for b in range(30)] + [20011, 0, 17000, 0] + [64] * 14], ids=["first", "middle"])
def test_splits_by_length(kv, oracle, bits, G, Gc, R, Hkv, g, mode, lengths, paged):
    import torch

    print("case uneven bits=%d G=%d Gc=%d R=%d heads=%d x %d paged=%s" % (bits, G, Gc, R, Hkv, g, paged), flush=True)
    B, cap = len(lengths), (max(lengths) // R + 1) * R
    blocks = sum(n // R * R // G for n in lengths)
    gpu = kv.KVCache(kv.make_config(1, B, Hkv * g, Hkv, 128, cap, G, Gc, R, BF16, mode, [bits], [bits], pool_blocks=blocks + 3 if paged else 0))
    orc = oracle.OracleCache(oracle.OracleConfig(1, B, Hkv * g, Hkv, 128, cap, G, Gc, R, BF16, mode, [bits], [bits]))
    if paged:
        slots = list(np.random.default_rng(G).permutation(blocks + 3))
        table = np.full((B, cap // G), 10 ** 6, dtype=np.int32)
        for b, n in enumerate(lengths):
            for x in range(n // R * R // G):
                table[b, x] = slots.pop()
        gpu.set_block_table(torch.from_numpy(table).to("cuda:0"))
    fill(gpu, orc, lengths, Hkv, BF16, 1900 + bits)
    q, got = check(kv, gpu, orc, B, Hkv * g, BF16, 1900)
    for b, n in enumerate(lengths):
        if n == 0:
            assert not got[b].any()
    assert kv.kv_decode_workspace_need(gpu.handle, 0) <= gpu.ws_bytes
    # the launch is uneven: the longest sequence has more splits than one count for all would give it
    assert kv.kv_decode_splits(gpu.handle, 0) > even_splits(kv, B, max(lengths) // R * R, Hkv, g, G, Gc, R, BF16, mode, bits) + 1


@pytest.mark.parametrize("B", [63, 64, 65, 131])
def test_splits_by_length_over_many_sequences(kv, oracle, B):
    """More sequences than a wavefront has lanes: the launch finds a split's sequence in several steps.  One long
    sequence at either end and in the middle, empty ones between."""
    print("case uneven batch=%d" % B, flush=True)
    gpu, orc = make_pair(kv, oracle, B=B, Hq=2, Hkv=1, T_max=32768, G=32, R=32, dtype=F16, k_bits=(4,))
    lengths = [(5 * b + 1) % 47 if b % 7 else 0 for b in range(B)]
    lengths[0], lengths[B // 2], lengths[B - 1] = 23000, 12500, 29001
    fill(gpu, orc, lengths, 1, F16, 2000)
    check(kv, gpu, orc, B, 2, F16, 2000)
    # the launch is uneven: the longest sequence has more splits than one count for all would give it
    assert kv.kv_decode_splits(gpu.handle, 0) > even_splits(kv, B, 28992, 1, 2, 32, 32, 32, F16, CHAN, 4) + 1


def spread(B, T):
    return [T * (1 + (5 * b + B - 1) % B) // B for b in range(B)]


@pytest.mark.parametrize("bits,G,R,lengths,uneven", [
    (8, 64, 64, spread(24, 8011), True), (4, 64, 64, spread(24, 8011), False), (4, 64, 128, spread(24, 8011), False),
    (4, 64, 64, [8011] + [150 + 7 * b for b in range(23)], True), (4, 32, 64, [2000 - 13 * b for b in range(64)], False),
    (2, 64, 128, [3990 - 13 * b for b in range(24)], False), (16, 32, 32, [4000] + [150 + 7 * b for b in range(23)], True)])
def test_splits_by_length_only_where_they_shorten_the_launch(kv, bits, G, R, lengths, uneven):
    """The plan of launches that were measured both ways: one long sequence among short ones and wide spreads at 8 bits get
    splits by length, launches that the device's rate bounds and those whose raw tokens would pile up do not."""
    import torch

    print("case uneven_or_not bits=%d G=%d R=%d B=%d" % (bits, G, R, len(lengths)), flush=True)
    B, Hkv, g, T = len(lengths), 8, 4, (max(lengths) // R + 1) * R
    gpu = kv.KVCache(kv.make_config(1, B, Hkv * g, Hkv, 128, T, G, G, R, BF16, CHAN, [bits], [bits]))
    row = torch.zeros((T, Hkv, 128), dtype=torch.bfloat16, device="cuda:0")
    for b, n in enumerate(lengths):
        gpu.append_seq(0, b, row[:n], row[:n])
    even = even_splits(kv, B, max(lengths) // R * R, Hkv, g, G, G, R, BF16, CHAN, bits)
    got = kv.kv_decode_splits(gpu.handle, 0)
    assert (got > even) if uneven else (got == even), (got, even)


def test_workspace_that_fits_one_count_only(kv, oracle):
    """A workspace too small for splits by length, but large enough for one count for all, is accepted: the launch has one
    count then, in kv_decode_attn and in the split and the merge call alike."""
    import torch

    print("case uneven_workspace", flush=True)
    B, Hkv, g, R = 96, 2, 4, 32
    lengths = spread(B, 2000)
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=2048, dtype=BF16, k_bits=(8,))
    fill(gpu, orc, lengths, Hkv, BF16, 2100)
    q, got = check(kv, gpu, orc, B, Hkv * g, BF16, 2100)
    even = even_splits(kv, B, 1984, Hkv, g, 32, 32, R, BF16, CHAN, 8)
    size = B * Hkv * g * even * 132 * 4
    assert kv.kv_decode_splits(gpu.handle, 0) > even and kv.kv_decode_workspace_need(gpu.handle, 0) > size, "the launch is uneven and takes more"
    want = orc.attend(0, q)
    qd = to_dev(q, BF16)
    outs = [torch.empty((B, Hkv * g, 128), dtype=torch.float32, device="cuda:0") for _ in range(2)]
    ws, st = gpu.workspace.data_ptr(), gpu._stream()
    gpu.workspace.fill_(255)  # (NaN in every partial result that this launch does not write)
    kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), outs[0].data_ptr(), ws, size, st)
    gpu.workspace.fill_(255)
    kv.kv_decode_attn_split(gpu.handle, 0, qd.data_ptr(), ws, size, st)
    kv.kv_decode_attn_merge(gpu.handle, 0, outs[1].data_ptr(), ws, size, st)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    assert float(np.max(np.abs(outs[0].cpu().numpy().astype(np.float64) - want))) <= TOL
    with pytest.raises(kv.KVError) as e:
        kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), outs[0].data_ptr(), ws, size - 1, st)
    assert e.value.status == kv.KV_E_WORKSPACE


@pytest.mark.parametrize("bits,G,R,raw", [(4, 32, 32, 31), (2, 32, 128, 127), (8, 64, 256, 255), (4, 128, 128, 1), (2, 64, 128, 97)])
@pytest.mark.parametrize("g", [1, 8])
def test_splits_for_the_raw_tokens(kv, oracle, bits, G, R, raw, g):
    """Few chunks and up to eight tiles of raw tokens: the tiles go to splits of their own, also when the step that
    attends appends the newest token itself."""
    import torch

    print("case resid_splits bits=%d G=%d R=%d raw=%d g=%d" % (bits, G, R, raw, g), flush=True)
    B, Hkv, T = 2, 2, 4 * R + raw - 1
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=5 * R, G=G, Gc=G, R=R, dtype=BF16, k_bits=(bits,))
    k, v = synth.make_kv(2200 + raw, B, T + 1, Hkv, 128, BF16)
    kd, vd = to_dev(k, BF16), to_dev(v, BF16)
    if T:
        gpu.append(0, kd[:, :T], vd[:, :T])
    q = synth.make_q(2200, B, Hkv * g, 128, BF16)
    got = gpu.append_attend(0, kd[:, T], vd[:, T], to_dev(q, BF16))
    torch.cuda.synchronize()
    orc.append(0, k, v)
    assert float(np.max(np.abs(got.cpu().numpy().astype(np.float64) - orc.attend(0, q)))) <= TOL
    again = gpu.attend(0, to_dev(q, BF16))
    torch.cuda.synchronize()
    assert torch.equal(got, again)
    img = orc.layer_image(0)
    assert np.array_equal(gpu.layers[0].cpu().numpy()[img["valid"]], img["bytes"][img["valid"]])


@pytest.mark.parametrize("bits,G,R,T,raw,own", [(4, 32, 512, 4096, 511, 16), (2, 64, 512, 4096, 320, 10), (8, 128, 512, 4096, 511, 16),
                                                (4, 32, 1024, 4096, 1023, 16), (4, 32, 1024, 4096, 100, 4), (4, 32, 1024, 16384, 1023, 0),
                                                (2, 128, 2048, 16384, 2047, 0)])
def test_long_raw_buffers(kv, oracle, bits, G, R, T, raw, own):
    """Raw buffers of many tiles: a split of its own for every tile, up to sixteen; beyond that, where such a split would
    take more tiles one after the other than all splits do that share them, they go to all, as many splits as
    without raw tokens."""
    import torch

    print("case long_raw bits=%d G=%d R=%d raw=%d" % (bits, G, R, raw), flush=True)
    B, Hkv, g = 1, 2, 4
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=T + R, G=G, Gc=G, R=R, dtype=BF16, k_bits=(bits,))
    k, v = synth.make_kv(2250 + raw, B, T + raw, Hkv, 128, BF16)
    kd, vd = to_dev(k, BF16), to_dev(v, BF16)
    gpu.append(0, kd[:, :T], vd[:, :T])
    assert gpu.lengths(0) == (T, 0)
    empty = kv.kv_decode_splits(gpu.handle, 0)
    gpu.append(0, kd[:, T:], vd[:, T:])
    orc.append(0, k, v)
    chunks = (T + (127 if G == 128 else 63)) // (128 if G == 128 else 64)
    assert empty == -(-T // 64 // 4), "one chunk of 64 tokens per wave"
    assert kv.kv_decode_splits(gpu.handle, 0) == (-(-chunks // 4) + own if own else empty)
    q = synth.make_q(2250, B, Hkv * g, 128, BF16)
    check_q = to_dev(q, BF16)
    got = gpu.attend(0, check_q)
    torch.cuda.synchronize()
    assert float(np.max(np.abs(got.cpu().numpy().astype(np.float64) - orc.attend(0, q)))) <= TOL


@pytest.mark.parametrize("mode,Hkv", [(CHAN, 1), (1, 2)])  # (1: the mean over the heads, in kernels of its own)
def test_merge_at_the_edges_of_its_forms(kv, oracle, mode, Hkv):
    """Split counts on either side of what each form of the merge kernel requests at once."""
    import torch

    print("case merge_edges mode=%d" % mode, flush=True)
    B, g, T = 1, 2, 32 * 257 + 9
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=32 * 260, dtype=BF16, mode=mode, k_bits=(4,))
    k, v = synth.make_kv(2300, B, T, Hkv, 128, BF16)
    gpu.append(0, to_dev(k, BF16), to_dev(v, BF16))
    orc.append(0, k, v)
    q = synth.make_q(2300, B, Hkv * g, 128, BF16)
    want = orc.attend(0, q)
    for ns in (1, 3, 4, 5, 8, 9, 35, 36, 37, 71, 72, 73, 127, 128, 129, 256):
        kv.kv_set_decode_splits(gpu.handle, ns)
        size = kv.kv_decode_workspace_need(gpu.handle, 0)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        out = torch.empty((B, Hkv * g, 128), dtype=torch.float32, device="cuda:0")
        qd = to_dev(q, BF16)
        kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), out.data_ptr(), ws.data_ptr(), size, gpu._stream())
        torch.cuda.synchronize()
        err = float(np.max(np.abs(out.cpu().numpy().astype(np.float64) - want)))
        assert err <= TOL, (ns, err)


@pytest.mark.parametrize("bits,mode,Hkv", [(4, CHAN, 2), (2, NONE, 2), (8, CHAN, 1), (4, 1, 4), (4, 1, 2), (16, CHAN, 2)])
@pytest.mark.parametrize("path", [0, 1])
def test_infinite_raw_value_through_the_merge(kv, oracle, bits, mode, Hkv, path):
    """An infinity of either sign among the raw values: the channel is infinite whatever the split count, also where
    a form of the merge requests more partial results than there are splits."""
    import torch

    print("case merge_infinity bits=%d mode=%d heads=%d path=%d" % (bits, mode, Hkv, path), flush=True)
    B, g, T = 2, 4, 32 * 48 + 11
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=32 * 50, dtype=BF16, mode=mode, k_bits=(bits,))
    kv.kv_set_decode_path(gpu.handle, path)
    k, v = synth.make_kv(2350 + bits, B, T, Hkv, 128, BF16)
    k[:, 1536:] = 0  # score 0: the rows' weights are far from binary32's smallest numbers
    v[1, 1536, 0, 5], v[1, 1536, 0, 70] = 0x7F80, 0xFF80  # the first raw row: the last one has another test of its own
    gpu.append(0, to_dev(k, BF16), to_dev(v, BF16))
    orc.append(0, k, v)
    q = synth.make_q(2350, B, Hkv * g, 128, BF16)
    want = orc.attend(0, q)
    finite = np.isfinite(want)
    assert np.count_nonzero(~finite) == 2 * g
    for ns in (0, 1, 2, 3, 4, 5, 8, 9, 13, 37, 40):
        kv.kv_set_decode_splits(gpu.handle, ns)
        ws = torch.empty(kv.kv_decode_workspace_need(gpu.handle, 0), dtype=torch.uint8, device="cuda:0")
        out = torch.empty((B, Hkv * g, 128), dtype=torch.float32, device="cuda:0")
        qd = to_dev(q, BF16)
        kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), gpu._stream())
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        assert np.all(got[1, :g, 5] == np.inf) and np.all(got[1, :g, 70] == -np.inf), ns
        assert np.max(np.abs(got[finite] - want[finite])) <= TOL, ns


@pytest.mark.parametrize("bits,G,Hkv,g,mode", [(4, 32, 2, 4, CHAN), (2, 64, 3, 8, NONE), (8, 128, 1, 1, CHAN), (16, 32, 2, 3, CHAN),
                                               (4, 32, 4, 4, 1), (2, 64, 2, 4, 1)])
def test_short_launches_write_the_output_themselves(kv, oracle, bits, G, Hkv, g, mode):
    """Around the lengths up to which a call is one launch: attend (which then writes the output in the split kernel)
    against the oracle and, bit for bit, against the split and the merge as calls of their own; a sequence
    that is switched off gets zeros."""
    import torch

    print("case direct bits=%d G=%d heads=%d x %d mode=%d" % (bits, G, Hkv, g, mode), flush=True)
    B, Hq = 3, Hkv * g
    for T in (1, 31, 64, 65, 129, 255, 256, 257, 300, 513):
        gpu, orc = make_pair(kv, oracle, B=B, Hq=Hq, Hkv=Hkv, T_max=640, G=G, Gc=G, R=G, dtype=BF16, mode=mode, k_bits=(bits,))
        k, v = synth.make_kv(2400 + T, B, T, Hkv, 128, BF16)
        gpu.append(0, to_dev(k, BF16), to_dev(v, BF16))
        orc.append(0, k, v)
        q = synth.make_q(2400, B, Hq, 128, BF16)
        qd = to_dev(q, BF16)
        got = gpu.attend(0, qd)
        two = torch.empty_like(got)
        kv.kv_decode_attn_split(gpu.handle, 0, qd.data_ptr(), gpu.workspace.data_ptr(), gpu.ws_bytes, gpu._stream())
        kv.kv_decode_attn_merge(gpu.handle, 0, two.data_ptr(), gpu.workspace.data_ptr(), gpu.ws_bytes, gpu._stream())
        torch.cuda.synchronize()
        assert torch.equal(got, two), T
        assert float(np.max(np.abs(got.cpu().numpy().astype(np.float64) - orc.attend(0, q)))) <= TOL, T
        kv.kv_cache_set_active(gpu.handle, [1, 0, 1])
        part = gpu.attend(0, qd)
        torch.cuda.synchronize()
        assert not part[1].any()
        assert float((part[::2] - got[::2]).abs().max()) <= TOL


@pytest.mark.parametrize("bits,G,R", [(4, 32, 32), (2, 64, 128), (8, 128, 128), (16, 32, 64)])
def test_need_read_on_an_empty_raw_buffer_serves_the_tokens_that_follow(kv, oracle, bits, G, R):
    """kv_decode_workspace_need, read when the raw buffer is empty, holds for every call until the next block: the raw
    tokens' own splits do not make a call ask for more."""
    import torch

    print("case need_until_next_block bits=%d G=%d R=%d" % (bits, G, R), flush=True)
    B, Hkv, g = 2, 2, 4
    T = 1024 // R * R
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv * g, Hkv=Hkv, T_max=T + 2 * R, G=G, Gc=G, R=R, dtype=BF16, k_bits=(bits,))
    k, v = synth.make_kv(2600 + bits, B, T + R, Hkv, 128, BF16)
    kd, vd = to_dev(k, BF16), to_dev(v, BF16)
    gpu.append(0, kd[:, :T], vd[:, :T])
    orc.append(0, k[:, :T], v[:, :T])
    need = kv.kv_decode_workspace_need(gpu.handle, 0)
    plain = B * Hkv * g * kv.kv_decode_splits(gpu.handle, 0) * 132 * 4  # the chunks' splits alone
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    out = torch.empty((B, Hkv * g, 128), dtype=torch.float32, device="cuda:0")
    st = gpu._stream()
    for s in range(R - 1):
        q = synth.make_q(2600 + s, B, Hkv * g, 128, BF16)
        qd = to_dev(q, BF16)
        kn, vn = kd[:, T + s], vd[:, T + s]
        kv.kv_append_decode_attn(gpu.handle, 0, kn.data_ptr(), vn.data_ptr(), kn.stride(0), kn.stride(1), qd.data_ptr(), out.data_ptr(), ws.data_ptr(), need, st)
        orc.append(0, k[:, T + s:T + s + 1], v[:, T + s:T + s + 1])
        again = torch.empty_like(out)
        kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), again.data_ptr(), ws.data_ptr(), need, st)
        torch.cuda.synchronize()
        assert torch.equal(out, again), s
        assert torch.equal(out, gpu.attend(0, qd)), s
        if s % 8 == 0 or s == R - 2:
            assert float(np.max(np.abs(out.cpu().numpy().astype(np.float64) - orc.attend(0, q)))) <= TOL, s
        assert kv.kv_decode_workspace_need(gpu.handle, 0) <= need
        if s % 8 == 1 and bits != 16:
            # a workspace for the chunks' splits alone is accepted, the raw tokens go to the same splits then
            kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), out.data_ptr(), ws.data_ptr(), plain, st)
            kv.kv_decode_attn_split(gpu.handle, 0, qd.data_ptr(), ws.data_ptr(), plain, st)
            kv.kv_decode_attn_merge(gpu.handle, 0, again.data_ptr(), ws.data_ptr(), plain, st)
            torch.cuda.synchronize()
            assert torch.equal(out, again), s
            assert float(np.max(np.abs(out.cpu().numpy().astype(np.float64) - orc.attend(0, q)))) <= TOL, s
            row = B * Hkv * g * 132 * 4  # (a launch with splits for the raw tokens may be the smaller of the two)
            with pytest.raises(kv.KVError) as e:
                kv.kv_decode_attn(gpu.handle, 0, qd.data_ptr(), out.data_ptr(), ws.data_ptr(), min(plain, row * kv.kv_decode_splits(gpu.handle, 0)) - 1, st)
            assert e.value.status == kv.KV_E_WORKSPACE
