"""Raw tail of a bulk append: stored by the quantiser's own launch when the call starts on an empty residual
buffer, by a launch after it when the buffer held rows (which the compression reads first).  Cache bytes bit
for bit against the oracle either way, for every quantiser kernel."""
import numpy as np
import pytest

from paper_2506_04642_amd import synth
from parity_util import append_both, check_bytes, make_pair, to_dev

pytestmark = pytest.mark.gpu

F16, BF16 = 0, 1
CHAN, CROSS, NONE = 0, 1, 2


@pytest.fixture(scope="module")
def kv():
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding

    return binding


@pytest.mark.parametrize("kb,vb,G,Gc,R,mode", [(4, 4, 32, 32, 32, CHAN), (2, 8, 32, 64, 64, CHAN), (8, 8, 64, 64, 64, NONE),
                                               (2, 2, 64, 32, 128, CROSS), (4, 4, 128, 128, 128, CHAN), (4, 2, 64, 64, 64, CHAN),
                                               (16, 16, 32, 32, 64, CHAN)])
@pytest.mark.parametrize("tail", [1, 31])
def test_tail_on_an_empty_and_on_a_begun_buffer(kv, oracle, kb, vb, G, Gc, R, mode, tail):
    print("case tail kb=%d vb=%d G=%d Gc=%d R=%d mode=%d tail=%d" % (kb, vb, G, Gc, R, mode, tail), flush=True)
    B, Hkv = 3, 3
    # empty buffer: blocks and a tail; the buffer filled and emptied by a call that leaves none; again blocks and a
    # tail on the empty buffer; then on the begun one
    chunks = [R + tail, R - tail, 2 * R + tail, R + 1]
    T = sum(chunks)
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv, Hkv=Hkv, T_max=(T + R) // R * R, G=G, Gc=Gc, R=R, dtype=BF16, mode=mode,
                         k_bits=(kb,), v_bits=(vb,))
    k, v = synth.make_kv(1800 + kb + G + tail, B, T, Hkv, 128, BF16)
    done = 0
    for n in chunks:
        append_both(gpu, orc, 0, np.ascontiguousarray(k[:, done:done + n]), np.ascontiguousarray(v[:, done:done + n]), BF16)
        done += n
        check_bytes(gpu, orc, 0)


def test_tail_of_sequences_in_different_states(kv, oracle):
    """One call, two runs of sequences: one starts on an empty buffer, the other on a begun one."""
    import torch

    print("case tail_runs", flush=True)
    B, Hkv, R = 4, 2, 32
    gpu, orc = make_pair(kv, oracle, B=B, Hq=Hkv, Hkv=Hkv, T_max=6 * R, dtype=F16, k_bits=(4,))
    k, v = synth.make_kv(1850, B, 5 * R, Hkv, 128, F16)
    for b in (2, 3):
        gpu.append_seq(0, b, to_dev(k[b, :9], F16), to_dev(v[b, :9], F16))
        orc.append_seq(0, b, k[b, :9], v[b, :9])
    n = 2 * R + 5
    append_both(gpu, orc, 0, np.ascontiguousarray(k[:, 9:9 + n]), np.ascontiguousarray(v[:, 9:9 + n]), F16)
    torch.cuda.synchronize()
    img = orc.layer_image(0)
    assert np.array_equal(gpu.layers[0].cpu().numpy()[img["valid"]], img["bytes"][img["valid"]])
