"""Attention over layers stored in 16 bits (the matrix-core kernel for raw rows) at the edges of its
chunks of 32 tokens, against the CPU oracle and against the vector-ALU kernel.

Tolerance: scores and output are sums of exact products (scores) or of binary32 products (output) in
binary32.  With |q . k| sums of 128 terms of size <= 60 and |v| <= 6, a score is off by at most
128 * 2^-24 * 60 * sqrt(128) / sqrt(128) < 5e-4 in the worst order and about 1e-5 for rounding errors of
random sign, the output by as much relative to |v|: 2e-4 absolute leaves a factor of several."""
import numpy as np
import pytest

from paper_2506_04642_amd import synth
import parity_util
from parity_util import append_both, check_attention, make_pair, to_dev

pytestmark = pytest.mark.gpu

F16, BF16 = 0, 1
TOL = 2e-4


@pytest.fixture(scope="module")
def kv():
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2506_04642_amd import binding

    return binding


@pytest.mark.parametrize("T", [1, 32, 33, 127, 128, 129, 1000, 5003])
@pytest.mark.parametrize("g", [1, 3, 8])
@pytest.mark.parametrize("G,R,dtype", [(32, 32, BF16), (64, 128, F16), (128, 128, BF16)])
def test_raw_layer_chunk_edges(kv, oracle, G, R, dtype, g, T):
    print("case raw layer G=%d R=%d g=%d T=%d" % (G, R, g, T), flush=True)
    parity_util.DECODE_PATH = 0
    gpu, orc = make_pair(kv, oracle, B=2, Hq=2 * g, Hkv=2, T_max=(T // R + 2) * R, G=G, Gc=G, R=R, dtype=dtype, k_bits=(16,))
    k, v = synth.make_kv(31 * T + g, 2, T, 2, 128, dtype)
    append_both(gpu, orc, 0, k, v, dtype)
    q = synth.make_q(T, 2, 2 * g, 128, dtype)
    check_attention(gpu, orc, 0, q, dtype, tol=TOL)
    if T >= 128:
        first = gpu.attend(0, to_dev(q, dtype))
        kv.kv_set_decode_splits(gpu.handle, 3)
        check_attention(gpu, orc, 0, q, dtype, tol=TOL)
        kv.kv_set_decode_splits(gpu.handle, 0)
        assert (gpu.attend(0, to_dev(q, dtype)) == first).all(), "a repeated call gives the same bits"


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("G", [32, 64])
def test_raw_layer_ragged_batch(kv, oracle, G, paged):
    """Sequences of 0, 1, a few and many tokens side by side; blocks through a table; more than 64 chunks
    per wave with one forced split (the table is then read again on the way)."""
    import torch

    print("case raw layer ragged G=%d paged=%s" % (G, paged), flush=True)
    lens = [0, 1, G - 1, G, 40 * G + 17, 9000]
    B, cap = len(lens), (max(lens) // G + 2) * G
    need = sum(n // G for n in lens)
    cfg = kv.make_config(1, B, 8, 2, 128, cap, G, G, G, BF16, 0, [16], [16], pool_blocks=need + 3 if paged else 0)
    ocfg = oracle.OracleConfig(1, B, 8, 2, 128, cap, G, G, G, BF16, 0, [16], [16])
    gpu, orc = kv.KVCache(cfg), oracle.OracleCache(ocfg)
    if paged:
        slots = list(np.random.default_rng(G).permutation(need + 3))
        table = np.full((B, cap // G), 10 ** 6, dtype=np.int32)
        for b, n in enumerate(lens):
            for j in range(n // G):
                table[b, j] = slots.pop()
        gpu.set_block_table(torch.from_numpy(table).to("cuda:0"))
    for b, n in enumerate(lens):
        if n:
            k, v = synth.make_kv(77 + b, 1, n, 2, 128, BF16)
            gpu.append_seq(0, b, to_dev(k, BF16)[0], to_dev(v, BF16)[0])
            orc.append_seq(0, b, k[0], v[0])
    q = synth.make_q(78, B, 8, 128, BF16)
    want = orc.attend(0, q)
    for splits in (0, 1, 7):
        kv.kv_set_decode_splits(gpu.handle, splits)
        got = gpu.attend(0, to_dev(q, BF16)).cpu().numpy().astype(np.float64)
        assert (got[0] == 0).all()
        for b in range(1, B):
            assert np.max(np.abs(got[b] - want[b])) <= TOL, (splits, b)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("dtype", [F16, BF16])
@pytest.mark.parametrize("T", [1, 17, 161, 300, 5003])
def test_raw_layer_infinite_value_in_the_last_row(kv, oracle, T, dtype, paged):
    """The raw buffer's last chunk is short and its last value row holds an infinity of either sign in two
    channels: these are infinite in the output, as any weighted sum of the rows that exist is, and the others
    are those of finite rows."""
    import torch

    print("case raw layer infinity T=%d dtype=%d paged=%s" % (T, dtype, paged), flush=True)
    B, g, R = 2, 4, 32
    cap = (T // R + 2) * R
    assert T % R != 0
    cfg = kv.make_config(1, B, 2 * g, 2, 128, cap, R, R, R, dtype, 0, [16], [16], pool_blocks=B * cap // R if paged else 0)
    gpu = kv.KVCache(cfg)
    if paged:
        gpu.set_block_table(torch.arange(B * cap // R, dtype=torch.int32).view(B, -1).flip(1).contiguous().to("cuda:0"))
    orc = oracle.OracleCache(oracle.OracleConfig(1, B, 2 * g, 2, 128, cap, R, R, R, dtype, 0, [16], [16]))
    k, v = synth.make_kv(41 * T + dtype, B, T, 2, 128, dtype)
    k[:, T - 1] = 0  # score 0: the row's weight is far from binary32's smallest numbers
    inf = 0x7F80 if dtype == BF16 else 0x7C00
    v[1, T - 1, 0, 5], v[1, T - 1, 0, 70] = inf, inf | 0x8000
    append_both(gpu, orc, 0, k, v, dtype)
    q = synth.make_q(T, B, 2 * g, 128, dtype)
    want = orc.attend(0, q)
    for splits in (0, 1, 3):
        kv.kv_set_decode_splits(gpu.handle, splits)
        got = gpu.attend(0, to_dev(q, dtype)).cpu().numpy().astype(np.float64)
        assert np.all(got[1, :g, 5] == np.inf) and np.all(got[1, :g, 70] == -np.inf), splits
        finite = np.isfinite(want)
        assert np.count_nonzero(~finite) == 2 * g
        assert np.max(np.abs(got[finite] - want[finite])) <= TOL, splits


@pytest.mark.parametrize("T,splits", [(1040, 0), (8213, 0), (8213, 1), (8213, 4), (20011, 1)])
@pytest.mark.parametrize("dtype", [F16, BF16])
def test_raw_layer_error_no_larger_than_the_vector_alu_kernels(kv, T, splits, dtype):
    """Against 64 bits (2-norm over all heads) the matrix-core kernel of the 16-bit layers is no further off than
    the vector-ALU kernel with as many splits.  Both errors are means over 2 x 32 x 128 outputs of rounding errors of
    random sign: a tenth covers their spread from seed to seed."""
    import torch

    print("case raw layer error T=%d splits=%d dtype=%d" % (T, splits, dtype), flush=True)
    B, Hkv, g, R = 2, 8, 4, 32
    cfg = kv.make_config(1, B, Hkv * g, Hkv, 128, (T // R + 2) * R, R, R, R, dtype, 0, [16], [16])
    gpu = kv.KVCache(cfg)
    k, v = synth.make_kv_torch(51 + T, B, T, Hkv, 128, dtype, "cuda:0")
    gpu.append(0, k, v)
    q = synth.make_q_torch(52, B, Hkv * g, 128, dtype, "cuda:0")
    kd, vd = (x.double().permute(0, 2, 1, 3).contiguous() for x in (k, v))  # [B, Hkv, T, 128]
    s = torch.matmul(q.double().view(B, Hkv, g, 128), kd.transpose(2, 3).contiguous()) / 128 ** 0.5
    want = torch.matmul(torch.softmax(s, 3), vd).view(B, Hkv * g, 128)
    err = []
    for path in (0, 1):
        kv.kv_set_decode_path(gpu.handle, path)
        kv.kv_set_decode_splits(gpu.handle, splits)
        err.append(float((gpu.attend(0, q).double() - want).norm() / want.norm()))
    print("  matrix cores %.3e vector ALU %.3e" % tuple(err), flush=True)
    assert err[0] <= 1.1 * err[1]
