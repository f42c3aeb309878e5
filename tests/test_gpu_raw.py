"""Striding and Random on the momentum itself, streamed: the edges of a workgroup's run of chunks, k = 1 ... s/2, all
payload formats, index output, replicas beyond a batch of loads, both optimizers, and the large launches' rules,
against the oracle (and the kept bits of the momentum exactly)."""
import numpy as np
import pytest

import oracle
from oracle import Config
from tests import parity
from tests.test_gpu_parity import H, make_inputs  # noqa: F401  (H: the fixture)
from tests.test_gpu_payload_formats import FORMATS, check_update, compress_case, oracle_payloads, update_on_samples

pytestmark = pytest.mark.gpu
SCHEMES = [oracle.SCHEME_STRIDE, oracle.SCHEME_RANDOM]


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("s,k,elements", [
    (16, 1, 2048), (16, 8, 2048 * 2 + 16), (32, 3, 2048 * 2 - 1), (32, 16, 2048 + 1), (64, 2, 2048 * 3 + 63),
    (64, 32, 2048 * 2), (96, 5, 3072 + 95), (96, 48, 3072 * 2), (128, 16, 2048 * 2 + 128), (128, 32, 4096 * 2 - 127),
    (128, 64, 4096 + 3), (192, 7, 3072 * 2 + 1), (192, 96, 3072 - 5), (256, 1, 4096), (256, 128, 4096 * 2 + 255)])
def test_edges(H, s, k, elements, scheme):
    formats = list({"f32+i32": (oracle.F32, False), **FORMATS}.items())
    for i in {0, 1 + (s // 16 + k) % 5}:                   # (the other formats by turns)
        val_dtype, idx_u8 = formats[i][1]
        n = (1 << 17 if i == 0 and s <= 64 else 0) + elements   # (a lane per chunk serves smaller shards)
        cfg = Config(chunk=s, topk=k, scheme=scheme, sign=i % 2 == 0, lr=1e-3, seed=11, step=5 + i, weight_decay=0.1)
        g, m, th = make_inputs(n, seed=s + k + i, grad_bf16=i % 2 == 1, params_bf16=i % 3 == 0)
        compress_case(H, cfg, g, m, val_dtype, idx_u8)
        idx, val = oracle_payloads(cfg, n, val_dtype, (1, 9, 33, 2, 5, 17)[i], 300)
        check_update(H, cfg, idx, val, val_dtype, idx_u8, th)
        check_update(H, cfg, idx, val, val_dtype, idx_u8, th, adam=i % 2 == 0)


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("s,k,signs", [(128, 16, False), (64, 8, False), (32, 4, False), (32, 8, True), (96, 12, True),
                                       (48, 6, False), (48, 6, True)])          # (48: the general kernels)
def test_non_finite_values(H, s, k, signs, scheme):
    """What is kept is sent as it is and leaves nothing behind, an infinity or a NaN no more than a number; what is
    not stays as it is, and the rest of the chunk with it."""
    n = max(s * (64 + 3), (1 << 17) + s)                   # (a whole tile of chunks and some)
    cfg = Config(chunk=s, topk=k, scheme=scheme, seed=3, step=2)
    g, m, _ = make_inputs(n, seed=1)
    m[::97], m[1::97], m[2::97] = np.nan, np.inf, -np.inf
    if signs:
        m_gpu, idx, words, coeff = H.gpu_compress_ternary(cfg, g, m, True)
    else:
        m_gpu, idx, val, coeff = H.gpu_compress(cfg, g, m)
    kept = np.zeros(coeff.size, dtype=bool)
    at = np.repeat(np.arange(coeff.size // s) * s, k) + idx
    kept[at] = True
    assert (kept[:n] & ~np.isfinite(m)).any()
    assert np.array_equal(np.isfinite(m), np.isfinite(coeff[:n]))
    if signs:
        number = ~np.isnan(coeff[at])                      # (a NaN is sent as either sign)
        assert np.array_equal(oracle.decode_ternary(cfg, n, words)[number], np.sign(coeff[at][number]))
    else:
        assert np.array_equal(val.view(np.uint32), coeff[at].view(np.uint32))
    kept = kept[:n]
    assert np.array_equal(m_gpu[~kept].view(np.uint32), coeff[:n][~kept].view(np.uint32))
    assert not m_gpu[kept].view(np.uint32).any()


@pytest.mark.parametrize("k,val_dtype,Rs", [
    # entries four at a time: two, four, eight or sixteen replicas a batch; one by one: four, eight, sixteen, 32; signs: 3, 9, 18
    (32, oracle.F32, (2, 3, 4, 5, 9)), (32, oracle.F16, (2, 3, 4, 5, 9, 17)), (7, oracle.F32, (3, 4, 5, 9, 17, 33)),
    (7, oracle.BF16, (4, 5, 9, 17)), (8, oracle.F32, (9, 33)), (19, oracle.TERNARY, (3, 4, 9, 10, 18, 19, 37, 64))])
def test_batches_of_replicas(H, k, val_dtype, Rs):
    """Both sides of every batch of replicas: three payloads, moved by chunks, stand for R."""
    s = 64
    n = (1 << 17) + 5 * s + 7
    cfg = Config(chunk=s, topk=k, scheme=oracle.SCHEME_RANDOM, sign=False, lr=1e-3, seed=11, step=5)
    _, _, th = make_inputs(n, seed=k)
    three = oracle_payloads(cfg, n, val_dtype, 3, 300)
    unit = -(-k // 16) if val_dtype == oracle.TERNARY else k
    for R in Rs:
        idx = np.stack([three[0][r % 3] for r in range(R)])
        val = np.stack([np.roll(three[1][r % 3], r * unit, axis=0) for r in range(R)])
        check_update(H, cfg, idx, val, val_dtype, val_dtype != oracle.F32, th)


@pytest.mark.parametrize("s,k,R,fmt,bf16", [(64, 8, 4, "f32+i32", True), (64, 32, 4, "f32+i32", False),
                                            (128, 16, 9, "bf16+u8", True), (128, 8, 40, "signs+u8", False),
                                            (96, 12, 8, "f32+i32", False), (192, 24, 3, "f16+i32", True),
                                            (256, 64, 4, "f32+i32", True), (32, 8, 8, "f32+i32", False),
                                            # signs: batches of 33 replicas, words of one entry and of 16, odd k
                                            (32, 1, 64, "signs+u8", True), (32, 16, 33, "signs+u8", True),
                                            (64, 2, 34, "signs+u8", True), (16, 2, 16, "signs+u8", False),
                                            (64, 3, 2, "signs+u8", False), (128, 13, 5, "signs+u8", True)])
def test_large_launches(H, s, k, R, fmt, bf16):
    cfg = Config(chunk=s, topk=k, scheme=oracle.SCHEME_RANDOM, seed=3, step=2)
    update_on_samples(H, cfg, (1 << 23) + 8192 * 3 + 5 * s + 1, R, fmt, bf16)


@pytest.mark.parametrize("s,k,bf16", [(32, 4, True), (128, 16, False)])
def test_compress_with_fewer_workgroups(H, s, k, bf16):
    n = (1 << 24) + 4096 + 7
    g, m, _ = make_inputs(n, seed=k, grad_bf16=bf16)
    cfg = Config(chunk=s, topk=k, scheme=oracle.SCHEME_RANDOM, seed=3, step=2)
    m_gpu, idx, val, coeff = H.gpu_compress(cfg, g, m)
    parity.check_compress(cfg, g, m, m_gpu, idx, val, coeff)
