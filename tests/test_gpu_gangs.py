"""Tiles in gangs against the oracle: more tiles than one gang and some left over, a partial tile, a ragged last
chunk, tied chunks; decompress on the sizes where its gangs begin."""
import pytest

import oracle
from oracle import Config
from tests import parity
from tests.test_gpu_parity import H, make_inputs  # noqa: F401  (H: the fixture)
from tests.test_gpu_payload_formats import check_update, compress_case, oracle_payloads, update_on_samples, with_ties

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,k,bf16", [(16, 4, True), (32, 2, False), (32, 16, True), (64, 2, True), (64, 8, False),
                                      (64, 32, True), (128, 1, True), (128, 4, False), (128, 20, True), (128, 64, False)])
def test_compress(H, s, k, bf16):
    g, m, _ = make_inputs(s * (64 * (32 + 3) + 17) + 5, seed=k, grad_bf16=bf16)
    g, m = with_ties(g, m, s)
    cfg = Config(chunk=s, topk=k, decay=0.5)
    m_gpu, idx, val, coeff = H.gpu_compress(cfg, g, m)
    parity.check_compress(cfg, g, m, m_gpu, idx, val, coeff)


@pytest.mark.parametrize("s,k,val_dtype", [(64, 32, oracle.F16), (32, 16, oracle.BF16), (64, 8, oracle.F16)])
def test_compress_narrow(H, s, k, val_dtype):
    g, m, _ = make_inputs(s * (64 * 32 + 1), seed=k)
    compress_case(H, Config(chunk=s, topk=k), *with_ties(g, m, s), val_dtype, True)


@pytest.mark.parametrize("scheme", [oracle.SCHEME_STRIDE, oracle.SCHEME_RANDOM])
@pytest.mark.parametrize("s,k,bf16", [(64, 32, True), (64, 16, True), (32, 16, True), (64, 32, False)])
def test_schemes_on_coefficients(H, s, k, scheme, bf16):
    n = s * (64 * (32 + 1) + 9) + 3
    g, m, th = make_inputs(n, seed=k, grad_bf16=bf16, params_bf16=bf16)
    cfg = Config(chunk=s, topk=k, scheme=scheme, dct=True, seed=5, step=3)
    m_gpu, idx, val, coeff = H.gpu_compress(cfg, g, m)
    parity.check_compress(cfg, g, m, m_gpu, idx, val, coeff)
    idx, val = oracle_payloads(cfg, n, oracle.F32, 3, seed=7)
    check_update(H, cfg, idx, val, oracle.F32, False, th)


@pytest.mark.parametrize("s,k,val_dtype,bf16", [(16, 2, oracle.F32, True), (32, 8, oracle.F32, False), (32, 4, oracle.F16, True),
                                                (64, 32, oracle.BF16, False), (32, 16, oracle.TERNARY, True)])
def test_compress_in_a_row(H, s, k, val_dtype, bf16, monkeypatch):
    """The same kernels on shards below gangs (the tests' own choice is those of large shards)."""
    monkeypatch.setenv("DETO_SMALL_SHARD_TILES", "8192")
    g, m, _ = make_inputs(s * (64 * 3 + 17) + 5, seed=k, grad_bf16=bf16)
    compress_case(H, Config(chunk=s, topk=k), *with_ties(g, m, s), val_dtype, val_dtype != oracle.F32)


# large launches in gangs (tests/test_gangs.py asks the rule): every kernel, both parameter types
PLAIN = [(64, 32, 4, True), (64, 32, 2, False), (64, 16, 1, False), (32, 16, 5, True), (32, 8, 1, False), (32, 16, 8, False),
         (128, 32, 5, True), (128, 64, 1, False)]
ADAMW = [(64, 16, 2, oracle.F32, False, True), (64, 4, 2, oracle.F32, False, False), (32, 4, 2, oracle.F32, False, True),
         (64, 16, 2, oracle.F16, True, True), (128, 16, 2, oracle.BF16, True, False), (64, 16, 2, oracle.F32, True, False),
         (128, 32, 2, oracle.F32, False, True)]


def plain_size(s):
    return (1 << 25) + 64 * s * 3 + 7 * s + 11


def adamw_size(s):
    return (1 << 23) + 64 * s * 3 + 7 * s + 11


@pytest.mark.parametrize("s,k,R,bf16", PLAIN)
def test_decompress(H, s, k, R, bf16):
    cfg = Config(chunk=s, topk=k, sign=R != 5, weight_decay=0.1)
    n = plain_size(s)
    gangs = n // (s * 64) // 32                             # whole ones: the tiles after them are in a row
    update_on_samples(H, cfg, n, R, "f32+i32", bf16, at=((gangs // 2) * 2048 - 128, gangs * 2048 - 128))


@pytest.mark.parametrize("s,k,R,val_dtype,idx_u8,bf16", ADAMW)
def test_decompress_adamw(H, s, k, R, val_dtype, idx_u8, bf16):
    n = adamw_size(s)
    _, _, th = make_inputs(n, seed=k, params_bf16=bf16)
    cfg = Config(chunk=s, topk=k, weight_decay=0.1)
    idx, val = oracle_payloads(cfg, n, val_dtype, R, seed=k)
    check_update(H, cfg, idx, val, val_dtype, idx_u8, th, False)


# coefficients without indices, a lane per chunk: half of the chunk kept
@pytest.mark.parametrize("s,k,scheme", [(64, 32, oracle.SCHEME_RANDOM), (32, 16, oracle.SCHEME_STRIDE)])
def test_decompress_coefficients(H, s, k, scheme):
    cfg = Config(chunk=s, topk=k, scheme=scheme, dct=True, seed=3, step=2)
    n = (1 << 24) + 64 * s * 3 + 7 * s + 11
    update_on_samples(H, cfg, n, 3, "f32+i32", True, at=((n // (s * 2048) // 2) * 2048 - 128,))
