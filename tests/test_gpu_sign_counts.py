"""Two-bit signs without transmitted indices, counted a word at a time where there are many replicas: both sides of those
lines and replicas past one, two and three batches, words of one to sixteen entries and two a chunk, on a lane per chunk
and on classes, all fields of a word the same in every replica, codes that count as zero, against the oracle."""
import numpy as np
import pytest

import oracle
from oracle import Config
from tests.test_gpu_parity import H, make_inputs  # noqa: F401  (H: the fixture)
from tests.test_gpu_payload_formats import check_update, oracle_payloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,k,dct", [(32, 1, True), (32, 4, True), (32, 16, True), (32, 8, False), (64, 16, True),
                                     (64, 32, True), (64, 21, True), (16, 2, True), (128, 17, True), (256, 100, True)])
@pytest.mark.parametrize("R", [16, 31, 33, 48, 64])
def test_counts(H, s, k, dct, R):
    scheme = oracle.SCHEME_STRIDE if R % 2 and s % k == 0 else oracle.SCHEME_RANDOM
    n = s * 64 + 5 * s + 7
    cfg = Config(chunk=s, topk=k, scheme=scheme, dct=dct, sign=R != 33, lr=1e-3, seed=11, step=5, weight_decay=0.1)
    _, _, th = make_inputs(n, seed=s + k, params_bf16=R % 3 == 0)
    # (three replicas' payloads, moved by chunks, stand for R)
    idx, val = oracle_payloads(cfg, n, oracle.TERNARY, 3, 300)
    nw = -(-k // 16)
    idx = np.stack([idx[r % 3] for r in range(R)])
    val = np.stack([np.roll(val[r % 3], r * nw, axis=0) for r in range(R)])
    words = val.reshape(R, -1).view(np.uint32)
    for row, code in ((1, 0x55555555), (2, 0xFFFFFFFF), (3, 0xAAAAAAAA), (66, 0xE4E4E4E4)):
        words[:, row * nw:(row + 1) * nw] = code
    check_update(H, cfg, idx, val, oracle.TERNARY, True, th)
    check_update(H, cfg, idx, val, oracle.TERNARY, True, th, adam=R == 33)
