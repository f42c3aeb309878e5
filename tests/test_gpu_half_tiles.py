"""Chunk 256 with k <= 32: half of a tile in LDS at a time, kept sets as mask words and lists of places.
Both sort lengths at their ends, quads of entries and single ones, every payload format, tied chunks,
full tiles, a partial tile and a ragged last chunk, against the oracle."""
import numpy as np
import pytest

import oracle
from oracle import Config
from tests.test_gpu_parity import H, make_inputs  # noqa: F401  (H: the fixture)
from tests.test_gpu_payload_formats import compress_case, with_ties

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,val_dtype,idx_u8", [
    (1, oracle.F32, True), (4, oracle.F16, True), (15, oracle.BF16, False), (16, oracle.F32, True),
    (17, oracle.F16, True), (31, oracle.F32, True), (32, oracle.BF16, True)])
def test_formats_and_ties(H, k, val_dtype, idx_u8):
    s = 256
    for chunks, ragged in ((64 * 2 + 5, 7), (64, 0)):
        g, m, _ = make_inputs(s * chunks + ragged, seed=k)
        g, m = with_ties(g, m, s)
        compress_case(H, Config(chunk=s, topk=k, decay=0.5), g, m, val_dtype, idx_u8)


@pytest.mark.parametrize("k", [1, 6, 16, 29, 32])
def test_plain_payload_and_the_end_of_the_range(H, k):
    from tests import parity
    s = 256
    g, m, _ = make_inputs(s * (64 + 63) + 1, seed=k)
    g, m = with_ties(g, m, s)
    g[3 * s:4 * s] = np.float32(1e-41)                     # subnormal magnitudes at the threshold
    m[3 * s:4 * s] = 0
    cfg = Config(chunk=s, topk=k)
    m_gpu, idx, val, coeff = H.gpu_compress(cfg, g, m)
    parity.check_compress(cfg, g, m, m_gpu, idx, val, coeff)


@pytest.mark.parametrize("k,u8", [(5, False), (16, True), (32, False)])
def test_non_finite_chunks(H, k, u8):
    """More NaN coefficients than k, infinities and overflowing sums: such a chunk still sends k ascending
    places (a chunk of NaN the first k) and leaves the other chunks' bits alone."""
    import torch
    from paper_2502_06728_amd import binding
    s, chunks = 256, 64 + 9
    g, m, _ = make_inputs(s * chunks, seed=k)
    bad, results = {2: float("nan"), 30: float("inf"), 66: float("nan"), 70: 3e38}, []
    for values in ({}, bad):
        mom = m.copy()
        for c, x in values.items():
            mom[c * s + 3] = x
            mom[c * s + 200] = -x
        mom, grad = torch.from_numpy(mom).to(H.DEV), torch.from_numpy(g).to(H.DEV)
        idx = torch.zeros(chunks * k, dtype=torch.uint8 if u8 else torch.int32, device=H.DEV)
        val = torch.zeros(chunks * k, device=H.DEV)
        for _ in range(2):
            binding.detonation_compress_packed(binding.Config(chunk=s, topk=k), grad, mom, idx, val)
        torch.cuda.synchronize()
        results.append((mom.cpu().numpy().view(np.uint32).reshape(chunks, s),
                        idx.cpu().numpy().astype(np.int64).reshape(chunks, k),
                        val.cpu().numpy().view(np.uint32).reshape(chunks, k)))
    others = [c for c in range(chunks) if c not in bad]
    for a, b in zip(*results):
        assert np.array_equal(a[others], b[others])
    idx = results[1][1]
    assert (np.diff(idx, axis=1) > 0).all() and idx.min() >= 0 and idx.max() < s
    for c in (2, 66):
        assert np.array_equal(idx[c], np.arange(k))
