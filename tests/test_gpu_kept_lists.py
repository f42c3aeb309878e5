"""Top-k compress by coefficient classes, the launches that list their kept places: one to as many as the
partial sort holds, quads of entries and single ones, lists in a row's padding (up to 16), in the mask words
(192) and on their own (128 with two classes is in the tests of gangs), ties, a partial tile and a ragged last
chunk, against the oracle."""
import pytest

import oracle
from oracle import Config
from tests import parity
from tests.test_gpu_parity import H, make_inputs  # noqa: F401  (H: the fixture)
from tests.test_gpu_payload_formats import compress_case, with_ties

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,k,val_dtype,idx_u8", [
    (96, 1, oracle.F16, True), (96, 16, oracle.BF16, False), (128, 3, oracle.F32, True),
    (128, 16, oracle.F16, True), (192, 13, oracle.BF16, True), (192, 17, oracle.F16, True),
    (192, 32, oracle.F32, True)])
def test_formats_and_ties(H, s, k, val_dtype, idx_u8):
    for chunks, ragged in ((64 + 5, 7), (64, 0)):
        g, m, _ = make_inputs(s * chunks + ragged, seed=k)
        g, m = with_ties(g, m, s)
        compress_case(H, Config(chunk=s, topk=k, decay=0.5), g, m, val_dtype, idx_u8)


@pytest.mark.parametrize("s,k", [(64, 1), (64, 16), (96, 16), (128, 15), (128, 16), (192, 16), (192, 29),
                                 (192, 32)])
def test_plain_payload(H, s, k):
    g, m, _ = make_inputs(s * (64 + 63) + 1, seed=k)
    g, m = with_ties(g, m, s)
    cfg = Config(chunk=s, topk=k)
    m_gpu, idx, val, coeff = H.gpu_compress(cfg, g, m)
    parity.check_compress(cfg, g, m, m_gpu, idx, val, coeff)
