"""The matrix-core compress kernels that stand in for the general ones (two-bit signs, chunk 16) give
the general kernels' bits: the same call with the momentum one element off its 16-byte alignment
goes to the general kernels, whose selection the oracle checks elsewhere."""
import pytest

from tests.test_gpu_parity import H  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

F32, BF16, F16, SIGNS = 0, 1, 2, 3


def run(H, s, k, n, val, u8, bf16, aligned):
    """Three calls on an evolving momentum: what every one leaves."""
    import torch
    from paper_2502_06728_amd import binding
    gen = torch.Generator(device=H.DEV)
    gen.manual_seed(s * 1000 + k)
    C = -(-n // s)
    g = torch.randn(n, generator=gen, device=H.DEV)
    g[:s * (C // 3)] = (g[:s * (C // 3)] * 4).round()        # many equal magnitudes
    m = torch.empty(n + 1, device=H.DEV)[:n] if aligned else torch.empty(n + 1, device=H.DEV)[1:]
    m.copy_(torch.randn(n, generator=gen, device=H.DEV))
    for c in range(0, C, 7):                                 # zero chunks and single spikes
        g[c * s:(c + 1) * s] = 0
        m[c * s:(c + 1) * s] = 0
        if c % 2:
            m[c * s + (5 * c) % (min(n, (c + 1) * s) - c * s)] = 1e-3 * (c + 1)
    m[2 * s:3 * s] *= 1e-38                                  # subnormal products,
    g[2 * s:3 * s] = 0
    m[3 * s:4 * s] = 3e38                                    # sums that overflow,
    m[4 * s + 1] = float("inf")                              # infinities and NaN in the input
    m[5 * s - 1] = -float("inf")
    m[s + s // 2] = float("nan")
    g = g.to(torch.bfloat16) if bf16 else g
    words = C * ((k + 15) // 16)
    idx = torch.zeros(C * k, dtype=torch.uint8 if u8 else torch.int32, device=H.DEV)
    v = torch.zeros(words if val == SIGNS else C * k, device=H.DEV,
                    dtype={F32: torch.float32, BF16: torch.bfloat16, F16: torch.float16,
                           SIGNS: torch.int32}[val])
    cfg, out = binding.Config(chunk=s, topk=k, decay=0.9), []

    def bits(t):
        if t.is_floating_point():                            # (a NaN's sign and payload are free)
            t = torch.where(t.isnan(), torch.full_like(t, float("nan")), t)
        return t.clone() if t.element_size() == 1 else t.view(
            torch.int16 if t.element_size() == 2 else torch.int32).clone()

    for call in range(3):
        coeff = torch.zeros(C * s, device=H.DEV)
        binding.detonation_compress_packed(cfg, g, m, idx, v, coeff)
        out += [bits(t) for t in (m, idx, v, coeff)]
    torch.cuda.synchronize()
    return out


# (k: one entry, a remainder of four, a multiple of four over a word's sixteen signs, all but one, all)
@pytest.mark.parametrize("s,k,val,u8,bf16", [
    (16, 1, SIGNS, True, True), (16, 4, F16, True, False), (16, 7, BF16, False, True),
    (16, 16, F32, True, False), (16, 15, F32, False, True), (32, 20, SIGNS, False, False),
    (64, 3, SIGNS, True, False), (64, 63, SIGNS, False, True), (96, 48, SIGNS, True, True),
    (128, 17, SIGNS, True, False), (128, 128, SIGNS, True, True), (160, 40, SIGNS, False, False),
    (192, 6, SIGNS, True, True), (224, 28, SIGNS, True, False), (256, 1, SIGNS, False, True),
    (256, 128, SIGNS, True, False), (256, 255, SIGNS, True, True)])
def test_bits_of_the_general_kernels(H, s, k, val, u8, bf16):
    import torch
    few = 4096 if s <= 32 else 2048 if s == 64 else 0        # (served by the general kernels anyway)
    for chunks in (few + 97, few + 64) + ((5,) if few == 0 else ()):   # whole tiles; a partial tile
        for ragged in (0, 3):
            n = s * chunks + ragged
            for a, b in zip(run(H, s, k, n, val, u8, bf16, True), run(H, s, k, n, val, u8, bf16, False)):
                assert torch.equal(a, b), (chunks, ragged, int((a != b).sum()))
