"""Every payload format (fp32, bf16, fp16 or two-bit signs; int32 or byte indices) at the chunk
sizes and k values that share run-time kernels, both halves against the oracle: full tiles, a
partial tile, a ragged last chunk, tied chunks, more replicas than one batch of loads."""
import numpy as np
import pytest

import oracle
from oracle import Config
from tests import parity
from tests.test_gpu_parity import H, make_inputs  # noqa: F401  (H: the fixture)

pytestmark = pytest.mark.gpu

FORMATS = {"bf16+u8": (oracle.BF16, True), "f16+i32": (oracle.F16, False),
           "signs+u8": (oracle.TERNARY, True), "signs+i32": (oracle.TERNARY, False),
           "f32+u8": (oracle.F32, True)}


def with_ties(g, m, s):
    """Zero chunks, and chunks of equal magnitudes, among the ordinary ones."""
    g, m = g.copy(), m.copy()
    C = g.size // s
    for c in range(0, C, 5):
        g[c * s:(c + 1) * s] = 0
        m[c * s:(c + 1) * s] = 0
        if c % 2:
            m[c * s + (7 * c) % s] = 1.0 + c
    return g, m


def device_payload(H, val, val_dtype, idx, idx_u8):
    import torch
    i = None
    if idx is not None:
        i = torch.from_numpy(np.ascontiguousarray(idx.astype(np.uint8 if idx_u8 else np.int32))).to(H.DEV)
    if val_dtype == oracle.TERNARY:
        return i, torch.from_numpy(np.ascontiguousarray(val).view(np.int32)).to(H.DEV)
    if val_dtype == oracle.F32:
        return i, torch.from_numpy(np.ascontiguousarray(val)).to(H.DEV)
    return i, H.bits16_to_dev(np.ascontiguousarray(val), val_dtype)


def compress_case(H, cfg, g, m, val_dtype, idx_u8):
    import torch
    from paper_2502_06728_amd import binding
    n, s, k = m.size, cfg.chunk, cfg.topk
    C = -(-n // s)
    if val_dtype == oracle.TERNARY:
        m_gpu, idx, words, coeff = H.gpu_compress_ternary(cfg, g, m, idx_u8)
        kept = coeff.reshape(C, s)[np.arange(C)[:, None], idx.reshape(C, k)].reshape(-1)
        parity.check_compress(cfg, g, m, m_gpu, idx, kept, coeff)
        assert np.array_equal(words, oracle.encode_ternary(cfg, n, kept))
    elif val_dtype == oracle.F32:
        gm = H.to_dev(m)
        idx = torch.zeros(C * k, dtype=torch.uint8 if idx_u8 else torch.int32, device=H.DEV)
        val = torch.zeros(C * k, dtype=torch.float32, device=H.DEV)
        coeff = torch.zeros(C * s, dtype=torch.float32, device=H.DEV)
        binding.detonation_compress_packed(H.bcfg(cfg), H.to_dev(g), gm, idx, val, coeff)
        torch.cuda.synchronize()
        parity.check_compress(cfg, g, m, H.to_host(gm), idx.cpu().numpy().astype(np.int32),
                              H.to_host(val), H.to_host(coeff))
    else:
        m_gpu, idx, vbits, coeff = H.gpu_compress_packed(cfg, g, m, val_dtype, idx_u8)
        parity.check_compress_packed(cfg, g, m, m_gpu, idx, vbits, coeff, val_dtype)


def oracle_payloads(cfg, n, val_dtype, R, seed):
    """R replicas' (idx [R, C*k], val, the values the receivers decode)."""
    f = {oracle.TERNARY: oracle.compress_t, oracle.F32: oracle.compress}.get(
        val_dtype, lambda c, g, m: oracle.compress_q(c, g, m, val_dtype))
    pays = [f(cfg, *make_inputs(n, seed=seed + r)[:2])[1:] for r in range(R)]
    return np.stack([p[0] for p in pays]), np.stack([p[1] for p in pays])


def check_presign(cfg, n, idx, val, val_dtype, y):
    """The averaged update before the sign against the oracle's, on the scale of the chunk's result and
    of its largest payload value (the sum over replicas can cancel)."""
    s, k, C = cfg.chunk, cfg.topk, -(-n // cfg.chunk)
    if val_dtype == oracle.TERNARY:
        want, decoded = oracle.presign_t(cfg, n, idx, val), np.ones((1, C, k))
    elif val_dtype == oracle.F32:
        want, decoded = oracle.presign(cfg, n, idx, val), val
    else:
        want = oracle.presign_q(cfg, n, idx, val, val_dtype)
        decoded = ((val.astype(np.uint32) << 16).view(np.float32) if val_dtype == oracle.BF16
                   else val.view(np.float16).astype(np.float32))
    largest = np.abs(decoded.astype(np.float64).reshape(-1, C, k)).max(axis=(0, 2))
    scale = np.maximum(np.repeat(largest, s)[:n], parity.parity_chunk_max(want, s))
    err = parity.rel_chunk_err(y, want, s, scale=scale)
    assert err <= parity.TOL_F32, f"pre-sign update differs: {err:.3e}"


def check_update(H, cfg, idx, val, val_dtype, idx_u8, th, adam=None):
    """Decompress on the device and judge it by the oracle on the same payload bytes."""
    import torch
    from paper_2502_06728_amd import binding
    n, s, R = th.size, cfg.chunk, val.shape[0]
    send = cfg.scheme == oracle.SCHEME_TOPK
    i, v = device_payload(H, val, val_dtype, idx if send else None, idx_u8)
    p = H.to_dev(th)
    y = torch.full((n,), float("nan"), dtype=torch.float32, device=H.DEV)
    if adam is None:
        binding.detonation_decompress_step_packed(H.bcfg(cfg), R, i, v, p, y)
        torch.cuda.synchronize()
        if val_dtype == oracle.TERNARY:
            val = np.stack([oracle.decode_ternary(cfg, n, w) for w in val])
        if val_dtype in (oracle.TERNARY, oracle.F32):
            parity.check_decompress(cfg, idx, val, th, H.to_host(p), H.to_host(y))
        else:
            parity.check_decompress_packed(cfg, idx, val, val_dtype, th, H.to_host(p), H.to_host(y))
        return
    rng = np.random.default_rng(n)
    m0 = rng.standard_normal(n).astype(np.float32)
    v0 = (rng.random(n) + 0.1).astype(np.float32)
    ma, va, vm = H.to_dev(m0), H.to_dev(v0), H.to_dev(v0)
    opt = binding.AdamW(0.9, 0.95, 1e-8, adam, 3)
    binding.detonation_decompress_adamw_step_packed(H.bcfg(cfg), opt, R, i, v, p, ma, va,
                                                    vm if adam else None, y)
    torch.cuda.synchronize()
    # (AdamW may run on other kernels than the plain update: its pre-sign update has its own check)
    check_presign(cfg, n, idx, val, val_dtype, H.to_host(y))
    # Q as the device computed it drives the oracle
    th_o, m_o, v_o, vm_o = oracle.adamw_update(cfg, oracle.AdamW(0.9, 0.95, 1e-8, adam, 3),
                                               H.to_host(y), th, m0, v0, v0)
    assert np.abs(H.to_host(ma) - m_o).max() <= 1e-5 * np.abs(m_o).max()
    assert np.abs(H.to_host(va) - v_o).max() <= 1e-5 * np.abs(v_o).max()
    if adam:
        assert np.abs(H.to_host(vm) - vm_o).max() <= 1e-5 * np.abs(vm_o).max()
    got, want, tol = H.to_host(p), th_o, parity.TOL_F32
    if th.dtype == np.uint16:
        from paper_2502_06728_amd import synth
        got, want, tol = synth.from_bf16_bits(got), synth.from_bf16_bits(th_o), parity.TOL_BF16
    got, want = got.astype(np.float64), want.astype(np.float64)
    assert (np.abs(got - want) <= tol * np.abs(want) + tol * cfg.lr).all()


TOPK_SHAPES = [(16, 1), (16, 2), (16, 3), (16, 8), (32, 1), (32, 3), (32, 12), (64, 1), (64, 2), (64, 5), (64, 20), (96, 3), (96, 20), (96, 48), (128, 7), (128, 16),
               (128, 64), (192, 6), (192, 24), (192, 33), (192, 96), (256, 8), (256, 32), (256, 33),
               (256, 128)]


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("s,k", TOPK_SHAPES)
def test_topk(H, s, k, fmt):
    val_dtype, idx_u8 = FORMATS[fmt]
    bf16 = k % 2 == 0
    # two full tiles, then a partial one of 37 chunks and a ragged one
    n = s * (64 * 2 + 37) + s // 3
    cfg = Config(chunk=s, topk=k, sign=True, lr=1e-3, weight_decay=0.01)
    g, m, th = make_inputs(n, seed=s + k, params_bf16=bf16)
    compress_case(H, cfg, *with_ties(g, m, s), val_dtype, idx_u8)
    idx, val = oracle_payloads(cfg, n, val_dtype, 6, 700)
    check_update(H, cfg, idx, val, val_dtype, idx_u8, th)
    check_update(H, cfg, idx, val, val_dtype, idx_u8, th, adam=bool(k % 3 == 0))


@pytest.mark.parametrize("fmt", ["bf16+u8", "signs+i32", "f32+u8"])
@pytest.mark.parametrize("s,k", [(16, 4), (32, 5), (64, 5), (96, 12), (128, 3), (192, 24), (256, 10)])
def test_unordered_payloads(H, s, k, fmt):
    """Duplicates and disorder add like the scatter-add they are; indices past the chunk are skipped."""
    val_dtype, idx_u8 = FORMATS[fmt]
    n = s * (64 + 9)
    C, R = n // s, 3
    cfg = Config(chunk=s, topk=k, sign=False)
    rng = np.random.default_rng(s * k)
    top = min(s + 3, 256)
    idx = np.stack([np.sort(rng.integers(0, s, size=(C, k)), axis=1).reshape(-1),     # repeats
                    rng.integers(0, top, size=C * k),                                  # anything
                    np.tile(np.arange(k), C)]).astype(np.int32)
    val = oracle_payloads(cfg, n, val_dtype, R, 40)[1]
    check_update(H, cfg, idx, val, val_dtype, idx_u8, make_inputs(n, 3)[2])


SCHEME_SHAPES = [(16, 3), (16, 8), (32, 3), (64, 2), (64, 7), (96, 12), (128, 4), (128, 16), (128, 64),
                 (192, 5), (256, 32), (256, 127)]


@pytest.mark.parametrize("fmt", ["f32+i32", "bf16+u8", "f16+i32", "signs+u8"])
@pytest.mark.parametrize("scheme", [oracle.SCHEME_STRIDE, oracle.SCHEME_RANDOM])
@pytest.mark.parametrize("dct", [False, True])
@pytest.mark.parametrize("s,k", SCHEME_SHAPES)
def test_striding_and_random(H, s, k, dct, scheme, fmt):
    val_dtype, idx_u8 = FORMATS.get(fmt, (oracle.F32, False))
    n = s * (64 + 37) + s // 3        # a full tile, 37 chunks and a ragged one
    cfg = Config(chunk=s, topk=k, scheme=scheme, dct=dct, sign=True, lr=1e-3, seed=11, step=5)
    g, m, th = make_inputs(n, seed=s + k, params_bf16=k % 2 == 0)
    compress_case(H, cfg, g, m, val_dtype, idx_u8)
    idx, val = oracle_payloads(cfg, n, val_dtype, 9 if k < 16 else 3, 300)
    check_update(H, cfg, idx, val, val_dtype, idx_u8, th)
    check_update(H, cfg, idx, val, val_dtype, idx_u8, th, adam=bool(k % 3 == 0))


@pytest.mark.parametrize("fmt", ["f32+i32", "bf16+u8", "signs+u8"])
@pytest.mark.parametrize("scheme", [oracle.SCHEME_STRIDE, oracle.SCHEME_RANDOM])
@pytest.mark.parametrize("s,k", [(64, 2), (96, 12), (128, 16), (128, 64), (192, 5), (256, 127)])
def test_striding_and_random_on_many_chunks(H, s, k, scheme, fmt):
    """In the raw domain up to 5,120 chunks stay on the general kernels: more than that."""
    val_dtype, idx_u8 = FORMATS.get(fmt, (oracle.F32, False))
    n = s * (64 * 81 + 37) + s // 3
    cfg = Config(chunk=s, topk=k, scheme=scheme, sign=True, lr=1e-3, seed=11, step=5)
    g, m, th = make_inputs(n, seed=s + k, params_bf16=k % 2 == 0)
    compress_case(H, cfg, g, m, val_dtype, idx_u8)
    idx, val = oracle_payloads(cfg, n, val_dtype, 3, 300)
    check_update(H, cfg, idx, val, val_dtype, idx_u8, th)
    check_update(H, cfg, idx, val, val_dtype, idx_u8, th, adam=bool(k % 3 == 0))


@pytest.mark.parametrize("s,k", [(128, 16), (64, 5), (256, 40)])
def test_random_without_index_output(H, s, k):
    """No index array at all, and a caller that passes indices in the raw domain."""
    import torch
    from paper_2502_06728_amd import binding
    n = s * (64 + 5) + 3
    cfg = Config(chunk=s, topk=k, scheme=oracle.SCHEME_RANDOM, seed=2, step=9, sign=False)
    g, m, th = make_inputs(n, seed=k)
    m_gpu, _, words, _ = H.gpu_compress_ternary(cfg, g, m, False, want_idx=False)
    m_o, idx_o, words_o = oracle.compress_t(cfg, g, m)
    assert np.array_equal(words, words_o) and np.array_equal(m_gpu, m_o)
    signs = oracle.decode_ternary(cfg, n, words_o)[None, :]
    p, y = H.to_dev(th), torch.empty(n, dtype=torch.float32, device=H.DEV)
    binding.detonation_decompress_step_packed(
        H.bcfg(cfg), 1, torch.from_numpy(idx_o.astype(np.uint8)).to(H.DEV),
        torch.from_numpy(words_o.view(np.int32)).to(H.DEV), p, y)
    torch.cuda.synchronize()
    parity.check_decompress(cfg, idx_o[None, :], signs, th, H.to_host(p), H.to_host(y))


@pytest.mark.parametrize("s,k,fmt", [(16, 4, "bf16+u8"), (16, 8, "f32+u8"), (16, 3, "signs+u8"),
                                     (32, 16, "signs+i32"), (64, 2, "signs+u8"), (64, 20, "signs+i32"),
                                     (96, 12, "signs+u8"), (128, 64, "signs+u8"), (192, 24, "signs+i32"),
                                     (256, 32, "signs+u8")])
def test_results_do_not_depend_on_alignment(H, s, k, fmt):
    """Sign payloads without a lane-per-chunk kernel, and narrow payloads at chunk 16: three calls in a
    row give the same bits on aligned buffers as on unaligned ones, which only the general
    kernels take.  (Momenta that differ in rounding alone, as those of another transform do, make
    near ties fall differently from the second call on.)"""
    import torch
    from paper_2502_06728_amd import binding
    val_dtype, idx_u8 = FORMATS[fmt]
    # (above the number of chunks up to which the general kernels serve aligned buffers too)
    n = s * (64 * {16: 65, 32: 65, 64: 33}.get(s, 8) + 37) + s // 3
    cfg = Config(chunk=s, topk=k, sign=True)
    g, m, _ = make_inputs(n, seed=s * k)
    g = torch.from_numpy(g).to(H.DEV)
    C = -(-n // s)
    length = C * -(-k // 16) if val_dtype == oracle.TERNARY else C * k
    types = {oracle.TERNARY: torch.int32, oracle.F32: torch.float32, oracle.BF16: torch.bfloat16}
    results = []
    for shift in (0, 1):
        mom = torch.empty(n + shift, dtype=torch.float32, device=H.DEV)[shift:]
        mom.copy_(torch.from_numpy(m))
        idx = torch.zeros(C * k, dtype=torch.uint8 if idx_u8 else torch.int32, device=H.DEV)
        val = torch.zeros(length, dtype=types[val_dtype], device=H.DEV)
        out = []
        for _ in range(3):
            binding.detonation_compress_packed(H.bcfg(cfg), g, mom, idx, val)
            out += [mom.clone(), idx.clone(), val.clone()]
        results.append(out)
    torch.cuda.synchronize()
    for a, b in zip(*results):
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


@pytest.mark.parametrize("fmt", ["bf16+u8", "f16+i32", "f32+u8"])
@pytest.mark.parametrize("s,k", [(96, 12), (128, 4), (128, 64), (192, 24), (192, 96), (256, 8), (256, 128)])
def test_both_kernels_sum_alike(H, s, k, fmt):
    """Narrow payloads above chunk 64 run with a wavefront per coefficient class up to k = s/2 and with
    two lanes per chunk beyond: the same coefficients bit for bit, so that a kernel's choice does
    not move near ties."""
    val_dtype, idx_u8 = FORMATS[fmt]
    n = s * 64 * 4
    g, m, _ = make_inputs(n, seed=s + k)
    coeffs = []
    for kk in (k, s // 2 + 1):
        cfg = Config(chunk=s, topk=kk, sign=True)
        if val_dtype == oracle.F32:
            import torch
            from paper_2502_06728_amd import binding
            C = n // s
            coeff = torch.zeros(n, dtype=torch.float32, device=H.DEV)
            binding.detonation_compress_packed(
                H.bcfg(cfg), H.to_dev(g), H.to_dev(m), torch.zeros(C * kk, dtype=torch.uint8, device=H.DEV),
                torch.zeros(C * kk, dtype=torch.float32, device=H.DEV), coeff)
            torch.cuda.synchronize()
            coeffs.append(H.to_host(coeff))
        else:
            coeffs.append(H.gpu_compress_packed(cfg, g, m, val_dtype, idx_u8)[3])
    assert np.array_equal(coeffs[0].view(np.uint32), coeffs[1].view(np.uint32))


def update_on_samples(H, cfg, n, R, fmt, bf16, at=()):
    """Decompress of n parameters from payloads drawn on the device; the first, the last and some other
    runs of chunks against the oracle."""
    import torch
    from paper_2502_06728_amd import binding, synth
    val_dtype, idx_u8 = FORMATS.get(fmt, (oracle.F32, False))
    s, k, send = cfg.chunk, cfg.topk, cfg.scheme == oracle.SCHEME_TOPK
    C = -(-n // s)
    gen = torch.Generator(device=H.DEV)
    gen.manual_seed(s * k)
    params = (torch.randn(n, generator=gen, device=H.DEV) * 0.02).to(torch.bfloat16 if bf16 else torch.float32)
    before = params.clone()
    y = torch.full((n,), float("nan"), dtype=torch.float32, device=H.DEV)
    idx = None
    if send:     # ascending places, others in every chunk and replica
        step = s // k
        first = torch.randint(0, step, (R, C, 1), generator=gen, device=H.DEV)
        idx = (first + step * torch.arange(k, device=H.DEV)).to(torch.uint8 if idx_u8 else torch.int32)
    if val_dtype == oracle.TERNARY:
        assert k <= 16
        code = torch.randint(0, 3, (R, C, k), generator=gen, device=H.DEV)
        code = torch.where(code == 2, 3, code)
        val = (code << (2 * torch.arange(k, device=H.DEV))).sum(-1).to(torch.int32).reshape(R, C, 1)
    else:
        val = torch.randn((R, C, k), generator=gen, device=H.DEV).to(H.VAL_TORCH[val_dtype])
    binding.detonation_decompress_step_packed(H.bcfg(cfg), R, None if idx is None else idx.reshape(R, -1),
                                              val.reshape(R, -1), params, y)
    torch.cuda.synchronize()
    tol = parity.TOL_BF16 if bf16 else parity.TOL_F32
    for c0 in (0, C // 3, *at, C - 256):
        c1 = min(c0 + 256, C)
        e0, e1 = c0 * s, min(c1 * s, n)
        v = val[:, c0:c1].contiguous().cpu()
        if val_dtype == oracle.TERNARY:
            v = v.numpy().view(np.uint32).reshape(R, -1)
        elif val_dtype == oracle.F32:
            v = v.numpy().reshape(R, -1)
        else:
            v = v.view(torch.int16).numpy().view(np.uint16).reshape(R, -1)
        if send:
            i = idx[:, c0:c1].to(torch.int32).cpu().numpy().reshape(R, -1)
        else:
            kept = oracle.select(cfg, np.zeros((c1 - c0) * s, dtype=np.float32), chunk0=c0)
            i = np.tile(kept.reshape(1, -1), (R, 1))
        got_y = H.to_host(y[e0:e1])
        check_presign(cfg, e1 - e0, i, v, val_dtype, got_y)
        got, want = H.to_host(params[e0:e1]), oracle.update(cfg, got_y, H.to_host(before[e0:e1]))
        if bf16:
            got, want = synth.from_bf16_bits(got), synth.from_bf16_bits(want)
        got, want = got.astype(np.float64), want.astype(np.float64)
        assert (np.abs(got - want) <= tol * np.abs(want) + tol * cfg.lr).all()


@pytest.mark.parametrize("s,k,R,fmt", [
    (32, 8, 4, "f32+i32"), (32, 4, 16, "f32+i32"), (64, 8, 4, "f32+i32"), (64, 32, 2, "f32+i32"),
    (64, 5, 3, "f32+i32"), (96, 5, 3, "f32+i32"), (96, 12, 2, "f32+i32"), (96, 20, 2, "bf16+u8"),
    (128, 1, 9, "f32+i32"), (128, 4, 3, "f32+i32"), (128, 8, 2, "f32+i32"), (128, 32, 2, "f32+i32"),
    (128, 5, 3, "f32+i32"), (128, 16, 3, "f16+i32"), (128, 5, 2, "signs+u8")])
def test_large_bf16_shards(H, s, k, R, fmt):
    """Above 2^25 bf16 parameters decompress takes other kernels (a lane per chunk at chunk 128, two
    classes without one, more classes at chunk 32 and 64)."""
    cfg = Config(chunk=s, topk=k, sign=True, lr=1e-3, weight_decay=0.01)
    update_on_samples(H, cfg, (1 << 25) + s * (64 * 3 + 37) + s // 3, R, fmt, True, at=((1 << 25) // s - 128,))


@pytest.mark.parametrize("s,k,R,tiles,fmt,bf16", [
    # a lane per chunk about one round long; many entries per element
    (96, 6, 2, 700, "f32+i32", False), (96, 24, 2, 1020, "f32+i32", False), (128, 1, 3, 700, "f32+i32", False),
    (128, 4, 2, 700, "f32+i32", False), (128, 16, 2, 700, "f32+i32", False), (128, 32, 2, 700, "f32+i32", True),
    (96, 48, 16, 5, "f32+i32", False), (128, 64, 16, 5, "f32+i32", False), (32, 16, 16, 1600, "f32+i32", False),
    (64, 32, 16, 5, "f32+i32", True),
    # two classes on many tiles, four at more entries
    (32, 3, 2, 1100, "f16+i32", False), (64, 5, 2, 1100, "signs+u8", False), (64, 2, 3, 1600, "f32+i32", False),
    (64, 8, 2, 1600, "bf16+u8", False), (64, 16, 3, 1600, "f32+i32", False), (32, 8, 2, 1600, "f32+i32", False)])
def test_launches_of_many_tiles(H, s, k, R, tiles, fmt, bf16):
    cfg = Config(chunk=s, topk=k, sign=True, lr=1e-3, weight_decay=0.01)
    update_on_samples(H, cfg, s * (64 * tiles + 37) + s // 3, R, fmt, bf16)


@pytest.mark.parametrize("dct", [False, True])
@pytest.mark.parametrize("scheme", [oracle.SCHEME_STRIDE, oracle.SCHEME_RANDOM])
@pytest.mark.parametrize("s,k,tiles,fmt", [(64, 8, 3100, "f32+i32"), (64, 8, 3100, "signs+u8"),
                                           (64, 4, 3100, "bf16+u8"), (32, 4, 3100, "f32+i32"),
                                           (32, 2, 3100, "signs+u8"), (16, 1, 6200, "f32+i32"),
                                           (64, 2, 1100, "signs+u8")])
def test_low_rates_on_many_tiles(H, s, k, tiles, fmt, scheme, dct):
    cfg = Config(chunk=s, topk=k, scheme=scheme, dct=dct, sign=True, lr=1e-3, seed=4, step=9)
    update_on_samples(H, cfg, s * (64 * tiles + 37) + s // 3, 3, fmt, False)
