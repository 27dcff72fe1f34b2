"""GPU parity of the decoder-block glue on 16-bit integer activations
against the CPU oracle.

Residual add, table lookups and RMSNorm are bit-exact (the same IEEE fp64
operations in the same order; sqrt and division are correctly rounded on
both sides).  SiLU tables and softmax go through exp, whose last bit IEEE
does not fix, and softmax sums in a different order: their codes must be
equal except at rounding ties of the fp64 value (|frac - 1/2| < 1e-9),
where one step either way is allowed.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _mq():
    import paper_2408_13933_amd as mq
    return mq


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _equal_but_ties(got, ref, pre, max_frac=1e-3):
    """Codes equal except one step where the fp64 value `pre` (in output
    steps, before the zero-point) lies within 1e-9 of a half-integer."""
    got = got.astype(np.int64)
    ref = ref.astype(np.int64)
    f = pre - np.floor(pre)
    tie = np.abs(f - 0.5) < 1e-9
    bad = (got != ref) & ~(tie & (np.abs(got - ref) <= 1))
    assert not np.any(bad), (np.argwhere(bad)[:5], got[bad][:5], ref[bad][:5])
    assert np.mean(got != ref) < max_frac


def _rope_pre(x, heads, ax, zx, ay, pos0=0, base=10000.0):
    """fp64 rotary embedding of the dequantized codes, in output steps
    (pairs i and i + D/2, angle (t + pos0) * base^(-2i/D))."""
    T, HD = x.shape
    D = HD // heads
    xh = (np.float64(np.float32(ax)) * (x.astype(np.float64) - zx)).reshape(T, heads, D)
    inv = base ** (-np.arange(0, D, 2, dtype=np.float64) / D)
    ang = (np.arange(T, dtype=np.float64) + pos0)[:, None] * inv[None, :]
    c, s = np.cos(ang)[:, None, :], np.sin(ang)[:, None, :]
    u, w = xh[..., :D // 2], xh[..., D // 2:]
    pre = np.concatenate([u * c - w * s, w * c + u * s], axis=-1).reshape(T, HD)
    return pre / np.float64(np.float32(ay))


@pytest.mark.parametrize("n", [1, 777, 1024 * 2048])
@pytest.mark.parametrize("out_bits", [16, 8])
def test_add_requant_parity(n, out_bits):
    mq = _mq()
    rng = np.random.default_rng(n + out_bits)
    x1 = rng.integers(-32768, 32768, n).astype(np.int16)
    x2 = rng.integers(-32768, 32768, n).astype(np.int16)
    args = (3.1e-4, -12, 7.7e-4, 300, 1.3e-3 if out_bits == 16 else 0.4, 5)
    y = mq.mq_add_requant(_dev(x1), args[0], args[1], _dev(x2), args[2], args[3], args[4],
                          args[5], out_bits)
    ref = oracle.add_requant(x1, args[0], args[1], x2, args[2], args[3], args[4], args[5],
                             out_bits)
    assert np.array_equal(y.cpu().numpy(), ref)


@pytest.mark.parametrize("ax,zx,ay,zy,out_bits", [(1e-3, -100, 0.05, 3, 8),
                                                  (4e-4, 0, 2e-4, -7, 16),
                                                  (2e-2, 1000, 0.03, 0, 8)])
def test_silu_table_and_lookup(ax, zx, ay, zy, out_bits):
    mq = _mq()
    lut = mq.mq_lut_build(mq.LUT_SILU, ax, zx, ay, zy, out_bits).cpu().numpy()
    ref = oracle.lut_build(oracle.LUT_SILU, ax, zx, ay, zy, out_bits)
    i = np.arange(-32768, 32768)
    v = np.float64(np.float32(ax)) * (i - zx)
    with np.errstate(over="ignore"):
        pre = v / (1.0 + np.exp(-v)) / np.float64(np.float32(ay))
    _equal_but_ties(lut, ref, pre)
    # the lookup itself, on the oracle's table
    rng = np.random.default_rng(7)
    x = rng.integers(-32768, 32768, (1024, 5632)).astype(np.int16)
    y = mq.mq_lut_apply(_dev(x), _dev(ref)).cpu().numpy()
    assert np.array_equal(y, ref[x.astype(np.int64) + 32768])


@pytest.mark.parametrize("M,K,gamma", [(1024, 2048, True), (3, 777, False), (64, 5632, True)])
@pytest.mark.parametrize("out_bits", [8, 16])
def test_rmsnorm_parity(M, K, gamma, out_bits):
    mq = _mq()
    rng = np.random.default_rng(M + K)
    x = rng.integers(-20000, 20000, (M, K)).astype(np.int16)
    x[0] = 17                                     # all at the zero-point: eps alone
    g = rng.uniform(0.5, 1.5, K).astype(np.float32) if gamma else None
    ax, zx, eps, ay, zy = 4e-4, 17, 1e-5, (0.02 if out_bits == 8 else 1e-4), -3
    y = mq.mq_rmsnorm(_dev(x), ax, zx, None if g is None else _dev(g), eps, ay, zy, out_bits)
    ref = oracle.rmsnorm(x, ax, zx, g, eps, ay, zy, out_bits)
    assert np.array_equal(y.cpu().numpy(), ref)


@pytest.mark.parametrize("M,K", [(2048, 1024), (7, 4099), (33, 1)])
def test_softmax_parity(M, K):
    import torch
    mq = _mq()
    rng = np.random.default_rng(M + K)
    x = rng.integers(-9000, 9000, (M, K)).astype(np.int16)
    x[0] = 55                                     # uniform row
    ax, zx, ay, zy = 1e-3, 12, 1.0 / 65535, -32768
    y = mq.mq_softmax(_dev(x), ax, zx, ay, zy, 16).cpu().numpy()
    ref = oracle.softmax(x, ax, zx, ay, zy, 16)
    xr = torch.tensor(np.float64(np.float32(ax)) * (x.astype(np.float64) - zx))
    pre = torch.softmax(xr, dim=1).numpy() / np.float64(np.float32(ay))
    _equal_but_ties(y, ref, pre)


@pytest.mark.parametrize("M,K,period,offset", [(4 * 256, 256, 256, 0), (3 * 100, 100, 100, 0),
                                               (2 * 64, 1024, 64, 960), (5, 4099, 5, 2)])
def test_softmax_causal_parity(M, K, period, offset):
    import torch
    mq = _mq()
    rng = np.random.default_rng(M + K + offset)
    x = rng.integers(-9000, 9000, (M, K)).astype(np.int16)
    ax, zx, ay, zy = 1e-3, 12, 1.0 / 65535, -32768
    y = mq.mq_softmax_causal(_dev(x), ax, zx, ay, zy, period, offset, 16).cpu().numpy()
    ref = oracle.softmax(x, ax, zx, ay, zy, 16, causal_period=period, causal_offset=offset)
    n = np.minimum(np.arange(M) % period + offset + 1, K)
    mask = np.arange(K)[None, :] < n[:, None]
    xr = np.float64(np.float32(ax)) * (x.astype(np.float64) - zx)
    xr = np.where(mask, xr, -np.inf)
    pre = torch.softmax(torch.tensor(xr), dim=1).numpy() / np.float64(np.float32(ay))
    _equal_but_ties(y, ref, pre)
    assert np.all(y[~mask] == zy)


# Rows of at most 2048 codes with K % 8 == 0 take the one-wave-per-row
# kernel whose exponentials come from two 256-entry factor tables; these
# cases cover one, two and four chunks per lane, a last lane past K, grids
# whose second row of a wave lies past M, the full code range (the largest
# difference, 65535, reads the last entry of both tables), scales whose
# tables underflow to zero and subnormals, and causal boundaries inside a
# chunk.
@pytest.mark.parametrize("M,K,out_bits,ax,causal", [
    (1, 8, 8, 1e-3, None),
    (17, 512, 8, 2e-3, (17, 0)),
    (40, 2048, 8, 5e-4, None),
    (1024, 1024, 8, 3e-4, (1024, 0)),
    (64, 1016, 16, 0.05, None),
    (33, 2048, 8, 1e-3, (33, 2000)),
    (300, 200, 16, 0.0113, (300, 0)),
    # rows of any length: no whole chunks, a last chunk of one to seven
    # codes, shorter than one chunk
    (1500, 777, 16, 3e-4, (777, 0)),
    (1030, 1025, 8, 3e-4, None),
    (40, 7, 16, 1e-3, (20, 0)),
    (1100, 513, 8, 2e-3, (550, 3)),
    (5, 2047, 16, 1e-3, None),
    # few long rows (a block each): one, two and four chunks per thread
    (32, 1531, 16, 1e-4, None),
    (32, 4095, 16, 1e-4, (32, 4000)),
    (3, 8191, 8, 2e-4, None),
])
def test_softmax_table_rows(M, K, out_bits, ax, causal):
    import torch
    mq = _mq()
    rng = np.random.default_rng(M * K + out_bits)
    x = rng.integers(-32768, 32768, (M, K)).astype(np.int16)
    x[:, 0] = -32768
    x[:, -1] = 32767
    x[M // 2] = rng.integers(100, 104, K)          # a narrow row
    zx = -5
    ay, zy = (1.0 / 255, -128) if out_bits == 8 else (1.0 / 65535, -32768)
    if causal is None:
        y = mq.mq_softmax(_dev(x), ax, zx, ay, zy, out_bits).cpu().numpy()
        ref = oracle.softmax(x, ax, zx, ay, zy, out_bits)
        n = np.full(M, K)
    else:
        period, offset = causal
        y = mq.mq_softmax_causal(_dev(x), ax, zx, ay, zy, period, offset, out_bits)
        y = y.cpu().numpy()
        ref = oracle.softmax(x, ax, zx, ay, zy, out_bits, causal_period=period,
                             causal_offset=offset)
        n = np.minimum(np.arange(M) % period + offset + 1, K)
    mask = np.arange(K)[None, :] < n[:, None]
    xr = np.float64(np.float32(ax)) * (x.astype(np.float64) - zx)
    xr = np.where(mask, xr, -np.inf)
    pre = torch.softmax(torch.tensor(xr), dim=1).numpy() / np.float64(np.float32(ay))
    _equal_but_ties(y, ref, pre)
    assert np.all(y[~mask] == zy)


@pytest.mark.parametrize("n", [1, 777, 1024 * 5632])
@pytest.mark.parametrize("out_bits", [8, 16])
def test_mul_requant_parity(n, out_bits):
    mq = _mq()
    rng = np.random.default_rng(n + out_bits + 5)
    x1 = rng.integers(-32768, 32768, n).astype(np.int16)
    x2 = rng.integers(-32768, 32768, n).astype(np.int16)
    args = (3.1e-4, -12, 7.7e-4, 300, 0.05 if out_bits == 8 else 1e-3, 5)
    y = mq.mq_mul_requant(_dev(x1), args[0], args[1], _dev(x2), args[2], args[3], args[4],
                          args[5], out_bits)
    ref = oracle.mul_requant(x1, args[0], args[1], x2, args[2], args[3], args[4], args[5], out_bits)
    assert np.array_equal(y.cpu().numpy(), ref)


@pytest.mark.parametrize("M,K,gamma,out_bits", [(1024, 2048, True, 8), (3, 777, False, 16),
                                               (64, 5632, True, 8), (5, 8, False, 8)])
def test_add_rmsnorm_equals_add_then_rmsnorm(M, K, gamma, out_bits):
    """The fused residual add and RMSNorm give the oracle's bits for both
    outputs (K = 777: the two-step fallback)."""
    mq = _mq()
    rng = np.random.default_rng(M * K)
    x1 = rng.integers(-32768, 32768, (M, K)).astype(np.int16)
    x2 = rng.integers(-32768, 32768, (M, K)).astype(np.int16)
    x2[0] = x1[0]                                  # a row of one repeated sum
    a1, z1, a2, z2, ah, zh = 3.1e-4, -12, 7.7e-4, 300, 1.3e-3, 5
    g = rng.uniform(0.5, 1.5, K).astype(np.float32) if gamma else None
    eps, ay, zy = 1e-5, (0.02 if out_bits == 8 else 1e-4), -3
    h_ref = oracle.add_requant(x1, a1, z1, x2, a2, z2, ah, zh, 16)
    y_ref = oracle.rmsnorm(h_ref, ah, zh, g, eps, ay, zy, out_bits)
    h, y = mq.mq_add_rmsnorm(_dev(x1), a1, z1, _dev(x2), a2, z2, ah, zh,
                             None if g is None else _dev(g), eps, ay, zy, out_bits)
    assert np.array_equal(h.cpu().numpy(), h_ref)
    assert np.array_equal(y.cpu().numpy(), y_ref)


@pytest.mark.parametrize("n,lut_bits,out_bits", [(1024 * 5632, 16, 8), (777, 8, 16), (1, 16, 16),
                                                (4099, 8, 8)])
def test_lut_mul_equals_lookup_then_product(n, lut_bits, out_bits):
    """The fused lookup and product give the bits of the oracle's table
    lookup followed by its product (and of the two GPU steps)."""
    mq = _mq()
    rng = np.random.default_rng(n + lut_bits)
    ax, zx = 1e-3, -100
    a1, z1 = (0.05, -7) if lut_bits == 8 else (4e-4, 11)
    lut = oracle.lut_build(oracle.LUT_SILU, ax, zx, a1, z1, lut_bits)
    x1 = rng.integers(-32768, 32768, n).astype(np.int16)
    x2 = rng.integers(-32768, 32768, n).astype(np.int16)
    a2, z2 = 7.7e-4, 300
    ay, zy = (0.05, 5) if out_bits == 8 else (1e-3, -5)
    ref = oracle.mul_requant(lut[x1.astype(np.int64) + 32768].astype(np.int16), a1, z1, x2, a2,
                             z2, ay, zy, out_bits)
    glut = _dev(lut)
    y = mq.mq_lut_mul(_dev(x1), glut, a1, z1, _dev(x2), a2, z2, ay, zy, out_bits)
    assert np.array_equal(y.cpu().numpy(), ref)
    import torch
    two = mq.mq_mul_requant(mq.mq_lut_apply(_dev(x1), glut).to(torch.int16), a1, z1, _dev(x2),
                            a2, z2, ay, zy, out_bits)
    assert np.array_equal(two.cpu().numpy(), ref)


@pytest.mark.parametrize("T,H,D,pos0,out_bits", [(1024, 32, 64, 0, 16), (300, 4, 64, 9, 8),
                                                 (70000, 1, 2, 3, 16), (5, 3, 6, 0, 8)])
def test_rope_table_then_apply(T, H, D, pos0, out_bits):
    """mq_rope_table + mq_rope_apply give mq_rope's bits; one table serves
    several tensors (queries and keys of any head count); past 65535 tokens
    the apply kernel's grid wraps over the token rows."""
    mq = _mq()
    rng = np.random.default_rng(T + D)
    x = rng.integers(-30000, 30000, (T, H * D)).astype(np.int16)
    xk = rng.integers(-30000, 30000, (T, 2 * D)).astype(np.int16)
    ax, zx = 2e-4, -7
    ay, zy = (3e-4, 4) if out_bits == 16 else (0.05, -2)
    table = mq.mq_rope_table(T, D, pos0=pos0)
    for xx, hh in ((x, H), (xk, 2)):
        y = mq.mq_rope_apply(_dev(xx), hh, ax, zx, ay, zy, table, out_bits).cpu().numpy()
        y1 = mq.mq_rope(_dev(xx), hh, ax, zx, ay, zy, out_bits, pos0=pos0).cpu().numpy()
        assert np.array_equal(y, y1)
        if T <= 1024:
            ref = oracle.rope(xx, hh, ax, zx, ay, zy, out_bits, pos0=pos0)
            _equal_but_ties(y, ref, _rope_pre(xx, hh, ax, zx, ay, pos0))
    if T > 65535:  # the last rows, against the oracle on those rows alone
        tail = np.ascontiguousarray(x[-5:])
        ref = oracle.rope(tail, H, ax, zx, ay, zy, out_bits, pos0=pos0 + T - 5)
        got = mq.mq_rope_apply(_dev(x), H, ax, zx, ay, zy, table, out_bits).cpu().numpy()[-5:]
        _equal_but_ties(got, ref, _rope_pre(tail, H, ax, zx, ay, pos0 + T - 5), max_frac=1.0)


@pytest.mark.parametrize("T,H,D,pos0,out_bits", [(1024, 32, 64, 0, 16), (1024, 4, 64, 0, 8),
                                                 (7, 3, 128, 1000, 16), (1, 2, 2, 5, 8)])
def test_rope_parity(T, H, D, pos0, out_bits):
    mq = _mq()
    rng = np.random.default_rng(T + H + D + pos0)
    x = rng.integers(-30000, 30000, (T, H * D)).astype(np.int16)
    ax, zx = 2e-4, -7
    ay, zy = (3e-4, 4) if out_bits == 16 else (0.05, -2)
    y = mq.mq_rope(_dev(x), H, ax, zx, ay, zy, out_bits, pos0=pos0).cpu().numpy()
    ref = oracle.rope(x, H, ax, zx, ay, zy, out_bits, pos0=pos0)
    _equal_but_ties(y, ref, _rope_pre(x, H, ax, zx, ay, pos0))


# The requant of the glue rounds a product with a reciprocal where that is far
# from every half-integer and evaluates the division otherwise; dyadic scales
# put half of all sums and products exactly on a tie, tiny and huge scales
# saturate both ways, and a zero row divides 0 by 0.
@pytest.mark.parametrize("a1,a2,ay,zy", [(1.0, 1.0, 2.0, -32768), (0.5, 0.25, 0.5, 3),
                                         (1.0, 3.0, 1e-30, 7), (1e-20, 1e-20, 1e20, -5),
                                         (3e38, 3e38, 1e-45, 0), (0.1, 0.3, 0.7, 32767)])
@pytest.mark.parametrize("out_bits", [16, 8])
def test_glue_requant_ties_and_ends(a1, a2, ay, zy, out_bits):
    mq = _mq()
    rng = np.random.default_rng(11)
    zy = int(np.clip(zy, -(1 << (out_bits - 1)), (1 << (out_bits - 1)) - 1))
    x1 = rng.integers(-32768, 32768, 8 * 1029 + 3).astype(np.int16)
    x2 = rng.integers(-32768, 32768, x1.size).astype(np.int16)
    x1[:64], x2[:64] = 5, 9                       # both at their zero-points
    x1[64:200] = rng.integers(-60, 60, 136)       # sums inside the int8 grid
    x2[64:200] = rng.integers(-60, 60, 136)
    for gpu, ref in ((mq.mq_add_requant, oracle.add_requant),
                     (mq.mq_mul_requant, oracle.mul_requant)):
        y = gpu(_dev(x1), a1, 5, _dev(x2), a2, 9, ay, zy, out_bits).cpu().numpy()
        assert np.array_equal(y, ref(x1, a1, 5, x2, a2, 9, ay, zy, out_bits))


@pytest.mark.parametrize("eps,ay", [(0.0, 0.5), (1e-5, 1e-45), (0.0, 3e38)])
@pytest.mark.parametrize("K", [2048, 4104, 8192])
def test_rmsnorm_ties_and_ends(K, eps, ay):
    """Rows of one magnitude (every output +-1, a tie of ay = 2), zero rows
    without eps (0 / 0: the low end), saturating scales, gains of 0 and of
    both signs."""
    mq = _mq()
    rng = np.random.default_rng(K)
    x = rng.integers(-32768, 32768, (6, K)).astype(np.int16)
    x[0] = np.where(rng.random(K) < 0.5, 107, -93)
    x[1] = 7
    g = rng.uniform(-2.0, 2.0, K).astype(np.float32)
    g[::5] = 0.0
    g[1::5] = 0.25
    for gamma in (None, g):
        y = mq.mq_rmsnorm(_dev(x), 0.013, 7, None if gamma is None else _dev(gamma), eps, ay, 0,
                          16).cpu().numpy()
        assert np.array_equal(y, oracle.rmsnorm(x, 0.013, 7, gamma, eps, ay, 0, 16))


@pytest.mark.parametrize("n", [1, 65536, 65536 + 13, 300000])
def test_lut_mul_table_in_memory_and_in_lds(n):
    mq = _mq()
    rng = np.random.default_rng(n)
    x1 = rng.integers(-32768, 32768, n).astype(np.int16)
    x2 = rng.integers(-32768, 32768, n).astype(np.int16)
    lut = rng.integers(-32768, 32768, 65536).astype(np.int16)
    ref = oracle.mul_requant(lut[x1.astype(np.int64) + 32768], 9e-5, -3, x2, 1.6e-4, 7, 0.067, 3, 8)
    y = mq.mq_lut_mul(_dev(x1), _dev(lut), 9e-5, -3, _dev(x2), 1.6e-4, 7, 0.067, 3, 8)
    assert np.array_equal(y.cpu().numpy(), ref)


# both forms of the rotation and the sizes between them: whole groups of eight
# pairs or not, 512 pairs per token, 2^18 in all
@pytest.mark.parametrize("T,H,D", [(513, 16, 64), (512, 16, 64), (600, 15, 64), (700, 40, 32),
                                   (600, 18, 60), (300, 9, 256)])
@pytest.mark.parametrize("out_bits", [16, 8])
def test_rope_forms(T, H, D, out_bits):
    mq = _mq()
    rng = np.random.default_rng(T + H + D)
    x = rng.integers(-30000, 30000, (T, H * D)).astype(np.int16)
    ax, zx = 2e-4, -7
    ay, zy = (3e-4, 4) if out_bits == 16 else (0.05, -2)
    y = mq.mq_rope(_dev(x), H, ax, zx, ay, zy, out_bits, pos0=3).cpu().numpy()
    ref = oracle.rope(x, H, ax, zx, ay, zy, out_bits, pos0=3)
    _equal_but_ties(y, ref, _rope_pre(x, H, ax, zx, ay, 3))


# pairs per token at the top of the 32-bit index: the last count of eight-pair
# threads whose last block ends inside it, and the last count accepted
@pytest.mark.parametrize("pairs", [2 ** 31 - 2056, 2 ** 31 - 264])
def test_rope_pair_index_range(pairs):
    import torch
    mq = _mq()
    D = 16
    H = pairs // (D // 2)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.empty((1, H * D), dtype=torch.int16, device="cuda")
    n = 1 << 20
    x.view(-1)[:H * D // n * n].view(-1, n)[:] = torch.randint(-30000, 30000, (n,), generator=g,
                                                               device="cuda").to(torch.int16)
    x[0, -4096 * D:] = torch.randint(-30000, 30000, (4096 * D,), generator=g,
                                     device="cuda").to(torch.int16)
    table = mq.mq_rope_table(1, D, pos0=77)
    y = torch.zeros((1, H * D), dtype=torch.int8, device="cuda")
    mq.mq_rope_apply(x, H, 2e-4, -7, 0.05, -2, table, 8, out=y)
    for lo in (0, H // 2, H - 4096):
        part = slice(lo * D, (lo + 4096) * D)
        ref = mq.mq_rope_apply(x[:, part].contiguous(), 4096, 2e-4, -7, 0.05, -2, table, 8)
        assert torch.equal(y[:, part], ref)
        assert len(torch.unique(ref)) > 100


# Two keys of scores 0 and -d (all others vanish) and an output scale that
# puts one of the quotients within an ulp or two of a half-integer: the
# definition, e / sum / ay one IEEE operation at a time, gives the code named
# (key 0 or key 1), two table exponentials and products with reciprocals its
# neighbour.  Found by a search over 3.9e9 pairs of d and ay.
NEAR_TIES = [("0x1.4a10cap-7", 769, "0x1.21e726p-27", 1, 51236),
             ("0x1.9a4926p-7", 327, "0x1.7bf898p-22", 1, 46326),
             ("0x1.36f662p-6", 609, "0x1.ff8a66p-33", 1, 41069),
             ("0x1.36f662p-6", 609, "0x1.89469ep-33", 1, 53419),
             ("0x1.ed0970p-9", 1650, "0x1.c1baf6p-14", 0, 9307)]


@pytest.mark.parametrize("ax,d,ay,key,code", NEAR_TIES)
@pytest.mark.parametrize("M,K,offset", [(1100, 777, 0), (3, 777, 0), (2, 4096, 0), (20, 2, 0),
                                        (1030, 1024, 1), (1030, 2047, 0)])
def test_softmax_near_ties(ax, d, ay, key, code, M, K, offset):
    """Rows of any length and alignment round as the definition does, in the
    kernels with a wave and with a block per row."""
    import torch
    mq = _mq()
    ax, ay = float.fromhex(ax), float.fromhex(ay)
    e = torch.exp(torch.tensor([0.0, -(ax * d)], dtype=torch.float64, device="cuda"))
    # (a tensor: torch multiplies by the reciprocal of a scalar divisor)
    t = torch.round(e / e.sum() / torch.full_like(e, ay)).tolist()
    assert t[key] == code
    want = [int(min(v, 65535.0)) - 32768 for v in t]
    x = torch.empty(M * K + offset, dtype=torch.int16, device="cuda")[offset:].view(M, K)
    x[:] = 30000 - 60000
    x[:, 0] = 30000
    x[:, K // 2] = 30000 - d
    y = mq.mq_softmax(x, ax, 0, ay, -32768, 16)
    assert y[:, [0, K // 2]].unique(dim=0).tolist() == [want]
