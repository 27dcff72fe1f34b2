"""GPU parity of the attention products' direct kernels against the CPU
oracle at the sizes where their tiles, windows and row maps change: rows that
are no multiple of 64, 16 or 4 codes, shorter than one load, views whose rows
start at any byte, tiles with few and many rows (heads of a group sharing a
tile), both causal promises, and a zero-point of -128 (whose negation is no
int8).  Integer sums: bit-exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _views(rng, H, G, M, N, K, pad, a_zp):
    """a [H][M][K] around a_zp, b [G][N][K] and an output view, each with `pad` extra
    elements per row, starting `pad` elements into its buffer."""
    import torch
    a = np.clip(a_zp + np.rint(4000 * rng.standard_normal((H, M, K))), -32768, 32767)
    a = a.astype(np.int16)
    b = rng.integers(-128, 128, (G, N, K)).astype(np.int8)

    def view(x):
        h, r, c = x.shape
        buf = torch.zeros(h * r * (c + pad) + pad, dtype=torch.from_numpy(x).dtype, device="cuda")
        v = buf[pad:].view(h, r, c + pad)[:, :, :c]
        v.copy_(torch.from_numpy(x))
        return v

    return a, b, view(a), view(b), view


# (H, G, M, N, K): M < 32 shares tiles between heads, K <= 128 is the wide
# kernel (one or two 64-deep steps), longer K the deep one
SHAPES = [(8, 2, 1, 33, 64), (8, 2, 1, 64, 131), (6, 2, 3, 70, 5), (4, 1, 16, 31, 1531),
          (32, 4, 1, 1531, 64), (4, 2, 31, 65, 128), (4, 2, 32, 65, 127), (2, 1, 33, 257, 80),
          (3, 3, 77, 64, 77), (2, 2, 100, 40, 1000), (64, 8, 161, 161, 64), (64, 8, 161, 64, 161),
          (2, 1, 40, 64, 16), (2, 1, 17, 300, 129)]


@pytest.mark.parametrize("H,G,M,N,K", SHAPES)
@pytest.mark.parametrize("pad,b_zp,out_bits", [(0, 0, 16), (1, -128, 8), (3, 127, 16)])
def test_direct_parity(H, G, M, N, K, pad, b_zp, out_bits):
    import paper_2408_13933_amd as mq
    import torch
    rng = np.random.default_rng(H * 1000 + M + N + K + pad)
    a_zp = int(rng.integers(-32768, 32768))
    a, b, ga, gb, view = _views(rng, H, G, M, N, K, pad, a_zp)
    # the largest sum lands at 0.9 of the output grid
    c = [(a[h].astype(np.int64) - a_zp) @ (b[h // (H // G)].astype(np.int64) - b_zp).T
         for h in range(H)]
    out = 3e-5 * 0.02 * float(np.max(np.abs(c))) / (0.9 * 2 ** (out_bits - 1))
    prm = (3e-5, a_zp, 0.02, b_zp, out, -7, out_bits)
    ref = oracle.attn_matmul(a, b, *prm)
    y = view(np.zeros((H, M, N), np.int16 if out_bits == 16 else np.int8))
    mq.mq_attn_matmul(ga, gb, *prm, out=y)
    got = y.cpu().numpy()
    assert np.array_equal(got, ref), int((got != ref).sum())
    assert len(np.unique(ref)) > 10
    if pad:  # nothing written between the rows
        whole = y.as_strided((H, M, N + pad), (M * (N + pad), N + pad, 1))
        assert int(whole[:, :-1, N:].abs().max() if M > 1 else 0) == 0


@pytest.mark.parametrize("H,G,T,past", [(8, 2, 100, 0), (4, 2, 77, 50), (8, 1, 20, 333)])
def test_direct_causal(H, G, T, past):
    """Scores up to the boundary, and the context of probabilities that hold
    their zero-point past it, with `past` keys before the first query."""
    import paper_2408_13933_amd as mq
    import torch
    rng = np.random.default_rng(T + past)
    L, D = T + past, 64
    hidden = np.triu(np.ones((T, L), bool), 1 + past)
    a, b, ga, gb, _ = _views(rng, H, G, T, L, D, 1, 55)
    prm = (3e-5, 55, 0.02, -9, 1e-3, 3, 16)
    ref = oracle.attn_matmul(a, b, *prm)
    s = torch.full((H, T, L), 12345, dtype=torch.int16, device="cuda")
    mq.mq_attn_matmul(ga, gb, *prm, out=s, out_causal=past)
    assert np.array_equal(s.cpu().numpy()[:, ~hidden], ref[:, ~hidden])
    p, v, gp, gv, _ = _views(rng, H, G, T, D, L, 1, -30000)
    p[:, hidden] = -32768
    gp.copy_(torch.from_numpy(p))
    prm = (1.0 / 65535, -32768, 0.03, 11, 0.5, 3, 8)
    got = mq.mq_attn_matmul(gp, gv, *prm, in_causal=past).cpu().numpy()
    assert np.array_equal(got, oracle.attn_matmul(p, v, *prm))


@pytest.mark.parametrize("rows,cols,ldx", [(15, 15, 15), (64, 64, 64), (65, 127, 131),
                                           (777, 256, 256), (128, 1, 3), (5, 200, 201)])
def test_transpose_edges(rows, cols, ldx):
    """Whole and partial 64 x 64 tiles, rows shorter than one load, rows that
    start at any byte."""
    import paper_2408_13933_amd as mq
    import torch
    x = np.random.default_rng(rows + cols).integers(-128, 128, (rows, ldx)).astype(np.int8)
    y = mq.mq_transpose_i8(torch.from_numpy(x).cuda()[:, :cols])
    assert np.array_equal(y.cpu().numpy(), x[:, :cols].T)


# a lane's byte offset inside a 16 x 32 tile is 12 rows and 30 codes at most,
# in 32 bits: the longest output row below 2^32 bytes for 16-bit codes, and
# rows beyond it
@pytest.mark.parametrize("ldy", [178956960, 178956976, 1 << 28])
def test_direct_long_output_rows(ldy):
    import paper_2408_13933_amd as mq
    import torch
    rng = np.random.default_rng(5)
    H, M, N, K = 1, 16, 32, 64
    a = rng.integers(-32768, 32768, (H, M, K)).astype(np.int16)
    b = rng.integers(-128, 128, (1, N, K)).astype(np.int8)
    prm = (3e-5, 7, 0.02, -3, 1e-2, 5, 16)
    ref = oracle.attn_matmul(a, b, *prm)
    buf = torch.empty((M - 1) * ldy + N, dtype=torch.int16, device="cuda")
    y = buf.as_strided((H, M, N), (M * ldy, ldy, 1))
    y.zero_()
    mq.mq_attn_matmul(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), *prm, out=y)
    assert np.array_equal(y.cpu().numpy(), ref)
