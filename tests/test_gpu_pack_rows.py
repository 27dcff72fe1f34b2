"""The weight packers, the fold and range learning at the sizes where their
kernels change: rows in registers (one, two and four chunks per thread, a last
chunk of few threads) against the element-wise kernels (longer, ragged or
unaligned rows), rounding ties, and values without a quotient.  Bit-exact
against the CPU oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _rows(rng, N, K):
    w = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    w[0] = 0.0
    w[1, : K // 2] = np.inf
    w[2, ::3] = np.nan
    w[3] = rng.integers(-254, 255, K) * np.float32(0.25)   # many exact ties: absmax 63.5
    w[3, 0] = 63.5
    w[4] = (rng.standard_normal(K) * 1e-42).astype(np.float32)  # subnormal scale
    w[5] = (rng.standard_normal(K) * 8e37).astype(np.float32)   # reciprocal of the scale subnormal
    w[5, -1] = 3.3e38
    w[6] = np.abs(w[7])
    return w


def _dev(a, off):
    """a on the GPU, `off` elements into its buffer."""
    import torch
    t = torch.empty(a.size + off, dtype=torch.from_numpy(a).dtype, device="cuda")[off:]
    t = t.view(a.shape)
    t.copy_(torch.from_numpy(a))
    return t


SHAPES = [(8, 0), (2048, 0), (2056, 0), (4096, 0), (4104, 0), (8192, 0), (8200, 0), (2044, 0),
          (2048, 1), (520, 0)]


@pytest.mark.parametrize("K,off", SHAPES)
@pytest.mark.parametrize("bits", [8, 4])
def test_pack_rows(K, off, bits):
    import paper_2408_13933_amd as mq
    w = _rows(np.random.default_rng(K + bits), 9, K)
    got = [t.cpu().numpy() for t in mq.mq_pack_weights(_dev(w, off), bits)]
    for g, r in zip(got, oracle.pack_weights(w, bits)):
        assert np.array_equal(g, r.astype(g.dtype), equal_nan=g.dtype.kind == "f")


@pytest.mark.parametrize("K,off", SHAPES)
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("per_tensor", [False, True])
def test_pack_rows_asym(K, off, bits, per_tensor):
    import paper_2408_13933_amd as mq
    w = _rows(np.random.default_rng(K + bits + 1), 1100 if per_tensor and K == 520 else 9, K)
    got = [t.cpu().numpy() for t in mq.mq_pack_weights_asym(_dev(w, off), bits, per_tensor)]
    for g, r in zip(got, oracle.pack_weights_asym(w, bits, per_tensor=per_tensor)):
        assert np.array_equal(g, r.astype(g.dtype))


@pytest.mark.parametrize("rows,K", [(1, 1), (5, 4), (300, 2048), (3, 2050), (700, 36), (2, 70000)])
def test_fold_columns(rows, K):
    """Columns of a thread's items wrap at every row length, in place too."""
    import paper_2408_13933_amd as mq
    rng = np.random.default_rng(rows + K)
    w = rng.standard_normal((rows, K)).astype(np.float32)
    s = rng.uniform(0.3, 3.0, K).astype(np.float32)
    g = _dev(w, 0)
    assert np.array_equal(mq.mq_fold_weights(g, _dev(s, 0)).cpu().numpy(), w * s)
    assert np.array_equal(mq.mq_fold_acts(g, _dev(s, 0), out=g).cpu().numpy(), w / s)


@pytest.mark.parametrize("n,off", [(1, 0), (4099, 0), (1 << 20, 0), ((1 << 21) + 5, 0), (5000, 1)])
def test_arl_backward_sizes(n, off):
    import paper_2408_13933_amd as mq
    rng = np.random.default_rng(n)
    x = (rng.standard_normal(n) * 5).astype(np.float32)
    g = rng.standard_normal(n).astype(np.float32)
    alpha, beta = 0.0625, -100.25
    gx, grads = mq.mq_arl_backward(_dev(x, off), _dev(g, off), alpha, beta, 8)
    t = x / np.float32(alpha)
    u = np.rint(t) - np.float32(beta)
    inside = (u >= 0) & (u <= 255)
    assert np.array_equal(gx.cpu().numpy(), np.where(inside, g, np.float32(0)))
    c = np.clip(u, 0, 255).astype(np.float64)
    ga = g.astype(np.float64) * (c + np.float64(np.float32(beta)) - np.where(inside, t, 0.0))
    gb = np.where(inside, 0.0, g.astype(np.float64) * alpha)
    # n fp64 additions in some order: at most n 2^-53 of the sum of magnitudes
    for got, terms in zip(grads[:2].cpu().numpy(), (ga, gb)):
        assert abs(got - terms.sum()) <= 2 * (n + 8) * 2.0 ** -53 * np.abs(terms).sum()
