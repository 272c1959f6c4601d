"""Resident sparse steps whose packed field sums reach both ends of their lanes: rows whose
couplings alone sum to the largest value a lane holds (255 of four replicas a word, 65535 of
two) and one more, in states where neighbouring replicas' sums are 0 and the whole; bit
for bit the oracle's.

A row's lane holds A = sum of |w| over the entries whose spin is -sign(w).  With couplings
w_ij = g_i g_j a_ij (g_i = +-1, a_ij > 0) and spins +-g, every A is 0 or the whole row sum."""
import numpy as np
import pytest

import oracle as orc
from paper_2501_19221_amd import instances as gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    import torch
    from paper_2501_19221_amd import qpa
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    e = qpa.Engine(0)
    yield e
    e.close()


def _gauged(u, v, a, n, seed, lin):
    """Ising instance of the edges (u, v) with couplings g_u g_v a, fields +-lin; and g."""
    rng = np.random.default_rng(seed)
    g = 2 * rng.integers(0, 2, n) - 1
    w = g[u] * g[v] * a
    key = np.concatenate([u * n + v, v * n + u])
    order = np.argsort(key)
    rows, cols = np.concatenate([u, v])[order], np.concatenate([v, u])[order]
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    b = (lin * (2 * rng.integers(0, 2, n) - 1)).astype(np.int32)
    return gen.Instance("ising", n, csr=gen.CSR(n, rp, cols.astype(np.int32),
                                                np.concatenate([w, w])[order].astype(np.int32)),
                        lin=b, meta={}), g


def _check(eng, inst, g, G, R, eta, lam0):
    import torch
    from paper_2501_19221_amd import qpa
    n, c = inst.n, inst.csr
    rows = np.repeat(np.arange(n), np.diff(c.rp))
    whole = np.bincount(rows, np.abs(c.w), n)
    x = np.empty((R, n), np.float32)
    for r in range(R):                             # +g, -g, then random ones
        sign = (1 if r % 2 == 0 else -1) * g if r < R - 2 else \
            2 * np.random.default_rng(r).integers(0, 2, n) - 1
        x[r] = 0.25 * sign
    A = [np.bincount(rows, np.where(x[r][c.col] * c.w < 0, np.abs(c.w), 0), n) for r in range(2)]
    assert ((A[0] == 0) | (A[0] == whole)).all() and (A[0] + A[1] == whole).all()
    T = 4
    prob = qpa.Problem.from_instance(inst)
    p = qpa.make_params(R, T, eta, 0.85, lam0, 0.1, 1)
    eng.tune_set(prob, p, G)
    lam = orc.lambda_linear(T, lam0)
    m = np.zeros_like(x)
    xd, md = torch.from_numpy(x).cuda(), torch.from_numpy(m).cuda()
    for t in range(T):
        h = eng.steps(prob, p, t, t + 1, xd, md, want_h=True).cpu().numpy()
        ho = orc.pa_steps_csr_int(c.rp, c.col, c.w, inst.lin, x, m, t, t + 1, lam, eta, 0.85,
                                  want_h=True)
        assert np.array_equal(h, ho), t
        assert np.array_equal(xd.cpu().numpy(), x) and np.array_equal(md.cpu().numpy(), m), t


# rings whose couplings alternate: every row sums to the two together; then a field.  n: one and
# two variables a thread (at three and more the spins are floats)
@pytest.mark.parametrize("n", [300, 1400])
@pytest.mark.parametrize("a,b,lin", [(200, 55, 0), (254, 1, 0), (127, 127, 1), (200, 56, 0),
                                     (255, 1, 0)])
def test_byte_sums(eng, n, a, b, lin):
    i = np.arange(n, dtype=np.int64)
    inst, g = _gauged(i, (i + 1) % n, np.where(i % 2 == 0, a, b), n, n + a, lin)
    inst.csr.w, inst.lin = inst.csr.w.astype(np.int16), inst.lin.astype(np.int16)
    assert np.abs(inst.csr.w).reshape(-1, 2).sum(1).max() == a + b
    for G in (1, 2, 4, 8):
        print("byte sums n=%d %d+%d+%d G=%d" % (n, a, b, lin, G), flush=True)
        _check(eng, inst, g, G, 2 * G + (G + 1) // 2 + 2, 0.001, 60.0)


def _chimera(m):
    c = gen.chimera_ising(m, seed=3).csr
    rows = np.repeat(np.arange(c.n), np.diff(c.rp)).astype(np.int64)
    keep = rows < c.col
    return rows[keep], c.col[keep].astype(np.int64), c.n


# Chimera C16 in groups of 8: the float spins (two buffers of n G floats) do not fit in LDS
# beside the entries, the spin bits do, in 16-bit sums below 2^16 and int32 sums from there on.
# Rows of 6 entries sum to 6 a + lin.
@pytest.mark.parametrize("a,lin", [(10922, 3), (10922, 4), (20000, 0)])
def test_word_sums(eng, a, lin):
    u, v, n = _chimera(16)
    G, nnz = 8, 2 * len(u)
    assert 2 * n * G * 4 + 4 * (n + 1) + 6 * nnz + 16 > 160 * 1024
    assert 256 * 16 + 4 * (n + 1) + 6 * nnz + 2 * n + 16 <= 160 * 1024
    inst, g = _gauged(u, v, np.full(len(u), a), n, a + lin, lin)
    inst.csr.w, inst.lin = inst.csr.w.astype(np.int16), inst.lin.astype(np.int16)
    assert np.bincount(np.repeat(np.arange(n), np.diff(inst.csr.rp)),
                       np.abs(inst.csr.w.astype(np.int64))).max() + lin == 6 * a + lin
    print("word sums 6 x %d + %d" % (a, lin), flush=True)
    _check(eng, inst, g, G, 2 * G + 5, 0.00001, 20000.0)


# one variable a thread, groups of 8: spin bits by the rule, two replicas a word
@pytest.mark.parametrize("a,lin", [(32767, 1), (16384, 0)])
def test_word_sums_one_variable_a_thread(eng, a, lin):
    n = 250
    i = np.arange(n, dtype=np.int64)
    inst, g = _gauged(i, (i + 1) % n, np.full(n, a), n, a, lin)
    inst.csr.w, inst.lin = inst.csr.w.astype(np.int16), inst.lin.astype(np.int16)
    print("word sums 2 x %d + %d, n=%d" % (a, lin, n), flush=True)
    _check(eng, inst, g, 8, 2 * 8 + 5, 0.00001, 20000.0)
