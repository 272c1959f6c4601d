"""The relaxed adjoint's row launches where rows differ most: more than one window of 64 entries
in a range of 256 columns, windows that end on a range's bound, empty and single-entry rows
beside full ones, every coupling type.  The bounds are those of the ER QUBO tests."""
import numpy as np
import pytest

import oracle as orc
from paper_2501_19221_amd import instances as gen
from test_gpu_adjoint import T, ETA, ALPHA, _compare, _gpu, _lam, _params, _sum, WL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    from paper_2501_19221_amd import qpa
    return qpa


@pytest.fixture(scope="module")
def eng(q):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    e = q.Engine(0)
    yield e
    e.close()


def _rows(n, full, dtype, seed):
    """Ising graph: vertices in `full` joined to all others, a sparse rest, a few isolated."""
    rng = np.random.default_rng(seed)
    a = np.triu(rng.random((n, n)) < 0.02, 1)
    iso = rng.choice(n, n // 20, replace=False)
    for f in full:
        a[f, f + 1:] = True
        a[:f, f] = True
    a[iso, :] = False
    a[:, iso] = False
    w = rng.integers(-9, 10, (n, n))
    w = np.triu(np.where(a & (w == 0), 1, w) * a, 1)
    w = w + w.T
    wt = w.astype(dtype) if np.issubdtype(dtype, np.integer) else (w / 8.0).astype(dtype)
    rows, cols = np.nonzero(w)
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    lin = rng.integers(-5, 6, n).astype(dtype)
    return gen.Instance("ising", n, csr=gen.CSR(n, rp, cols.astype(np.int32), wt[rows, cols]),
                        lin=lin, meta={})


def _refs(inst, R, seed, norm):
    x0, _ = orc.pa_init(inst.n, R, seed, np.float32(WL.sigma0))
    lam, c = _lam(), inst.csr
    r32 = orc.relaxed_grad32_csr(c.rp, c.col, c.w, inst.lin, x0, T, lam, ETA, ALPHA, norm=norm)
    r64 = orc.relaxed_grad_csr(c.rp, c.col, c.w.astype(np.float64),
                               inst.lin.astype(np.float64), x0, T, lam.astype(np.float64), ETA,
                               ALPHA, norm=norm)
    return r32[:4], r64


@pytest.mark.parametrize("dtype", [np.int8, np.int32, np.float32])
@pytest.mark.parametrize("n,R", [(70, 3), (600, 66)])
def test_uneven_rows(q, eng, n, R, dtype):
    full = [0, 1, 2, 3, 5, 64, n - 1]
    inst = _rows(n, full, dtype, n)
    norm = 1.0 / R
    print("uneven rows n=%d R=%d %s" % (n, R, np.dtype(dtype).name), flush=True)
    got = _gpu(q, eng, [q.Problem.from_instance(inst)], _params(q, R, 5))
    _compare("uneven rows", got, _refs(inst, R, 5, norm), nontrivial=False)
