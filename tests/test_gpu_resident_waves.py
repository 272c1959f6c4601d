"""Resident sparse steps where the waves of a workgroup hold rows of different lengths (none,
up to six, seven or eight, and more entries than are kept in registers): all waves take the
same step loop, bit for bit the oracle's."""
import numpy as np
import pytest

import oracle as orc
from paper_2501_19221_amd import instances as gen

pytestmark = pytest.mark.gpu


def _instance(n, long_rows, seed):
    """Rows 0 .. 63 empty, the last 64 rows of `long_rows` entries each, rings between."""
    rng = np.random.default_rng(seed)
    u, v = [np.arange(64, n - 1)], [np.arange(65, n)]
    top = np.arange(n - 64, n)
    for d in range(2, 2 + (long_rows - 2) // 2):
        u.append(top)
        v.append(n - 64 + (top - (n - 64) + d) % 64)
    u, v = np.concatenate(u), np.concatenate(v)
    key = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
    u, v = key // n, key % n
    w = (2 * rng.integers(0, 2, len(u)) - 1).astype(np.int8)
    order = np.argsort(np.concatenate([u * n + v, v * n + u]))
    rows = np.concatenate([u, v])[order]
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    return gen.Instance("ising", n, csr=gen.CSR(n, rp, np.concatenate([v, u])[order].astype(np.int16),
                                                np.concatenate([w, w])[order]),
                        lin=rng.integers(-2, 3, n).astype(np.int8), meta={})


@pytest.mark.parametrize("n", [320, 1500])
@pytest.mark.parametrize("long_rows", [6, 8, 20])
def test_waves_of_different_rows(n, long_rows):
    import torch
    from paper_2501_19221_amd import qpa
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    inst = _instance(n, long_rows, n + long_rows)
    c = inst.csr
    assert int(np.diff(c.rp).max()) >= long_rows and int(np.diff(c.rp).min()) == 0
    eng = qpa.Engine(0)
    prob = qpa.Problem.from_instance(inst)
    T, eta, alpha = 70, 0.01, 0.85
    lam = orc.lambda_linear(T, 60.0)
    for G in (1, 4, 8):
        R = 2 * G + 1
        p = qpa.make_params(R, T, eta, alpha, 60.0, 0.1, 1)
        eng.tune_set(prob, p, G)
        print("n=%d rows of up to %d, G=%d" % (n, long_rows, G), flush=True)
        x, m = orc.pa_init(n, R, 1, np.float32(0.1))
        orc.pa_steps_csr_int(c.rp, c.col, c.w.astype(np.int32), inst.lin.astype(np.int64), x, m, 0,
                             T, lam, eta, alpha)
        out = eng.solve(prob, p, want_state=True)
        assert np.array_equal(out["x"].cpu().numpy(), x)
        assert np.array_equal(out["m"].cpu().numpy(), m)
    eng.close()
