"""The resident sparse kernel for float couplings (spins as floats in LDS), bit for bit against
the oracle (the same chain of rounded sums, so no tolerance applies): every replica group
and number of variables per thread, rows of none to more than the cached entries, partial
groups, fields of a last step, and an instance whose float spins do not fit in LDS."""
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


def _instance(n, deg, seed):
    rng = np.random.default_rng(seed)
    rows = [dict() for _ in range(n)]
    for i in range(n):
        k = 11 if (i % 9 == 4 and deg > 3) else int(rng.integers(0, deg + 1))
        for j in rng.integers(0, n, min(k, n - 1)):
            if i != int(j):
                rows[i][int(j)] = rows[int(j)][i] = np.float32(rng.uniform(-1, 1))
    cols = [sorted(r) for r in rows]
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    col = np.array([j for c in cols for j in c], np.int16)
    w = np.array([rows[i][j] for i in range(n) for j in cols[i]], np.float32)
    lin = rng.uniform(-1, 1, n).astype(np.float32)
    return gen.Instance("ising", n, csr=gen.CSR(n, rp, col, w), lin=lin, meta={})


# variables per thread 1, 1, 2, 4, 8; n = 2048 at G = 8 takes the general kernel (the float
# spins of 8 replicas fill 128 KiB)
@pytest.mark.parametrize("n,deg", [(5, 3), (700, 6), (1100, 6), (2048, 5), (2100, 3), (4200, 1)])
def test_all_groups(eng, n, deg):
    from paper_2501_19221_amd import qpa
    import torch
    inst = _instance(n, deg, n)
    prob = qpa.Problem.from_instance(inst)
    c = inst.csr
    vpt = 1 if n <= 1024 else 2 if n <= 2048 else 4 if n <= 4096 else 8
    T, eta, alpha = 67, 0.05, 0.85
    lam = orc.lambda_linear(T, 4.0)
    for G in (1, 2, 4, 8):
        if G * vpt > 16:
            continue
        R = 2 * G + (G + 1) // 2
        p = qpa.make_params(R, T, eta, alpha, 4.0, 0.1, 1)
        eng.tune_set(prob, p, G)
        print("n=%d G=%d" % (n, G), flush=True)
        x, m = orc.pa_init(n, R, 1, np.float32(0.1))
        xd, md = torch.from_numpy(x).cuda(), torch.from_numpy(m).cuda()
        for t0, t1 in ((0, 1), (1, 66), (66, T)):
            h = eng.steps(prob, p, t0, t1, xd, md, want_h=True)
            ho = orc.pa_steps_csr_float(c.rp, c.col, c.w, inst.lin, x, m, t0, t1, lam, eta,
                                        alpha, want_h=True)
            assert np.array_equal(h.cpu().numpy(), ho)
            assert np.array_equal(xd.cpu().numpy(), x) and np.array_equal(md.cpu().numpy(), m)
        out = eng.solve(prob, p, want_state=True)
        assert np.array_equal(out["x"].cpu().numpy(), x)
