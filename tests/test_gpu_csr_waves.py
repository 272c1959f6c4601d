"""The streamed sparse step for groups of 64 replicas, bit for bit against the oracle (the same
order and rounding of every sum, so no tolerance applies): 4 and 8 variables a wave with
ragged ends, rows of none to many passes of entries, stored diagonals, integer and float."""
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


def _instance(n, dtype, kind, seed):
    rng = np.random.default_rng(seed)
    rows = [dict() for _ in range(n)]
    hubs = {0: 37, n // 2: 16, n - 1: 5}           # more passes than one, an exact fill
    pairs = [(i, int(j)) for i in range(0, n, 2) for j in rng.integers(0, n, 2)]
    pairs += [(h, int(j)) for h, c in hubs.items() if h < n for j in rng.integers(0, n, c)]
    for i, j in pairs:
        if i != j:
            w = int(rng.integers(-9, 10)) or 1
            rows[i][j] = rows[j][i] = w if dtype != np.float32 else np.float32(w / 7.0)
    if kind == "qubo":
        for i in range(0, n, 3):
            rows[i][i] = 6
    cols = [sorted(r) for r in rows]
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    col = np.array([j for c in cols for j in c], np.int32)
    w = np.array([rows[i][j] for i in range(n) for j in cols[i]], dtype)
    lin = rng.integers(-4, 5, n).astype(dtype)
    return gen.Instance(kind, n, csr=gen.CSR(n, rp, col, w), lin=lin, meta={})


@pytest.mark.parametrize("dtype,kind", [(np.int8, "ising"), (np.int16, "qubo"),
                                        (np.int32, "ising"), (np.float32, "ising")])
@pytest.mark.parametrize("n,R", [(1, 40), (3, 64), (997, 65), (33005, 33)])
def test_streamed_groups_of_64(eng, n, R, dtype, kind):
    from paper_2501_19221_amd import qpa
    import torch
    inst = _instance(n, dtype, kind, n)
    prob = qpa.Problem.from_instance(inst)
    c = inst.csr
    canon = orc.qubo_to_ising_csr_int(c.rp, c.col, c.w, inst.lin)[:4] if kind == "qubo" else \
        (c.rp, c.col, c.w, inst.lin)
    T, eta, alpha = 4, 0.004, 0.85
    lam = orc.lambda_linear(T, 30.0)
    p = qpa.make_params(R, T, eta, alpha, 30.0, 0.1, 1, flags=qpa.QPA_SOLVE_STREAMED)
    print("n=%d R=%d %s %s" % (n, R, np.dtype(dtype).name, kind), flush=True)
    x, m = orc.pa_init(n, R, 1, np.float32(0.1))
    xd, md = torch.from_numpy(x).cuda(), torch.from_numpy(m).cuda()
    step = orc.pa_steps_csr_float if dtype == np.float32 else orc.pa_steps_csr_int
    h = eng.steps(prob, p, 0, T, xd, md, want_h=True)
    ho = step(*canon, x, m, 0, T, lam, eta, alpha, want_h=True)
    assert np.array_equal(h.cpu().numpy(), ho)
    assert np.array_equal(xd.cpu().numpy(), x) and np.array_equal(md.cpu().numpy(), m)
