"""The resident sparse kernel that packs four replicas in a word, bit for bit against the
oracle (all sums are small integers, so no tolerance applies): rows longer than the cached
entries, stored diagonals, row sums on either side of the byte bound, every replica group
and number of variables per thread, partial groups, and the fields of a last step."""
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


def _instance(n, deg, top, seed):
    """QUBO with stored diagonals: row i has about deg entries up to +-3 and every seventh
    row of a long-row instance many; row 0 of the canonical Ising form sums to `top`."""
    rng = np.random.default_rng(seed)
    d = {}
    for i in range(n):
        k = 11 if (i % 7 == 3 and deg > 3) else int(rng.integers(0, deg + 1))
        for j in rng.integers(0, n, min(k, n - 1)):
            j = int(j)
            if i != j and 0 not in (i, j):
                d[min(i, j), max(i, j)] = int(rng.integers(1, 4)) * (1 if rng.random() < .5 else -1)
    row = {}
    for (i, j), w in d.items():
        row.setdefault(i, {})[j] = w
        row.setdefault(j, {})[i] = w
    for i in range(0, n, 3):                       # diagonals, folded into the field
        row.setdefault(i, {})[i] = int(rng.integers(-5, 6))
    cols = [sorted(row.get(i, {})) for i in range(n)]
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    col = np.array([j for c in cols for j in c], np.int16)
    w = np.array([row[i][j] for i in range(n) for j in cols[i]], np.int16)
    lin = rng.integers(-4, 5, n).astype(np.int16)
    # b_0 = c_0 + Q_00 + sum_j Q_0j; row 0 has no neighbours, so |b_0| = top
    lin[0] = top - row[0][0]
    return gen.Instance("qubo", n, csr=gen.CSR(n, rp, col, w), lin=lin, meta={})


# variables per thread: 1, 1, 2, 4, 8; the last two rows' LDS holds degree 2-3 only
@pytest.mark.parametrize("n,deg", [(5, 3), (700, 6), (1100, 9), (2100, 3), (4200, 1)])
@pytest.mark.parametrize("top", [255, 256])
def test_all_groups(eng, n, deg, top):
    from paper_2501_19221_amd import qpa
    import torch
    inst = _instance(n, deg, top, n)
    prob = qpa.Problem.from_instance(inst)
    c = inst.csr
    canon = orc.qubo_to_ising_csr_int(c.rp, c.col, c.w, inst.lin)
    assert max(abs(int(b)) for b in canon[3]) == top
    vpt = 1 if n <= 1024 else 2 if n <= 2048 else 4 if n <= 4096 else 8
    T, eta, alpha = 67, 0.01, 0.85
    lam = orc.lambda_linear(T, 60.0)
    for G in (1, 2, 4, 8):
        if G * vpt > 16:
            continue
        R = 2 * G + (G + 1) // 2
        p = qpa.make_params(R, T, eta, alpha, 60.0, 0.1, 1)
        eng.tune_set(prob, p, G)
        print("n=%d top=%d G=%d" % (n, top, G), flush=True)
        x, m = orc.pa_init(n, R, 1, np.float32(0.1))
        xd, md = torch.from_numpy(x).cuda(), torch.from_numpy(m).cuda()
        for t0, t1 in ((0, 1), (1, 66), (66, T)):     # the middle one crosses a 64-step block
            h = eng.steps(prob, p, t0, t1, xd, md, want_h=True)
            ho = orc.pa_steps_csr_int(*canon[:4], x, m, t0, t1, lam, eta, alpha, want_h=True)
            assert np.array_equal(h.cpu().numpy(), ho)
            assert np.array_equal(xd.cpu().numpy(), x) and np.array_equal(md.cpu().numpy(), m)
        out = eng.solve(prob, p, want_state=True)
        assert np.array_equal(out["x"].cpu().numpy(), x)
