"""Sparse instances whose couplings are not symmetric are refused whichever side of the
diagonal the fault is on, in the thread-per-row, wave-per-row and batched passes; the same
instances without the fault are taken."""
import numpy as np
import pytest

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


def _instance(n, deg, dtype, fault, seed=3):
    rng = np.random.default_rng(seed)
    d = {}
    for i in range(n):
        for j in rng.integers(0, n, deg):
            if i != int(j):
                v = int(rng.integers(1, 50))
                d[i, int(j)] = d[int(j), i] = v
    keys = sorted(k for k in d if k[0] < k[1])
    a, b = keys[len(keys) // 2], keys[len(keys) // 3]
    up, lo = a, (a[1], a[0])
    if fault == "upper only":
        del d[lo]
    elif fault == "lower only":
        del d[up]
    elif fault == "lower weight":
        d[lo] += 1
    elif fault == "upper weight":
        d[up] += 1
    elif fault == "one missing on each side":
        del d[lo]
        del d[b]
    elif fault == "stored zero":
        k = next((i, j) for i in range(n - 1, 0, -1) for j in range(i) if (i, j) not in d)
        d[k] = 0
    rows = [sorted((j, v) for (i, j), v in d.items() if i == r) for r in range(n)] \
        if n <= 60 else None
    if rows is None:
        rows = [[] for _ in range(n)]
        for (i, j), v in sorted(d.items()):
            rows[i].append((j, v))
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    col = np.array([j for r in rows for j, _ in r], np.int32)
    w = np.array([v for r in rows for _, v in r], dtype)
    return gen.Instance("ising", n, csr=gen.CSR(n, rp, col, w), lin=np.zeros(n, dtype), meta={})


@pytest.mark.parametrize("n,deg,dtype", [(40, 2, np.int16), (700, 3, np.float32),
                                         (300, 12, np.int16)])
@pytest.mark.parametrize("fault", ["none", "upper only", "lower only", "lower weight",
                                   "upper weight", "one missing on each side", "stored zero"])
def test_faults_on_either_side(eng, n, deg, dtype, fault):
    from paper_2501_19221_amd import qpa
    prob = qpa.Problem.from_instance(_instance(n, deg, dtype, fault))
    p = qpa.make_params(4, 2, 0.001, 0.8, 2.0)
    runs = [lambda: eng.solve(prob, p)]
    if dtype == np.int16:
        good = qpa.Problem.from_instance(_instance(n, deg, dtype, "none", seed=4))
        runs.append(lambda: eng.solve_batch([good, prob, good], p))
    for run in runs:
        if fault == "none":
            run()
            continue
        with pytest.raises(qpa.QpaError) as ei:
            run()
        assert ei.value.status == qpa.QPA_E_ASYM, ei.value
