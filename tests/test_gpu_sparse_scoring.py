"""Spins and energies of sparse instances at the edges of the scoring kernels (replica groups
of 4 and 16, turned tiles of 64 x 64 down to one replica), and a state that goes through
the replica-fastest layout unchanged: integers equal, float energies to the rounding of
their FP64 sums (n terms: n 2^-52 of the sum of magnitudes)."""
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


def _graph(n, dtype, seed):
    rng = np.random.default_rng(seed)
    if n > 20000:                       # a circulant graph, i -- i + 1 and i -- i + 7
        i = np.arange(n)
        w1, w7 = rng.integers(-8, 9, n), rng.integers(-8, 9, n)
        cols = np.stack([(i + 1) % n, (i - 1) % n, (i + 7) % n, (i - 7) % n], 1)
        w = np.stack([w1, w1[(i - 1) % n], w7, w7[(i - 7) % n]], 1)
        order = np.argsort(cols, 1)
        cols, w = np.take_along_axis(cols, order, 1), np.take_along_axis(w, order, 1)
        w = w.astype(dtype) if dtype != np.float32 else (w * 0.37).astype(np.float32)
        return gen.Instance("ising", n, csr=gen.CSR(n, (4 * np.arange(n + 1)).astype(np.int32),
                                                    cols.reshape(-1).astype(np.int32),
                                                    w.reshape(-1)),
                            lin=rng.integers(-3, 4, n).astype(dtype), meta={})
    a = {}
    for _ in range(2 * n):
        i, j = sorted(int(v) for v in rng.integers(0, n, 2))
        if i != j:
            a[i, j] = int(rng.integers(1, 9)) * (1 if rng.random() < 0.5 else -1)
    rows = [[] for _ in range(n)]
    for (i, j), w in a.items():
        rows[i].append((j, w))
        rows[j].append((i, w))
    rows = [sorted(r) for r in rows]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    col = np.array([j for r in rows for j, _ in r], np.int32)
    w = np.array([v for r in rows for _, v in r], dtype)
    if dtype == np.float32:
        w = (w * np.float32(0.37)).astype(dtype)
    lin = rng.integers(-3, 4, n).astype(dtype)
    return gen.Instance("ising", n, csr=gen.CSR(n, rp, col, w), lin=lin, meta={})


# then more than 2^20 elements, which take the turned tiles; then more than 2^20 variables with
# 2 to 8 replicas, whose spins are packed in bytes
@pytest.mark.parametrize("n,R", [(n, R) for n in (1, 63, 1025, 4099)
                                 for R in (1, 4, 5, 17, 64, 130)] +
                         [(1_048_579, 1), (350_003, 3), (16_411, 65), (4_099, 257)] +
                         [(1_048_576, 2), (1_048_579, 4), (1_048_577, 5), (1_048_578, 8),
                          (1_048_575, 8), (1_048_576, 9)])
def test_initial_state_scored(eng, n, R):
    from paper_2501_19221_amd import qpa
    import torch
    print("n=%d R=%d" % (n, R), flush=True)
    x, m = orc.pa_init(n, R, 3, np.float32(0.1))
    s = np.where(x >= 0, 1, -1).astype(np.int8)
    for dtype in (np.int8, np.float32):
        inst = _graph(n, dtype, n)
        c, prob = inst.csr, qpa.Problem.from_instance(inst)
        p = qpa.make_params(R, 0, 0.1, 0.8, 1.0, 0.1, 3, flags=qpa.QPA_SOLVE_STREAMED)
        out = eng.solve(prob, p, want_state=True)
        assert np.array_equal(out["spins"].cpu().numpy(), s)
        assert np.array_equal(out["x"].cpu().numpy(), x)
        row = np.repeat(np.arange(n), np.diff(c.rp))
        w64 = c.w.astype(np.float64)
        e = np.array([0.5 * np.sum(w64 * s[r][row] * s[r][c.col]) +
                      np.sum(inst.lin.astype(np.float64) * s[r]) for r in range(R)])
        if dtype == np.int8:
            assert np.array_equal(out["energy_i64"].cpu().numpy(), e.astype(np.int64))
        else:
            mag = 0.5 * np.abs(w64).sum() + np.abs(inst.lin).sum()
            assert np.max(np.abs(out["energy"].cpu().numpy() - e)) <= n * 2.0 ** -52 * mag
        # in and out of the replica-fastest layout: no step in between
        xd, md = torch.from_numpy(x).cuda(), torch.from_numpy(x + 1).cuda()
        pt = qpa.make_params(R, 4, 0.1, 0.8, 1.0, 0.1, 3, flags=qpa.QPA_SOLVE_STREAMED)
        eng.steps(prob, pt, 2, 2, xd, md)
        assert np.array_equal(xd.cpu().numpy(), x) and np.array_equal(md.cpu().numpy(), x + 1)
