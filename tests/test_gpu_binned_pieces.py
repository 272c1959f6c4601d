"""The binned step at the edges of its pieces, against the streamed step (itself held to the
oracle) and the oracle, bit for bit: runs of exactly 256 entries and one more, runs of
many pieces, bins whose only run lies more than 63 chunks in, one, two and four sums per
word, odd numbers of (row, replica) pairs at the end."""
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


def _ring(n, hop, w, seed):
    """Ising ring i -- i + hop (mod n), n > 2 hop: two entries a row, random signs."""
    rng = np.random.default_rng(seed)
    s = (2 * rng.integers(0, 2, n) - 1) * w
    i = np.arange(n, dtype=np.int64)
    a, b = (i + hop) % n, (i - hop) % n
    wa, wb = s[i], s[b]
    swap = a > b
    col = np.stack([np.where(swap, b, a), np.where(swap, a, b)], 1).reshape(-1)
    wts = np.stack([np.where(swap, wb, wa), np.where(swap, wa, wb)], 1).reshape(-1)
    rp = (2 * np.arange(n + 1)).astype(np.int32)
    dt = np.int8 if w < 128 else np.int16
    lin = rng.integers(-2, 3, n).astype(dt)
    return gen.Instance("ising", n, csr=gen.CSR(n, rp, col.astype(np.int32), wts.astype(dt)),
                        lin=lin, meta={})


def _run(eng, inst, R, T, flag):
    from paper_2501_19221_amd import qpa
    prob = qpa.Problem.from_instance(inst)
    p = qpa.make_params(R, T, 0.05, 0.8, 6.0, 0.1, 1, flags=flag)
    out = eng.solve(prob, p, want_state=True)
    return {k: out[k].cpu().numpy() for k in ("x", "m", "spins", "energy_i64")}


# n = 128: a run of 256 entries; 129: one more; 70001: several chunks (R = 8, 4) and bins
@pytest.mark.parametrize("w", [1, 300, 32767])
@pytest.mark.parametrize("n,R", [(128, 1), (129, 2), (70001, 1), (70001, 2), (70001, 4),
                                 (140001, 7)])
def test_small_rings_against_oracle(eng, n, R, w):
    from paper_2501_19221_amd import qpa
    inst = _ring(n, 40, w, n)
    print("ring n=%d R=%d w=%d" % (n, R, w), flush=True)
    T = 5
    got = _run(eng, inst, R, T, qpa.QPA_SOLVE_BINNED)
    x, m = orc.pa_init(n, R, 1, np.float32(0.1))
    c = inst.csr
    orc.pa_steps_csr_int(c.rp, c.col, c.w, inst.lin, x, m, 0, T, orc.lambda_linear(T, 6.0), 0.05,
                         0.8)
    assert np.array_equal(got["x"], x) and np.array_equal(got["m"], m)


def test_runs_beyond_63_chunks(eng):
    """R = 8: 69 chunks of 131072 variables; every bin's entries lie in one or two of them."""
    from paper_2501_19221_amd import qpa
    inst = _ring(9_000_001, 3, 5, 2)
    print("ring n=9000001 R=8", flush=True)
    a = _run(eng, inst, 8, 3, qpa.QPA_SOLVE_BINNED)
    b = _run(eng, inst, 8, 3, qpa.QPA_SOLVE_STREAMED)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
