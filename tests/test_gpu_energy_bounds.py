"""Integer dense energies at the largest row sums that are accepted: every row's sum of
|J| plus |b| is 2^24 - 1, in states whose 32 row fields all add with one sign, so that the FP32
matrix sums use all 24 bits and the int32 sums of 16 rows reach 80 / 128 of their range.
Against int64 sums on the host, equal."""
import numpy as np
import pytest

from paper_2501_19221_amd import instances as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["ising", "qubo"])
@pytest.mark.parametrize("n", [17, 32, 33, 100, 130])
def test_largest_rows(kind, n):
    import torch
    from paper_2501_19221_amd import qpa
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    top = 2 ** 24 - 1
    rng = np.random.default_rng(n)
    g = 2 * rng.integers(0, 2, n) - 1
    a = (top // (n - 1) - 1) | 1                              # odd
    a -= 2 * (a * (n - 1) > top)
    J = np.int64(a) * np.outer(g, g)
    np.fill_diagonal(J, 0)
    b = (top - a * (n - 1)) * g.astype(np.int64)
    assert (np.abs(J).sum(1) + np.abs(b) == top).all()
    if kind == "ising":
        dense, lin, K = J, b, 0
    else:       # fields of a QUBO: row sum (diagonal included) plus linear term
        dense = J.copy()
        np.fill_diagonal(dense, rng.integers(-1000, 1001, n))
        lin = b - dense.sum(1)
    R = 70
    s = np.empty((R, n), np.int8)
    for r in range(R):
        s[r] = g if r % 4 == 0 else -g if r % 4 == 1 else 2 * rng.integers(0, 2, n) - 1
    s64 = s.astype(np.int64)
    if kind == "ising":
        e = np.einsum("ri,ij,rj->r", s64, np.triu(J, 1), s64) + s64 @ b
    else:
        z = (s64 + 1) // 2
        e = np.einsum("ri,ij,rj->r", z, dense, z) + z @ lin
    inst = gen.Instance(kind, n, dense=dense.astype(np.int32), lin=lin.astype(np.int32), meta={})
    print("energies %s n=%d rows of 2^24 - 1" % (kind, n), flush=True)
    eng = qpa.Engine(0)
    p = qpa.make_params(R, 1, 0.1, 0.8, 1.0)
    out = eng.energy(qpa.Problem.from_instance(inst), p, torch.from_numpy(s).cuda())
    got = [o for o in out if o is not None and o.dtype == torch.int64][0].cpu().numpy()
    assert np.array_equal(got, e)
    eng.close()
