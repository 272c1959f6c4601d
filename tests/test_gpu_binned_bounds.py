"""The binned step where its packed sums reach both ends of their lanes: rings whose two
couplings and field sum to just below and just above what four sums a word (2^8) and two
(2^16) hold, bit for bit against the oracle.  From a random state a quarter of all sums are
the whole of a row's |w| and a quarter 0, in neighbouring replicas too."""
import numpy as np
import pytest

import oracle as orc
from paper_2501_19221_amd import instances as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,lin", [(126, 2), (127, 1), (127, 2), (128, 0), (32766, 2),
                                   (32767, 1), (32767, 2)])
@pytest.mark.parametrize("n,R", [(70001, 4), (70001, 8), (9001, 3)])
def test_ring_sums(n, R, w, lin):
    import torch
    from paper_2501_19221_amd import qpa
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(w + lin)
    i = np.arange(n)
    s = (2 * rng.integers(0, 2, n) - 1) * w
    cols = np.stack([(i + 1) % n, (i - 1) % n], 1)
    wts = np.stack([s, s[(i - 1) % n]], 1)
    order = np.argsort(cols, 1)
    cols, wts = np.take_along_axis(cols, order, 1), np.take_along_axis(wts, order, 1)
    inst = gen.Instance("ising", n, csr=gen.CSR(n, (2 * np.arange(n + 1)).astype(np.int32),
                                                cols.reshape(-1).astype(np.int32),
                                                wts.reshape(-1).astype(np.int16)),
                        lin=(lin * (2 * rng.integers(0, 2, n) - 1)).astype(np.int16), meta={})
    T, eta, lam0 = 4, 0.05 / w, 6.0 * w
    print("binned sums n=%d R=%d 2 x %d + %d" % (n, R, w, lin), flush=True)
    eng = qpa.Engine(0)
    p = qpa.make_params(R, T, eta, 0.8, lam0, 0.1, 1, flags=qpa.QPA_SOLVE_BINNED)
    out = eng.solve(qpa.Problem.from_instance(inst), p, want_state=True)
    x, m = orc.pa_init(n, R, 1, np.float32(0.1))
    c = inst.csr
    A = [np.where(x[r][cols] * wts < 0, w, 0).sum(1) for r in range(R)]
    assert all((a == 0).mean() > 0.2 and (a == 2 * w).mean() > 0.2 for a in A)
    orc.pa_steps_csr_int(c.rp, c.col, c.w, inst.lin, x, m, 0, T, orc.lambda_linear(T, lam0),
                         float(np.float32(eta)), float(np.float32(0.8)))
    assert np.array_equal(out["x"].cpu().numpy(), x) and np.array_equal(out["m"].cpu().numpy(), m)
    eng.close()
