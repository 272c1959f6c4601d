"""Relaxed gradient at the numbers of steps where its table of partial sums wraps round (32
steps are kept): a dense and a sparse instance in one batch against the oracle's
single-precision pass, whose trajectories are the same, so that only the order of the FP64 sums
differs (at most 65 steps of 130 x 20 + 90 x 20 terms)."""
import numpy as np
import pytest

import oracle as orc
from paper_2501_19221_amd import instances as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 31, 32, 33, 64, 65])
def test_partial_sums_of_steps(T):
    import torch
    from paper_2501_19221_amd import qpa
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dense = gen.sk_ising(130, 0.1, seed=3)
    er = gen.er_qubo(90, 0.2, 100, np.random.default_rng(4))
    R, seed, eta, alpha = 20, 9, float(np.float32(0.002)), float(np.float32(0.8))
    lam = orc.lambda_linear(T, 4.0)
    norm = 1.0 / (2 * R)
    x0 = orc.pa_init(dense.n, R, seed, np.float32(0.1))[0]
    refs = [orc.relaxed_grad32_dense(dense.dense, dense.lin, x0, T, lam, eta, alpha, norm=norm)]
    c = er.csr
    rp, col, w, b, _ = orc.qubo_to_ising_csr_int(c.rp, c.col, c.w, er.lin)
    x0 = orc.pa_init(er.n, R, seed + 1, np.float32(0.1))[0]
    refs.append(orc.relaxed_grad32_csr(rp, col, w, b, x0, T, lam, eta, alpha, norm=norm))
    eng = qpa.Engine(0)
    print("relaxed gradient T=%d" % T, flush=True)
    p = qpa.make_params(R, T, eta, alpha, 4.0, 0.1, seed, lambda_table=lam)
    got = eng.relaxed_grad([qpa.Problem.from_instance(i) for i in (dense, er)], p, 10)
    for k, g in enumerate(got):
        r = np.asarray(refs[0][k]) + np.asarray(refs[1][k])
        g = g.cpu().numpy().reshape(r.shape)
        assert np.allclose(g, r, rtol=1e-9, atol=1e-10 * np.max(np.abs(r))), (k, g, r)
    eng.close()
