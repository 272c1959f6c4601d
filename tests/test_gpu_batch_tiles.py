"""The int8 tiles of a batch (64 replicas x 128 variables) at their edges, bit for bit against
the oracle: one reduction chunk and several, ragged last tiles, replica counts around a
tile, entry lists and dense rows side by side."""
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


@pytest.mark.parametrize("R", [1, 8, 33, 64, 65, 100])
def test_int8_tile_edges(eng, R):
    from paper_2501_19221_amd import qpa
    rng = np.random.default_rng(R)
    insts = []
    for n in (7, 127, 128, 129, 255, 256, 257, 385, 640):
        insts += [gen.er_qubo(n, 0.1, 100, rng), gen.er_qubo(n, 0.6, 100, rng)]
    T, eta, alpha, lam0 = 9, 0.0002, 0.8, 200.0
    p = qpa.make_params(R, T, eta, alpha, lam0, 0.1, 5, flags=qpa.QPA_BATCH_DENSE)
    print("int8 tiles R=%d" % R, flush=True)
    outs = eng.solve_batch([qpa.Problem.from_instance(i) for i in insts], p, want_state=True)
    paths = qpa.qpa_batch_paths(eng.ctx, len(insts))
    assert (paths[2::2] == qpa.QPA_PATH_BATCH_SPARSE_I8).all(), paths
    assert (paths[5::2] == qpa.QPA_PATH_BATCH_DENSE_I8).all(), paths
    lam = orc.lambda_linear(T, lam0)
    for k, (inst, out) in enumerate(zip(insts, outs)):
        c = inst.csr
        rp, col, w, b, _ = orc.qubo_to_ising_csr_int(c.rp, c.col, c.w, inst.lin)
        x, m = orc.pa_init(inst.n, R, 5 + k, np.float32(0.1))
        orc.pa_steps_csr_int(rp, col, w, b, x, m, 0, T, lam, eta, alpha)
        assert np.array_equal(out["x"].cpu().numpy(), x), k
        assert np.array_equal(out["m"].cpu().numpy(), m), k
