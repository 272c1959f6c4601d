"""Batch instances whose int8 tiles lie in the place of their sparse state (tiles cheaper with the
variables padded to 128, not to 256), bit for bit against the oracle, beside one whose
weights the tiles cannot hold, which stays on the sparse kernel in that place, and one with
tile buffers of its own."""
import numpy as np
import pytest

import oracle as orc
from paper_2501_19221_amd import instances as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [1, 31, 32, 64, 65, 100, 300])
def test_tiles_in_the_state_s_place(R):
    import torch
    from paper_2501_19221_amd import qpa
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(R)
    insts = [gen.er_qubo(n, 0.1, 100, rng) for n in (102, 106, 110, 118, 118)]
    wide = gen.er_qubo(112, 0.1, 1000, rng)                     # |w| past 127
    own = gen.er_qubo(300, 0.1, 100, rng)
    insts += [wide, own]
    T, eta, alpha, lam0 = 9, 0.0002, 0.8, 200.0
    p = qpa.make_params(R, T, eta, alpha, lam0, 0.1, 5)
    eng = qpa.Engine(0)
    print("tiles in the state's place R=%d" % R, flush=True)
    outs = eng.solve_batch([qpa.Problem.from_instance(i) for i in insts], p, want_state=True)
    paths = qpa.qpa_batch_paths(eng.ctx, len(insts))
    assert (paths[:5] == qpa.QPA_PATH_BATCH_SPARSE_I8).any() or R == 1, paths
    assert paths[5] == qpa.QPA_PATH_BATCH_SPARSE, paths
    lam = orc.lambda_linear(T, lam0)
    for k, (inst, out) in enumerate(zip(insts, outs)):
        c = inst.csr
        rp, col, w, b, K = orc.qubo_to_ising_csr_int(c.rp, c.col, c.w, inst.lin)
        x, m = orc.pa_init(inst.n, R, 5 + k, np.float32(0.1))
        orc.pa_steps_csr_int(rp, col, w, b, x, m, 0, T, lam, eta, alpha)
        assert np.array_equal(out["x"].cpu().numpy(), x), k
        assert np.array_equal(out["m"].cpu().numpy(), m), k
        s = np.where(x >= 0, 1, -1).astype(np.int64)
        assert np.array_equal(out["spins"].cpu().numpy(), s), k
        dense = np.zeros((inst.n, inst.n), np.int64)
        dense[np.repeat(np.arange(inst.n), np.diff(c.rp)), c.col] = c.w
        z = (s + 1) // 2
        e = np.einsum("ri,ij,rj->r", z, dense, z) + z @ inst.lin.astype(np.int64)
        assert np.array_equal(out["energy_i64"].cpu().numpy(), e), k
    eng.close()
