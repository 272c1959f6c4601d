"""Symmetry check of instances with more long rows than one pass of the row kernel holds (4096
blocks of four rows): faults in the last rows, on either side of the diagonal, are found."""
import numpy as np
import pytest

from paper_2501_19221_amd import instances as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16384, 16385, 40003])
@pytest.mark.parametrize("fault", ["none", "upper weight", "lower weight", "upper missing",
                                   "lower missing"])
def test_faults_in_the_last_rows(n, fault):
    import torch
    from paper_2501_19221_amd import qpa
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    hops = np.arange(1, 10)                          # 18 entries a row
    i = np.arange(n)[:, None]
    cols = np.concatenate([(i + hops) % n, (i - hops) % n], 1)
    w = np.concatenate([np.broadcast_to(hops, (n, 9)), np.broadcast_to(hops, (n, 9))], 1)
    order = np.argsort(cols, 1)
    cols, w = np.take_along_axis(cols, order, 1), np.take_along_axis(w, order, 1).astype(np.int16)
    row = n - 2
    if fault != "none":
        side = cols[row] > row if fault.startswith("upper") else cols[row] < row
        k = int(np.flatnonzero(side)[0])
    if fault.endswith("weight"):
        w[row, k] += 1
    keep = np.ones(w.shape, bool)
    if fault.endswith("missing"):
        keep[row, k] = False
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    inst = gen.Instance("ising", n, csr=gen.CSR(n, rp, cols[keep].astype(np.int32), w[keep]),
                        lin=np.zeros(n, np.int16), meta={})
    assert inst.csr.nnz >= 16 * n
    eng = qpa.Engine(0)
    p = qpa.make_params(2, 0, 0.001, 0.8, 2.0)
    print("symmetry n=%d %s" % (n, fault), flush=True)
    if fault == "none":
        eng.solve(qpa.Problem.from_instance(inst), p)
    else:
        with pytest.raises(qpa.QpaError) as ei:
            eng.solve(qpa.Problem.from_instance(inst), p)
        assert ei.value.status == qpa.QPA_E_ASYM, ei.value
    eng.close()
