"""Workspace sizes are part of the interface: a caller keeps a buffer of the size it was once
told.  Bounds in bytes for calls that have been asked for; no call may need more."""
import ctypes
import os

import pytest


@pytest.fixture(scope="module")
def q():
    from paper_2501_19221_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    from paper_2501_19221_amd import qpa
    return qpa


def problem(q, n, couplings, nnz=None, index="QPA_I16"):
    """Dense (nnz None) or sparse; the arrays are never read."""
    p = q.qpa_problem()
    p.n = n
    p.kind = q.QPA_KIND_ISING
    p.coupling_dtype = getattr(q, couplings)
    if nnz is None:
        p.format = q.QPA_FMT_DENSE
        p.dense = 0x1000
    else:
        p.format = q.QPA_FMT_CSR
        p.index_dtype = getattr(q, index)
        p.row_ptr = p.col = p.weights = 0x1000
        p.nnz = nnz
    return p


def batch_size(q, probs, a):
    out = ctypes.c_size_t()
    arr = (q.qpa_problem * len(probs))(*probs)
    st = q._lib.qpa_workspace_size_batch(None, len(probs), arr, ctypes.byref(a),
                                         ctypes.byref(out))
    assert st == q.QPA_OK
    return out.value


# n, entries a row, couplings, replicas, flags, BF16, instances: bytes.  Sizes just past a
# multiple of 256 and few entries, where the padded tile buffers are far the larger ones
@pytest.mark.parametrize("n,deg,couplings,R,flags,bf16,count,bound", [
    (513, 20, "QPA_I8", 2, 0, False, 1, 466944),
    (513, 8, "QPA_I8", 300, 0, False, 3, 6711552),
    (257, 20, "QPA_F32", 64, 0, True, 1, 269568),
    (513, 100, "QPA_I8", 2, 0, False, 1, 462592),
    (38, 20, "QPA_I8", 16, 0, False, 3, 210944),
    (300, 100, "QPA_F32", 4, 0, True, 1, 287744),
    (100, 20, "QPA_I8", 64, 0, False, 1, 605952),
    (1001, 100, "QPA_I8", 64, 0, False, 1, 4494336),
    (128, 100, "QPA_I8", 64, 2, False, 1, 632832),
    (4096, 400, "QPA_I8", 300, 0, False, 1, 69532416),
])
def test_batch(q, n, deg, couplings, R, flags, bf16, count, bound):
    a = q.make_params(R, 10, 0.1, 0.8, 4.0, flags=flags,
                      precision=q.QPA_PREC_BF16 if bf16 else q.QPA_PREC_FP32)
    assert batch_size(q, [problem(q, n, couplings, n * deg)] * count, a) <= bound


# couplings, n, replicas: bytes.  Odd sizes, whose canonical rows are padded, and sizes whose
# energies take the most partial sums
@pytest.mark.parametrize("couplings,n,R,bound", [
    ("QPA_F32", 117, 1, 97024),
    ("QPA_I32", 65, 1, 58112),
    ("QPA_I32", 129, 1, 439296),
    ("QPA_F32", 209, 3, 755712),
    ("QPA_I32", 1001, 200, 9542656),
])
def test_dense_solve(q, couplings, n, R, bound):
    out = ctypes.c_size_t()
    p = problem(q, n, couplings)
    a = q.make_params(R, 100, 0.1, 0.8, 1.0)
    assert q._lib.qpa_workspace_size(None, ctypes.byref(p), ctypes.byref(a),
                                     ctypes.byref(out)) == q.QPA_OK
    assert out.value <= bound


@pytest.mark.parametrize("couplings,n,R,bound", [
    ("QPA_I32", 1, 4096, 237568),
    ("QPA_F32", 5, 1, 48384),
    ("QPA_I32", 20, 256, 135680),
    ("QPA_F32", 33, 4096, 2537472),
    ("QPA_I32", 65, 257, 493312),
    ("QPA_F32", 127, 31, 374272),
    ("QPA_F32", 1001, 200, 8536576),
    ("QPA_F32", 4096, 1024, 141338112),
    ("QPA_F32", 5001, 2048, 280956416),
])
def test_dense_sbm(q, couplings, n, R, bound):
    out = ctypes.c_size_t()
    p = problem(q, n, couplings)
    a = q.make_sbm_params(R, 10, 0.5)
    assert q._lib.qpa_workspace_size_sbm(None, ctypes.byref(p), ctypes.byref(a),
                                         ctypes.byref(out)) == q.QPA_OK
    assert out.value <= bound


# (couplings, n), replicas, steps, checkpoint interval: bytes
@pytest.mark.parametrize("couplings,n,R,T,k,bound", [
    ("QPA_F32", 1, 4096, 500, 50, 3892480),
    ("QPA_I32", 1, 1, 1, 1, 45568),
    ("QPA_F32", 5, 1, 5, 2, 94976),
    ("QPA_I32", 33, 64, 100, 10, 1080832),
    ("QPA_F32", 128, 128, 500, 1, 66621952),
    ("QPA_F32", 300, 100, 20, 20, 11527424),
    ("QPA_I32", 1001, 200, 100, 10, 66074112),
    ("QPA_F32", 2048, 65, 500, 50, 206635264),
    ("QPA_F32", 5001, 4096, 500, 50, 14897613312),
])
def test_relaxed_dense(q, couplings, n, R, T, k, bound):
    p = problem(q, n, couplings)
    a = q.make_params(R, T, 0.1, 0.8, 1.0)
    assert q.qpa_workspace_size_relaxed(None, p, a, k) <= bound
