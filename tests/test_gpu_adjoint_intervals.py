"""Relaxed gradient at several checkpoint intervals, where the steps at the ends of the
segments form their FP64 sums in another launch than the others.  The loss is the same bit for
bit; sparse instances of one type give the gradients bit for bit too.  A dense instance and a
batch of two coupling types group those sums differently: each gradient is a sum of N terms in
FP64, so two orders of it agree to N 2^-53 of the sum of magnitudes, here bounded by 1e-10 of
the largest step gradient (N < 2^17; cancellation of less than 2^13)."""
import numpy as np
import pytest

from paper_2501_19221_amd import instances as gen

pytestmark = pytest.mark.gpu


def _batch(kind):
    rng = np.random.default_rng(6)
    er = gen.er_qubo(300, 0.1, 100, rng)
    if kind == "one type":
        return [er, gen.er_qubo(150, 0.2, 100, rng)], True
    if kind == "dense":
        return [gen.sk_ising(300, 0.1, seed=8)], False
    return [er, gen.er_qubo(150, 0.2, 100, rng, idx_dtype=np.int32),
            gen.sk_ising(90, 0.1, seed=9)], False


@pytest.mark.parametrize("kind", ["one type", "dense", "mixed"])
def test_intervals(kind):
    import torch
    from paper_2501_19221_amd import qpa
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    insts, exact = _batch(kind)
    eng = qpa.Engine(0)
    probs = [qpa.Problem.from_instance(i) for i in insts]
    T = 70
    p = qpa.make_params(70, T, 0.002, 0.8, 4.0, 0.1, 3)
    ref = None
    for k in (70, 1, 7, 33, 100):
        print("checkpoint interval %d, %s" % (k, kind), flush=True)
        got = [g.cpu().numpy() for g in eng.relaxed_grad(probs, p, k)]
        ref = got if ref is None else ref
        assert np.array_equal(got[0], ref[0]), k
        bound = 0.0 if exact else 1e-10 * np.max(np.abs(ref[3]))
        for a, b in zip(got[1:], ref[1:]):          # d_eta, d_alpha sum T steps, d_lambda one
            assert np.max(np.abs(a - b)) <= bound * (T if a.size == 1 else 1), k
    eng.close()
