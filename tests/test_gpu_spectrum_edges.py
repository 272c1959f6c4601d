"""The spectrum at the edges of its sort and packing, equal to the oracle: replica counts around
a wave and a workgroup, one group over several waves, states that differ in the last word
only, more than 64 words a state."""
import numpy as np
import pytest

from test_gpu_spectrum import _check, eng, q  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [2, 63, 64, 65, 128, 1023, 1025, 2049])
@pytest.mark.parametrize("n", [65, 520, 4161])
def test_sizes(eng, R, n):  # noqa: F811
    rng = np.random.default_rng(R * n)
    print("R=%d n=%d" % (R, n), flush=True)
    base = (2 * rng.integers(0, 2, n) - 1).astype(np.int8)
    pool = np.repeat(base[None], 6, 0)
    pool[1, -1] *= -1                       # the last spin
    pool[2, 0] *= -1
    pool[3, 63 % n] *= -1
    pool[4:] = (2 * rng.integers(0, 2, (2, n)) - 1).astype(np.int8)
    # most samples are one state; three states share an energy
    pick = np.where(rng.random(R) < 0.7, 0, rng.integers(0, 6, R))
    e = np.array([3.0, 3.0, -2.0, 3.0, 7.0, -2.0])[pick]
    for flags in (0, 1):
        _check(eng, pool[pick], e, 4, flags)
        _check(eng, pool[pick], e, R, flags)
