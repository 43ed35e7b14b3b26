"""The salience kernels' units against the float64 oracle: batches of ragged
documents whose 128 x 128 units cross the runs handed to one XCD, with last
blocks of one row, a full block and everything around a 32-row tile.
Tolerances as derived in test_gpu_salience."""
import numpy as np
import pytest

from test_gpu_salience import _free, check_doc, oracle_for, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,p", [(2, 2, 8), (6, 2, 16), (4, 1, 33)])
def test_units_of_ragged_batches(hq, hkv, p):
    rng = np.random.default_rng(hq)
    lens = [385, 1, 384, 129, 256, 33, 255, 417, 128, 95, 97, 353] + \
        [int(n) for n in rng.integers(1, 420, 12)]
    ks = [int(rng.integers(0, n + 1)) for n in lens]
    step, q, k = run_case(lens, hq, hkv, p, n_select=ks, seed=20 + hq,
                          q_scale=float(hq))
    ora = oracle_for(step, q, k, p, range(len(lens)))
    for d in range(len(lens)):
        check_doc(step, d, ora)
    del step
    _free()
