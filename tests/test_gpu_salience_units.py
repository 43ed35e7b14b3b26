"""The salience kernels' units against the float64 oracle: batches of ragged
documents whose 128 x 128 units cross the runs handed to one XCD, with last
blocks of one row, a full block and everything around a 32-row tile.
Tolerances as derived in test_gpu_salience."""
import numpy as np
import pytest

import workloads

from test_gpu_salience import (_free, check_doc, cpu_top_k, oracle_for,
                               run_case)

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


@pytest.mark.parametrize("n,p", [(511, 8), (512, 8), (513, 16), (640, 32),
                                 (515, 64)])
def test_wide_strips_and_selection(n, p):
    """Both sides of the length from which a strip has more waves, every list
    size."""
    lens = [n, 3, n - 130]
    step, q, k = run_case(lens, 4, 2, p, n_select=[n // 3, 1, n - 131],
                          seed=30 + p, with_attention=False)
    ora = oracle_for(step, q, k, p, range(3), with_attention=False)
    for d in range(3):
        check_doc(step, d, ora, with_attention=False)
    del step
    _free()


@pytest.mark.parametrize("docs,n,p", [(64, 512, 8), (65, 512, 8),
                                      (16, 1024, 16), (17, 1024, 16),
                                      (16, 1023, 16), (3, 1024, 32)])
def test_strips_of_few_and_many_documents(docs, n, p):
    """Both sides of the numbers of strips, and for lists of 16 of the length,
    up to which a strip has sixteen waves."""
    lens = [n] + [n - 1] * (docs - 2) + [5]
    step, q, k = run_case(lens, 1, 1, p, n_select=[m // 3 for m in lens],
                          seed=50 + docs, with_attention=False)
    some = [0, docs // 2, docs - 2, docs - 1]
    ora = oracle_for(step, q, k, p, some, with_attention=False)
    for d in some:
        check_doc(step, d, ora, with_attention=False)
    del step
    _free()


def test_selection_of_equal_values():
    """All u equal, two values, infinities and zeros of both signs: the lower
    positions are taken first."""
    import torch
    import paper_2609_03311_amd as D
    n = 1000
    rng = np.random.default_rng(5)
    rows = [np.zeros(n), np.full(n, 0.25), rng.choice([0.5, 0.25], n),
            rng.choice([np.inf, 1e-30, 0.0, 3.0], n),
            np.float32(1) + rng.integers(0, 40, n) * 2.0 ** -23]
    u = torch.tensor(np.concatenate(rows), dtype=torch.float32,
                     device="cuda")
    cu = torch.arange(0, (len(rows) + 1) * n, n, dtype=torch.int32,
                      device="cuda")
    for k in (1, 333, 999):
        cs = torch.arange(0, (len(rows) + 1) * k, k, dtype=torch.int32,
                          device="cuda")
        sel = torch.full((len(rows) * k,), -1, dtype=torch.int32,
                         device="cuda")
        D.dopr_select_top_k(cu, cs, u, sel, max_doclen=n)
        torch.cuda.synchronize()
        for r, x in enumerate(rows):
            got = sel[r * k:(r + 1) * k].cpu().numpy()
            assert np.array_equal(got, cpu_top_k(x.astype(np.float32), k))


def test_rows_of_many_heads():
    """A token of 133,200 q heads is 34 MB, so row 126 of a block starts past
    2^32 bytes.  Every head holds the same query, so the mean over heads is
    one head's attention; the fp32 sum of n equal terms is within n 2^-24 of
    n times one."""
    import torch
    n, hq, p = 127, 133200, 8
    q1, k = workloads.salience_inputs([n], 1, 1, "cuda", 40, 2.0)
    q = q1.expand(n, hq, 128).contiguous()
    step, _, _ = run_case([n], hq, 1, p, n_select=[16], q=q, k=k)
    ora = oracle_for(step, q1, k, p, [0])
    tol = hq * 2.0 ** -24
    low = np.tril(np.ones((n, n), bool))
    a = step.attn_mean[0].cpu().numpy().astype(np.float64)[low]
    ref = ora["attention"][0][low]
    assert (np.abs(a - ref) <= tol * ref + 1e-12).all()
    u, uo = step.u.cpu().numpy(), ora["u"][0]
    assert (np.abs(u - uo) <= tol * uo + 1e-12).all()
    del step, q
    _free()


@pytest.mark.parametrize("hq,hkv", [(1, 1), (2, 2), (6, 3), (6, 2), (7, 1)])
@pytest.mark.parametrize("longest", [64, 130])
def test_short_documents(hq, hkv, longest):
    """Documents of up to 64 tokens take one tile per wave: lengths around its
    tiles, alone and beside a longer document."""
    lens = [1, 2, 31, 32, 33, 48, 63, 64, longest, 65 if longest > 64 else 7]
    step, q, k = run_case(lens, hq, hkv, 4, n_select=[m // 2 for m in lens],
                          seed=60 + hq)
    ora = oracle_for(step, q, k, 4, range(len(lens)))
    for d in range(len(lens)):
        check_doc(step, d, ora)
    del step
    _free()
