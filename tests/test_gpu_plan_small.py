"""The two-launch scheduler of small batches at the sizes where it can go
wrong (one pair; a wave's, a block's and its own largest number of pairs; the
first batch past it, which takes the general scheduler; document-id spaces on
either side of the sort's digits; everything skipped), against the oracle's
grouping, and its work items and queue orders through the attention."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_harness import compare, run, setup

pytestmark = pytest.mark.gpu

LIMIT = 8192  # pairs the small scheduler takes


@pytest.mark.parametrize("n_pairs", [1, 63, 65, 1023, 1025, LIMIT - 1, LIMIT,
                                     LIMIT + 1])
@pytest.mark.parametrize("n_docs", [1, 255, 256, 65537])
def test_grouping(n_pairs, n_docs):
    import torch
    from paper_2609_03311_amd import (dopr_check_status, dopr_group_pairs,
                                      dopr_prefix_attn_workspace,
                                      dopr_store_create)
    rng = np.random.default_rng(n_pairs * 7 + n_docs)
    lens = rng.integers(-1, 3, n_docs).astype(np.int32)
    ids = rng.integers(-1, n_docs + 1, n_pairs)
    hot = rng.integers(0, n_docs)
    ids[rng.random(n_pairs) < 0.3] = hot
    ids = ids.astype(np.int32)
    store = dopr_store_create(1, 2, 128, lens)
    ws = torch.empty(dopr_prefix_attn_workspace(
        store, n_pairs=n_pairs, n_q_heads=2, max_tokens=1,
        total_tokens=n_pairs), dtype=torch.uint8, device="cuda")
    got = dopr_group_pairs(store, torch.from_numpy(ids).cuda(), ws)
    for a, b in zip(got, oracle.group(ids, lens)):
        assert np.array_equal(a.cpu().numpy(), b)
    dopr_check_status(store)


@pytest.mark.parametrize("variant", [8, 6])
@pytest.mark.parametrize("order", [1, 2])
def test_items_and_orders(variant, order):
    """A hot document cut into many items beside short ones, and pairs
    without a document: both queue orders, against the oracle."""
    rng = np.random.default_rng(3 + order)
    lens = np.array([40, 5, 300, 0, 64, -1], np.int32)
    ids = rng.choice(6, 260, p=[.5, .1, .1, .1, .1, .1]).astype(np.int32)
    toks = rng.choice([1, 3, 33, 70], 260).astype(np.int32)
    st = workloads.custom(lens, ids, toks, 12, 2, name=f"items_{variant}")
    case = setup(st, seed=21, kernel_variant=variant)
    case.step.queue_order = order
    assert run(case) != 0
    bad = np.nonzero(ids == 5)[0][:4]
    compare(case, np.sort(np.concatenate([np.arange(60), bad])))


def _attend(case):
    """The attention alone (the score head reads the row of each pair's last
    token, which malformed ranges put outside the batch)."""
    import torch
    from paper_2609_03311_amd import dopr_check_status
    o, p = case.online, case.prm
    case.step.attention(0, case.doc_ids, case.cu, o["q"], o["k"], o["v"],
                        p["q_norm_w"], p["k_norm_w"])
    torch.cuda.synchronize()
    return dopr_check_status(case.store)


def test_overlapping_token_ranges_are_refused():
    """Ranges that go back and overlap would stack more rows than the plan
    holds: SEQLEN, and nothing is run."""
    import torch
    from paper_2609_03311_amd import DOPR_ERR_SEQLEN
    st = workloads.custom(np.array([8], np.int32), np.zeros(5, np.int32),
                          np.array([20] * 5, np.int32), 4, 2)
    case = setup(st, seed=4, kernel_variant=8)
    case.cu = torch.tensor([0, 100, 0, 100, 0, 100], dtype=torch.int32,
                           device="cuda")
    case.step.max_tokens = 100
    case.step.workspace = torch.empty(1 << 24, dtype=torch.uint8,
                                      device="cuda")
    case.step.out.fill_(7.0)
    assert _attend(case) == DOPR_ERR_SEQLEN
    assert bool((case.step.out == 7.0).all())


@pytest.mark.parametrize("variant", [8, 6, 4])
def test_overlapping_token_ranges_are_refused_past_the_limit(variant):
    """The same of the general scheduler: rows beyond its tables are found
    before any table is written from them.  A batch whose malformed range
    leaves room is still run, that pair excepted."""
    import torch
    from paper_2609_03311_amd import DOPR_ERR_SEQLEN, pipeline
    n = LIMIT + 8
    st = workloads.custom(np.array([8, 3], np.int32),
                          np.arange(n, dtype=np.int32) % 2,
                          np.ones(n, np.int32), 4, 2)
    case = setup(st, seed=5, kernel_variant=variant)
    step = pipeline.OnlineStep(case.store, n_pairs=n, n_q_heads=4,
                               total_tokens=n, max_tokens=100,
                               kernel_variant=variant, with_lse=True)
    case.step = step
    good = case.cu
    case.cu = (torch.arange(n + 1, dtype=torch.int32, device="cuda") % 2) * 100
    step.out.fill_(7.0)
    assert _attend(case) == DOPR_ERR_SEQLEN
    assert bool((step.out == 7.0).all())
    case.cu = good.clone()
    case.cu[n - 1] = n + 5  # the pairs on its two sides are malformed
    step.out.fill_(7.0)
    assert _attend(case) == DOPR_ERR_SEQLEN
    assert bool((step.out[n - 2:] == 7.0).all())
    bad = step.out[:n - 2].clone()
    case.cu = good
    assert _attend(case) == 0
    assert torch.equal(step.out[:n - 2], bad)


def test_timed_interval_leaves_the_plan_out():
    """The timing events hold the attention alone: the launch that fills a small
    batch's tables also zeroes a pair without a document, here 256 MB by one
    block (2 ms), beside one pair of one token (microseconds)."""
    import torch
    st = workloads.custom(np.array([4, -1], np.int32),
                          np.array([0, 1], np.int32),
                          np.array([1, 1 << 17], np.int32), 8, 2)
    case = setup(st, seed=6, kernel_variant=2)
    o, p = case.online, case.prm

    def call(**kw):
        case.step.attention(0, case.doc_ids, case.cu, o["q"], o["k"], o["v"],
                            p["q_norm_w"], p["k_norm_w"], **kw)

    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()  # (creates the handle)
    call()
    ev[0].record()
    call(timing=(ev[1].cuda_event, ev[2].cuda_event))
    ev[3].record()
    torch.cuda.synchronize()
    whole, inside = ev[0].elapsed_time(ev[3]), ev[1].elapsed_time(ev[2])
    assert inside < 0.25 * whole, (whole, inside)
    assert bool((case.step.out[1:] == 0).all())


@pytest.mark.parametrize("variant", [6, 8])
def test_rotary_table_of_a_long_store(variant):
    """A document of 300,000 slots in the store makes the rotary table one of a
    launch of its own; the batch does not name it and keeps its bits."""
    import torch
    rng = np.random.default_rng(8)
    ids = rng.integers(0, 3, 40).astype(np.int32)
    toks = rng.choice([1, 17, 40], 40).astype(np.int32)
    outs = []
    for extra in ([], [300_000]):
        st = workloads.custom(np.array([16, 5, 70] + extra, np.int32), ids,
                              toks, 4, 1)
        case = setup(st, seed=7, kernel_variant=variant)
        if extra:  # the same prefixes as in the short store
            case.store = case.step.store = _store_with(case, keep)
        keep = (case.k_src, case.v_src)
        assert _attend(case) == 0
        outs.append((case.step.out.clone(), case.step.lse.clone()))
    assert torch.equal(outs[0][0].view(torch.int16),
                       outs[1][0].view(torch.int16))
    assert torch.equal(outs[0][1], outs[1][1])


def _store_with(case, keep):
    from paper_2609_03311_amd import pipeline
    for mine, theirs in zip((case.k_src, case.v_src), keep):
        mine[:theirs.shape[0]] = theirs
    return pipeline.make_store(case.st.doc_len, 1, case.k_src, case.v_src)
