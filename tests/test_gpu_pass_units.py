"""The pass kernel's work units (128 stacked rows, keys in batches of two
32-key chunks) at the sizes where they can go wrong: token counts and prefix
lengths around a chunk, a batch and a unit, one-token pairs, every way the
lanes share a token's rotary pairs, and non-finite values next to masked
keys.  Each row's sums are formed in the block kernels' order, so the outputs
must be bitwise those of variant 2."""
import numpy as np
import pytest

import workloads
from gpu_harness import compare, run, setup

pytestmark = pytest.mark.gpu

TOKENS = [1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 160]
SLOTS = [0, 1, 7, 8, 31, 32, 33, 63, 64, 65, 96, 97, 256, 257]


def _outputs(case, variant, order=0):
    import torch
    from paper_2609_03311_amd import pipeline
    st, o, p = case.st, case.online, case.prm
    step = pipeline.OnlineStep(case.store, n_pairs=st.n_pairs,
                               n_q_heads=st.n_q_heads,
                               total_tokens=st.n_tokens,
                               max_tokens=int(st.seqlens.max()),
                               kernel_variant=variant, with_lse=True,
                               queue_order=order)
    step.out.fill_(float("nan"))
    step.attention(0, case.doc_ids, case.cu, o["q"], o["k"], o["v"],
                   p["q_norm_w"], p["k_norm_w"])
    torch.cuda.synchronize()
    return step.out, step.lse


@pytest.mark.parametrize("n_rep,d", [(1, 128), (2, 128), (3, 128), (4, 128),
                                     (8, 128), (1, 64), (2, 64), (4, 64)])
def test_units_match_the_block_kernel(n_rep, d):
    import torch
    rng = np.random.default_rng(100 * n_rep + d)
    lens = np.array(SLOTS + [-1], np.int32)
    # every length with two to four pairs of random token counts, then a
    # document with many one-token pairs, and two pairs without a document
    ids = np.concatenate([np.repeat(np.arange(len(SLOTS)),
                                    rng.integers(2, 5, len(SLOTS))),
                          np.full(150, 4), [len(SLOTS), len(SLOTS)]])
    toks = rng.choice(TOKENS, len(ids))
    toks[-152:-2] = 1
    order = rng.permutation(len(ids))
    st = workloads.custom(lens, ids[order], toks[order], 2 * n_rep, 2,
                          name=f"units_{n_rep}_{d}", head_dim=d)
    case = setup(st, seed=9, kernel_variant=8)
    assert run(case) != 0  # the pairs without a document are reported
    ok = np.nonzero(st.doc_ids != len(SLOTS))[0]
    compare(case, ok[:24])
    out8, lse8 = _outputs(case, 8)
    out2, lse2 = _outputs(case, 2)
    assert torch.equal(out8.view(torch.int16), out2.view(torch.int16))
    assert torch.equal(lse8, lse2)


@pytest.mark.parametrize("d", [128, 64])
def test_non_finite_values_stay_with_their_pair(d):
    """Infinite values in the v of a document's only pair: the rows of other
    documents keep their bits (a chunk's rows past its pair's end are read as
    zeros, not as the next pair's values)."""
    import torch
    lens = np.array([33, 40, 5], np.int32)
    ids = np.array([0, 0, 1, 0, 2, 2], np.int32)
    toks = np.array([33, 40, 65, 7, 1, 129], np.int32)
    st = workloads.custom(lens, ids, toks, 8, 2, name="inf", head_dim=d)
    case = setup(st, seed=10, kernel_variant=8)
    clean, _ = _outputs(case, 8)
    clean = clean.clone()
    bad = 2                                # pair whose values are infinite
    a, b = int(st.cu_seqlens[bad]), int(st.cu_seqlens[bad + 1])
    case.online["v"][a:b] = float("inf")
    o8, _ = _outputs(case, 8)
    o2, _ = _outputs(case, 2)
    keep = torch.ones(st.n_tokens, dtype=torch.bool, device=o8.device)
    keep[a:b] = False
    assert torch.equal(o8[keep].view(torch.int16),
                       clean[keep].view(torch.int16))
    assert torch.equal(torch.isnan(o8), torch.isnan(o2))
    assert torch.equal(torch.nan_to_num(o8.float()),
                       torch.nan_to_num(o2.float()))


@pytest.mark.parametrize("d,slots,tokens", [
    (128, 40, 4095), (128, 40, 4096), (128, 300, 4095), (128, 300, 4096),
    (128, 300, 32), (128, 8, 1), (64, 300, 33), (64, 257, 32), (64, 256, 32),
    (64, 256, 1)])
def test_automatic_choice_on_both_sides_of_its_line(d, slots, tokens):
    """The pass kernel, except at head size 64 for at most 128 stacked rows
    with a prefix of more than 256 slots: that batch's plan holds no own keys.
    All give the block kernel's bits."""
    import torch
    import paper_2609_03311_amd as D
    lens = np.array([slots, 7, 0], np.int32)
    n = min(32, tokens)
    toks = np.full(n, min(129, tokens // n), np.int32)
    toks[-1] += tokens - toks.sum()
    st = workloads.custom(lens, np.arange(n) % 3, toks, 8, 2, name="line",
                          head_dim=d)
    case = setup(st, seed=11)
    assert run(case) == 0
    compare(case, np.arange(0, n, 5))
    out0, lse0 = _outputs(case, 0)
    out2, lse2 = _outputs(case, 2)
    assert torch.equal(out0.view(torch.int16), out2.view(torch.int16))
    assert torch.equal(lse0, lse2)
    need = [D.dopr_prefix_attn_workspace(
                case.store, n_pairs=st.n_pairs, n_q_heads=st.n_q_heads,
                max_tokens=int(toks.max()), total_tokens=tokens,
                kernel_variant=v) for v in (0, 2)]
    khat = 2 * tokens * 2 * d
    block = d == 64 and slots > 256 and 4 * tokens <= 128
    assert (need[0] >= need[1] + khat) == (not block)


@pytest.mark.parametrize("n_rep", [(1 << 15) - 1, 1 << 15, 65537])
def test_groups_of_many_heads(n_rep):
    """The pass kernel divides rows by n_rep with a multiplied reciprocal and
    keeps a head number in 24 bits: from 2^15 heads per kv head on the block
    kernels run in its place (at 65,537 the reciprocal would take a row of one
    token for the next token's)."""
    import torch
    import paper_2609_03311_amd as D
    toks = np.array([2, 1, 2], np.int32)
    st = workloads.custom(np.array([5, 33], np.int32),
                          np.array([0, 1, 0], np.int32), toks, n_rep, 1,
                          name=f"heads_{n_rep}", head_dim=64)
    case = setup(st, seed=12, kernel_variant=2)
    need = {v: D.dopr_prefix_attn_workspace(
                case.store, n_pairs=3, n_q_heads=n_rep, max_tokens=2,
                total_tokens=5, kernel_variant=v) for v in (0, 8, 2)}
    for v in (0, 8):
        assert (need[v] > need[2]) == (n_rep < 1 << 15), (v, need)
    out2, lse2 = _outputs(case, 2)
    for v in (8, 0):
        out, lse = _outputs(case, v)
        assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
        assert torch.equal(lse, lse2)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("rounds,extra", [(0, 1), (0, 9), (1, -1), (1, 0),
                                          (1, 1), (3, -1), (3, 0), (3, 1),
                                          (4, 5)])
def test_units_dealt_out(rounds, extra, order):
    """As many units as the launch has blocks (two per CU, in multiples of
    eight), times the three rounds that are dealt out, and next to that: every
    unit is run once, in the queues' own order and longest first."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = rounds * 2 * ((cus + 7) // 8 * 8) + extra
    rng = np.random.default_rng(n)
    st = workloads.custom(rng.integers(0, 40, n).astype(np.int32),
                          rng.permutation(n).astype(np.int32),
                          rng.integers(1, 4, n).astype(np.int32), 1, 1,
                          name=f"dealt_{n}")
    case = setup(st, seed=13, kernel_variant=8)
    out2, lse2 = _outputs(case, 2)
    out, lse = _outputs(case, 8, order)
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
    assert torch.equal(lse, lse2)
