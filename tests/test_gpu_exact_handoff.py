"""The pass kernel's hand-over to the exact pass: units over the logit bound
(by the gains of the whole call, or by one document's stored keys), rows whose
normaliser leaves the reference-free range, and self-check mode.  Batches of
several units per block, flagged units beside clean ones.

Against variant 2, bitwise, where both kernels send the same rows through the
same softmax mode (a unit with a row that the bounded reference cannot hold
takes the exact mode whole, so the units must be the same); else against exact
mode (variant 4) on the same operands.  There the weights are rounded to bf16
under another reference, 2^-9 of each at most on either side, and O, an average
of values v with these weights, once more: |dO| <= 2 (2^-9 + 2^-9) max|v|.  The
LSE is checked to 1e-3 of its largest value."""
import numpy as np
import pytest

import workloads
from gpu_harness import compare, log, setup

pytestmark = pytest.mark.gpu

HEAD_SIZES = [128, 64]


def _batch(d, pairs=420, tokens=(1, 65, 129), seed=1):
    rng = np.random.default_rng(seed)
    lens = np.array([0, 40, 300, 97, 5, 256], np.int32)
    ids = rng.choice(len(lens), pairs, p=[.05, .1, .45, .1, .1, .2])
    return workloads.custom(lens, ids.astype(np.int32),
                            rng.choice(tokens, pairs).astype(np.int32), 8, 2,
                            name=f"handoff_{d}", head_dim=d)


def _attend(case, variant, norm=True, rows_per_item=0):
    import torch
    from paper_2609_03311_amd import dopr_check_status, pipeline
    st, o, p = case.st, case.online, case.prm
    step = pipeline.OnlineStep(case.store, n_pairs=st.n_pairs,
                               n_q_heads=st.n_q_heads,
                               total_tokens=st.n_tokens,
                               max_tokens=int(st.seqlens.max()),
                               kernel_variant=variant, with_lse=True,
                               rows_per_item=rows_per_item)
    step.out.fill_(float("nan"))
    step.lse.fill_(float("nan"))
    step.attention(0, case.doc_ids, case.cu, o["q"], o["k"], o["v"],
                   p["q_norm_w"] if norm else None,
                   p["k_norm_w"] if norm else None)
    torch.cuda.synchronize()
    assert dopr_check_status(case.store) == 0
    return step.out, step.lse


def _same_bits(a, b, rows=slice(None)):
    import torch
    same = torch.equal(a[0][rows].view(torch.int16),
                       b[0][rows].view(torch.int16))
    assert same and torch.equal(a[1][rows], b[1][rows])


def _close(case, a, b):
    import torch
    tol = 2.0 ** -7 * max(case.online["v"].float().abs().max().item(),
                          case.v_src.float().abs().max().item())
    assert torch.isfinite(a[0].float()).all() and torch.isfinite(a[1]).all()
    d = (a[0].float() - b[0].float()).abs().max().item()
    dl = (a[1] - b[1]).abs().max().item()
    log(f"max|dO| {d:.3e} (bound {tol:.3e}) max|dlse| {dl:.3e}")
    assert d <= tol and dl <= 1e-3 * b[1].abs().max().item()


@pytest.mark.parametrize("d", HEAD_SIZES)
@pytest.mark.parametrize("pairs,tokens", [(420, (1, 65, 129)), (9000, (1, 2))],
                         ids=["small_plan", "general_plan"])
def test_gains_over_the_bound(d, pairs, tokens):
    """Every unit is over the bound by the gains alone: the items are cut like
    the block kernels', to the size asked for or, these batches being small, to
    128 rows."""
    case = setup(_batch(d, pairs, tokens), seed=31, kernel_variant=8)
    for w in ("q_norm_w", "k_norm_w"):
        case.prm[w] = case.prm[w] * 6
    exact = _attend(case, 4)
    for rpi in (0, 64, 4096):
        got = _attend(case, 8, rows_per_item=rpi)
        _same_bits(got, _attend(case, 2, rows_per_item=rpi or 128))
        _close(case, got, exact)
    _same_bits(_attend(case, 0), _attend(case, 2, rows_per_item=128))
    _same_bits(_attend(case, 5), exact)


@pytest.mark.parametrize("d", HEAD_SIZES)
@pytest.mark.parametrize("pairs,tokens", [(420, (1, 65, 129)), (9000, (1, 2))],
                         ids=["small_plan", "general_plan"])
def test_documents_over_the_bound_beside_others(d, pairs, tokens):
    """Two documents' stored keys are twelve times longer than the gains
    allow: their units go to the exact pass, the others are run here."""
    import torch
    from paper_2609_03311_amd import pipeline
    st = _batch(d, pairs, tokens, seed=2)
    case = setup(st, seed=32, kernel_variant=8)
    k = case.k_src.float()
    for doc in (2, 4):
        a = int(case.doc_off[doc])
        k[a:a + int(st.doc_len[doc])] *= 12.0
    case.k_src.copy_(k.to(torch.bfloat16))
    case.store = pipeline.make_store(st.doc_len, st.n_kv_heads, case.k_src,
                                     case.v_src)
    got = _attend(case, 8)
    clean = np.nonzero(np.isin(st.doc_ids, [0, 1, 3, 5]))[0]
    rows = torch.from_numpy(np.concatenate(
        [np.arange(st.cu_seqlens[p], st.cu_seqlens[p + 1]) for p in clean]))
    _same_bits(got, _attend(case, 2), rows.cuda())
    _close(case, got, _attend(case, 4))
    case.step.store, case.step.out, case.step.lse = case.store, *got
    case.step.score_head(case.cu, case.prm["norm_w"], case.prm["w_head"])
    compare(case, clean[:12])


@pytest.mark.parametrize("d", HEAD_SIZES)
def test_rows_out_of_range_beside_others(d):
    """Without QK-norm, queries of some pairs scaled by 40: rows whose
    normaliser the reference-free softmax cannot hold flag their unit."""
    st = _batch(d, seed=3)
    case = setup(st, seed=33, kernel_variant=8)
    q = case.online["q"]
    for p in range(0, st.n_pairs, 7):
        q[int(st.cu_seqlens[p]):int(st.cu_seqlens[p + 1])] *= 40
    exact = _attend(case, 4, norm=False)
    _close(case, _attend(case, 8, norm=False), exact)
    _close(case, _attend(case, 0, norm=False), exact)
    _same_bits(_attend(case, 5, norm=False), exact)


@pytest.mark.parametrize("d", HEAD_SIZES)
def test_self_check_through_the_pass_kernel(d):
    """Self-check mode on a batch that takes the pass kernel: every unit is
    queued once more and comes out of the exact pass."""
    case = setup(_batch(d, seed=4), seed=34, kernel_variant=5)
    assert case.st.n_tokens * 4 >= 16384
    _same_bits(_attend(case, 5), _attend(case, 4))
