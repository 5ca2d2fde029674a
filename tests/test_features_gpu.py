"""GPU parity of MBR decoding, the gold-tree loss, one-stage labelled decoding
and the labelling stage: the HIP library through the C ABI against the
float64 oracle.

Tolerances (as for the other entry points):
  log Z, loss   |gpu - oracle| <= 1e-5 * max(1, |log Z|)  (the loss is log Z
                minus an exact float64 sum of gold scores, so it inherits log
                Z's absolute error)
  marginals, gradients   |gpu - oracle| <= 1e-4 on every valid cell
  trees, labels          bit-exact.  MBR trees are compared with the oracle's
                CKY over the kernel's own float32 marginals (the decision is
                taken on those values on both sides); the oracle's own MBR
                tree, on its float64 marginals rounded to float32, may differ
                at near ties, so against it the GPU tree must score within
                the marginal tolerance per span.
"""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2008_03736_amd import binding as B
from paper_2008_03736_amd import workloads as W

pytestmark = pytest.mark.gpu

LOGZ_RTOL = 1e-5
MARG_ATOL = 1e-4
TH = 16


@pytest.fixture(scope="module")
def torch():
    import torch as _t

    if not _t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load()
    return _t


def _dev(torch):
    return torch.device("cuda", 0)


def check_close(gpu, ref, scale_ref, what):
    err = np.abs(np.asarray(gpu, np.float64) - ref)
    bound = LOGZ_RTOL * np.maximum(1.0, np.abs(scale_ref))
    bad = np.nonzero(err > bound)[0]
    assert bad.size == 0, f"{what} mismatch at {bad[:5]}: gpu {np.asarray(gpu)[bad[:5]]} ref {ref[bad[:5]]}"


def check_cells(gpu, ref, lengths, n1, what, fill=None):
    v = W.valid_mask(np.asarray(lengths), n1)
    err = np.abs(gpu[v].astype(np.float64) - ref[v])
    worst = float(err.max()) if err.size else 0.0
    assert worst <= MARG_ATOL, f"max |{what} error| {worst:.3e}"
    if fill is not None:
        assert np.all(gpu[~v] == np.float32(fill)), f"{what}: padding written"
    return worst


# --------------------------------------------------------------------------
# MBR decoding (Sec. 3.3)


def mbr_check(torch, b, flags=0, expect_fused=None):
    dev = _dev(torch)
    s = torch.from_numpy(b.scores).to(dev)
    with B.Plan(b.lengths, n1=b.n1, flags=flags, device=dev) as plan:
        info = plan.info
        marg = torch.full_like(s, -7.0)
        lz, mu, sp, be = plan.mbr_decode(s, marginals=marg)
        torch.cuda.synchronize()
    lz, mu, sp, be = (x.cpu().numpy() for x in (lz, mu, sp, be))
    if expect_fused is not None:
        assert info["mbr_fused"] == expect_fused
    lz_ref, mu_ref = orc.marginals(b.scores, b.lengths, threads=TH)
    check_close(lz, lz_ref, lz_ref, "logZ")
    worst = check_cells(mu, mu_ref, b.lengths, b.n1, "marginal", fill=-7.0)
    # the decision, on the kernel's own float32 marginals: bit-exact
    sp_ref, be_ref, _ = orc.mbr(b.scores, b.lengths, threads=TH, marginals_f32=np.where(
        W.valid_mask(b.lengths, b.n1), mu, np.nan).astype(np.float32))
    bad = np.nonzero((sp != sp_ref).any(axis=(1, 2)))[0]
    assert bad.size == 0, f"MBR trees differ for sentences {bad[:10]}"
    assert np.array_equal(be, be_ref.astype(np.float32))
    # against the oracle's own MBR decoding: at least as good up to the
    # marginal tolerance per span
    sp_o, be_o, mu32 = orc.mbr(b.scores, b.lengths, threads=TH)
    for bi, n in enumerate(b.lengths):
        n = int(n)
        got = sum(float(mu_ref[bi, i, j]) for i, j in sp[bi, : 2 * n - 1])
        opt = sum(float(mu_ref[bi, i, j]) for i, j in sp_o[bi, : 2 * n - 1])
        assert got >= opt - 2 * (2 * n - 1) * MARG_ATOL, (bi, got, opt)
    return worst, info


@pytest.mark.parametrize("name", ["tiny", "mixed", "longer"])
def test_mbr_workloads(torch, name):
    worst, info = mbr_check(torch, W.make(name), expect_fused=1)
    print(f"MBR {name}: max |marginal error| {worst:.2e}")


def test_mbr_stress_workspace_sentences(torch):
    # n = 256: marginals and CKY on the workspace kernels, as two launches
    b = W.make("stress")
    worst, info = mbr_check(torch, b)
    assert info["spill_count"] == b.B
    print(f"MBR stress: max |marginal error| {worst:.2e}")


def test_mbr_mixed_lds_and_workspace(torch):
    # bundles in LDS beside workspace sentences in one plan, and edge lengths
    b = W.custom([1, 2, 3, 97, 99, 143, 150, 40, 1, 12], seed=31, sd=2.0)
    mbr_check(torch, b, expect_fused=1)


def test_mbr_force_spill_separate_launches(torch):
    b = W.custom([1, 2, 9, 33, 70], seed=32, sd=2.0)
    mbr_check(torch, b, flags=B.CRF_FORCE_SPILL, expect_fused=0)


def test_mbr_all_zero_scores(torch):
    # equal scores: Catalan-ratio marginals, many exact ties in the MBR chart
    mbr_check(torch, W.custom([1, 2, 5, 40, 99], sd=0.0))


# --------------------------------------------------------------------------
# Gold-tree loss (Sec. 2.3, Eq. bracket-loss)


def _right_branching(lengths, n1):
    R = 2 * (n1 - 1) - 1
    out = np.full((len(lengths), R, 2), -1, np.int32)
    for b, n in enumerate(lengths):
        rows = []
        for i in range(n - 1):
            rows += [(i, n), (i, i + 1)]
        rows.append((n - 1, n))
        out[b, : len(rows)] = rows
    return out


def loss_check(torch, b, gold, grad=None, flags=0):
    dev = _dev(torch)
    s = torch.from_numpy(b.scores).to(dev)
    gy = torch.from_numpy(np.ascontiguousarray(gold, np.int32)).to(dev)
    g = None if grad is None else torch.tensor(grad, dtype=torch.float32, device=dev)
    with B.Plan(b.lengths, n1=b.n1, flags=flags, device=dev) as plan:
        gr = torch.full_like(s, 5.5)
        lv, gr = plan.gold_loss(s, gy, grad_loss=g, grad_scores=gr)
        torch.cuda.synchronize()
    lv, gr = lv.cpu().numpy(), gr.cpu().numpy()
    l_ref, g_ref = orc.loss(b.scores, b.lengths, gold, grad=grad, threads=TH)
    lz_ref = orc.logz(b.scores, b.lengths, threads=TH)
    check_close(lv, l_ref, lz_ref, "loss")
    return check_cells(gr, g_ref, b.lengths, b.n1, "gradient", fill=5.5)


@pytest.mark.parametrize("name", ["tiny", "mixed", "longer", "stress"])
def test_loss_workloads(torch, name):
    b = W.make(name)
    gold, _ = orc.cky(b.scores, b.lengths, threads=TH)       # one gold tree per sentence
    w1 = loss_check(torch, b, gold)
    w2 = loss_check(torch, b, _right_branching(b.lengths, b.n1))
    print(f"loss {name}: max |gradient error| {w1:.2e} (CKY trees), {w2:.2e} (right-branching)")


def test_loss_upstream_gradient_and_spill(torch):
    b = W.custom([1, 2, 7, 30, 99, 150], seed=41, sd=2.0)
    gold, _ = orc.cky(b.scores, b.lengths)
    loss_check(torch, b, gold, grad=[1.0, 2.0, -0.5, 0.0, 3.0, 0.25])
    loss_check(torch, b, gold, grad=[1.0, 2.0, -0.5, 0.0, 3.0, 0.25], flags=B.CRF_FORCE_SPILL)


def test_loss_skips_rows_that_are_not_spans(torch):
    # a row that is not a span of its sentence is skipped (memory-safe); a
    # repeated span adds its score again but the indicator once
    b = W.custom([9, 20], seed=42, sd=1.5)
    gold, _ = orc.cky(b.scores, b.lengths)
    l_ref, g_ref = orc.loss(b.scores, b.lengths, gold)
    bad = gold.copy()
    i0, j0 = gold[0, 4]
    bad[0, 4] = (7, 3)                        # dropped: its score leaves s(x,y), its cell the indicator
    i1, j1 = gold[1, 2]
    i2, j2 = gold[1, 6]
    bad[1, 6] = (i1, j1)                      # a repeat replaces row 6
    dev = _dev(torch)
    s = torch.from_numpy(b.scores).to(dev)
    with B.Plan(b.lengths, device=dev) as plan:
        lv, gr = plan.gold_loss(s, torch.from_numpy(bad).to(dev))
        torch.cuda.synchronize()
    lv, gr = lv.cpu().numpy(), gr.cpu().numpy()
    s0, s1, s2 = (float(b.scores[0, i0, j0]), float(b.scores[1, i1, j1]), float(b.scores[1, i2, j2]))
    exp_l = l_ref + np.array([s0, s2 - s1])
    lz_ref = orc.logz(b.scores, b.lengths)
    check_close(lv, exp_l, lz_ref, "loss")
    exp_g = g_ref.copy()
    exp_g[0, i0, j0] += 1.0                   # no longer gold
    exp_g[1, i2, j2] += 1.0
    check_cells(gr, exp_g, b.lengths, b.n1, "gradient")


# --------------------------------------------------------------------------
# One-stage labelled decoding (Sec. 4.2, Eq. tree-label-score)


def lcky_check(torch, b, flags=0):
    dev = _dev(torch)
    s = torch.from_numpy(b.scores).to(dev)
    with B.Plan(b.lengths, n1=b.n1, num_labels=b.num_labels, flags=flags, device=dev) as plan:
        sp, lab, be = plan.cky_decode_labeled(s)
        torch.cuda.synchronize()
    sp, lab, be = sp.cpu().numpy(), lab.cpu().numpy(), be.cpu().numpy()
    s4 = b.scores if b.scores.ndim == 4 else b.scores[..., None]
    sp_ref, lab_ref, be_ref = orc.labeled_cky(s4, b.lengths, threads=TH)
    bad = np.nonzero((sp != sp_ref).any(axis=(1, 2)) | (lab != lab_ref).any(axis=1))[0]
    assert bad.size == 0, f"labelled trees differ for sentences {bad[:10]}"
    assert np.array_equal(be, be_ref.astype(np.float32))


def test_labeled_cky_workload(torch):
    lcky_check(torch, W.make("labeled"))


@pytest.mark.parametrize("labels", [1, 2, 33, 138, 139])
def test_labeled_cky_label_counts(torch, labels):
    lcky_check(torch, W.custom([1, 2, 5, 17, 40, 64], seed=400 + labels, sd=1.0, labels=labels))


def test_labeled_cky_step_shape_boundaries(torch):
    # both sides of every change of step shape (a step per width), and of LDS
    lcky_check(torch, W.custom([2, 3, 4, 5, 6, 9, 10, 17, 18, 33, 34, 49, 50, 65, 66, 97, 98, 129, 130, 141, 142, 143],
                               seed=45, sd=1.0, labels=2))


def test_labeled_cky_ties_and_workspace(torch):
    # integer scores: equal labels and equal trees; a 150-word sentence on the
    # workspace kernel
    lcky_check(torch, W.custom([3, 8, 30, 150], seed=43, labels=4, integer=(-1, 1)))
    lcky_check(torch, W.custom([2, 9, 20], seed=44, labels=5, sd=1.0), flags=B.CRF_FORCE_SPILL)


# --------------------------------------------------------------------------
# Labelling stage (Sec. 2.1, Eq. label-argmax)


@pytest.mark.parametrize("labels,integer", [(26, None), (138, None), (7, (-1, 1)), (1, None)])
def test_label_spans_two_stage(torch, labels, integer):
    # bracketing scores decode the trees; separate label scores label them
    b = W.make("tiny")
    lab = W.custom(b.lengths, seed=50 + labels, sd=1.0, labels=labels, integer=integer)
    s4 = lab.scores if lab.scores.ndim == 4 else np.ascontiguousarray(lab.scores[..., None])
    dev = _dev(torch)
    s = torch.from_numpy(b.scores).to(dev)
    ls = torch.from_numpy(s4).to(dev)
    with B.Plan(b.lengths, n1=b.n1, device=dev) as plan:
        spans, _ = plan.cky_decode(s)
        got = plan.label_spans(ls, spans)
        torch.cuda.synchronize()
    spans, got = spans.cpu().numpy(), got.cpu().numpy()
    ref = orc.label_spans(s4, b.lengths, spans, threads=TH)
    assert np.array_equal(got, ref)
    assert (got[spans[..., 0] < 0] == -1).all()


def test_label_spans_rows_that_are_not_spans(torch):
    b = W.custom([6, 11, 1], seed=51, sd=1.0, labels=9)
    rng = np.random.default_rng(3)
    R = 2 * (b.n1 - 1) - 1
    sp = rng.integers(-2, b.n1 + 2, size=(b.B, R, 2)).astype(np.int32)
    sp[0, 0] = (0, 6)
    sp[1, 1] = (3, 4)
    dev = _dev(torch)
    with B.Plan(b.lengths, n1=b.n1, device=dev) as plan:
        got = plan.label_spans(torch.from_numpy(b.scores).to(dev), torch.from_numpy(sp).to(dev))
        torch.cuda.synchronize()
    ref = orc.label_spans(b.scores, b.lengths, sp)
    assert np.array_equal(got.cpu().numpy(), ref)
    assert (ref != -1).sum() >= 2 and (ref == -1).sum() >= 1
