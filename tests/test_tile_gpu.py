"""Tile charts (crf_tile.hip) against the oracle where they can go wrong: the
edges of the four-post blocks, bundles of mixed lengths and of many short
sentences, the stage counts at which lanes start to share a tile, the lengths
at which a chart moves from half a CU's LDS to a whole one and out of LDS, the
rescale points, and bundles whose linear-domain values leave float32's range.

Tolerances as in test_parity_gpu.py: float32 against float64, 1e-5 relative on
log Z and 1e-4 on marginals; trees and scores bit for bit.
"""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2008_03736_amd import binding as B
from paper_2008_03736_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = {
    # every position of the last post in its block, one block to four
    "block_edges": dict(lengths=list(range(1, 17)) * 3),
    # a bundle of one block count holds several lengths
    "mixed_bundles": dict(lengths=[20, 21, 22, 23] * 40 + [3, 2, 1] * 70),
    # many sentences a bundle: the caps on tiles and row pieces per thread
    "many_short": dict(lengths=[1, 2, 3] * 400 + [4, 5, 8, 11] * 150),
    # around the first rescale (12 blocks) and half a CU (25 and 26 blocks)
    "rescale_and_half_cu": dict(lengths=[43, 44, 47, 48, 95, 96, 99]),
    "whole_cu": dict(lengths=[99, 100, 103, 104, 127, 128, 139]),
    # 140 words and more: past LDS
    "past_tiles": dict(lengths=[139, 140, 142, 143, 5]),
    # (CKY alone keeps these in LDS, a width a step)
    "one_block_past": dict(lengths=[140, 12, 141, 99, 30, 140]),
    "padding": dict(lengths=[9, 1, 30, 2], n1=41),
    # integer scores: ties between splits inside a block, between blocks and
    # between the lanes that share a tile
    "ties": dict(lengths=list(range(2, 60, 3)) + [90, 99], integer=(-1, 1)),
    "near_forbidden": dict(lengths=[12, 40, 75, 99, 120], sd=3.0, forbid=0.2),
    # values past float32's range, above (overflow) or below (sums lost to
    # underflow): the log domain takes the whole bundle.  (Its float32 chart
    # values grow with the spread, and their rounding with them: measured up
    # to 7e-5 at sd 12, on this chart and on the one-width-a-step one.)
    "log_domain_6": dict(lengths=[6, 25, 26, 27, 27, 60, 110], sd=6.0),
    "log_domain_10": dict(lengths=[6, 25, 26, 27, 27, 60, 99], sd=10.0),
    # charts in the workspace beside bundles in LDS: one block past LDS, splits
    # past 8 bits, the rescales of long sentences
    "workspace": dict(lengths=[140, 143, 255, 256, 260, 30]),
    # few long sentences of which one has more than 450 words: teams take
    # those, tile charts behind theirs the ones of 140 and 141
    "teams_beside_tiles": dict(lengths=[460, 30, 141, 150, 140, 142, 12]),
    # too many long sentences for teams, and one of more than 450 words
    "workspace_many": dict(lengths=[150] * 16 + [460], sd=1.0),
    # scores of a trained model: one tree's spans far above the rest
    "planted": dict(lengths=[8, 25, 26, 50, 99, 130], sd=1.0, plant=9.0),
}


def make(lengths, seed=0, sd=2.0, n1=None, integer=None, forbid=0.0, plant=0.0):
    b = W.custom(lengths, seed=seed, sd=sd, n1=n1, integer=integer, forbid=forbid)
    if plant:
        rng = np.random.default_rng(seed + 1)
        for k, n in enumerate(b.lengths):
            todo = [(0, int(n))]
            while todo:
                i, j = todo.pop()
                b.scores[k, i, j] += np.float32(plant)
                if j - i >= 2:
                    m = int(rng.integers(i + 1, j))
                    todo += [(i, m), (m, j)]
    return b


@pytest.mark.parametrize("name,flags", [(n, 0) for n in sorted(CASES)] + [
    (n, B.CRF_FORCE_SPILL) for n in ("block_edges", "rescale_and_half_cu", "ties", "near_forbidden", "log_domain_6",
                                     "planted")])
def test_tile_charts(name, flags):
    import torch

    b = make(seed=60 + len(name), **CASES[name])
    dev = torch.device("cuda", 0)
    s = torch.from_numpy(b.scores).to(dev)
    rng = np.random.default_rng(5)
    grad = rng.standard_normal(b.B).astype(np.float32)
    g = torch.from_numpy(grad).to(dev)
    lz_ref, mu_ref = orc.marginals(b.scores, b.lengths, grad=grad, threads=16)
    sp_ref, be_ref = orc.cky(b.scores, b.lengths, threads=16)
    valid = W.valid_mask(b.lengths, b.n1)
    with B.Plan(b.lengths, n1=b.n1, flags=flags, device=dev) as plan:
        mu = torch.full_like(s, 7.5)
        lz, mu, sp, be = plan.parse(s, grad_logZ=g, marginals=mu)
        lzf = plan.inside_fwd(s)
        _, mu2 = plan.inside_fwd_bwd(s, grad_logZ=g, marginals=torch.full_like(s, 7.5))
        sp2, be2 = plan.cky_decode(s)
        loss, gs = plan.gold_loss(s, sp, grad_loss=g, grad_scores=torch.full_like(s, 7.5))
        _, mum, spm, _ = plan.mbr_decode(s)
        torch.cuda.synchronize()
    tol = 1e-5 * np.maximum(1.0, np.abs(lz_ref))
    for x in (lz, lzf):
        assert np.all(np.abs(x.cpu().numpy() - lz_ref) <= tol)
    scale = np.maximum(1.0, np.abs(grad))[:, None, None]
    for x in (mu, mu2):
        x = x.cpu().numpy()
        assert np.all(x[~valid] == 7.5), "cells that are no span keep the caller's values"
        assert np.max((np.abs(x - mu_ref) / scale)[valid]) <= 1e-4
    for x, y in ((sp, be), (sp2, be2)):
        assert np.array_equal(x.cpu().numpy(), sp_ref) and np.array_equal(y.cpu().numpy(), be_ref.astype(np.float32))
    # the loss of the best tree and its gradient
    ls_ref, gr_ref = orc.loss(b.scores, b.lengths, sp_ref, grad=grad)
    assert np.all(np.abs(loss.cpu().numpy() - ls_ref) <= 2e-5 * np.maximum(1.0, np.abs(lz_ref)))
    gs = gs.cpu().numpy()
    assert np.all(gs[~valid] == 7.5) and np.max((np.abs(gs - gr_ref) / scale)[valid]) <= 1e-4
    # MBR: the tree of the marginals that the call returned
    mum = np.where(valid, mum.cpu().numpy(), np.float32(np.nan))
    assert np.array_equal(spm.cpu().numpy(), orc.cky(mum, b.lengths, threads=16)[0])


def test_log_domain_shift_near_forbidden():
    # the log domain's shift comes from spans of a quarter of the sentence's
    # width, of which those with a near-forbidden score must be left out
    # however wide they are.  Chart values then reach some 2^9 (log2 units),
    # and a marginal's exponent takes about ten roundings of them:
    # 10 * 2^-15 * ln 2 (1e-3 off with those spans in the mean).
    import torch

    b = W.custom([350, 300, 350], seed=400, sd=5.0, forbid=0.05)
    s = torch.from_numpy(b.scores).to("cuda:0")
    lz_ref, mu_ref = orc.marginals(b.scores, b.lengths, threads=16)
    with B.Plan(b.lengths, n1=b.n1, device=s.device) as plan:
        lz, mu = plan.inside_fwd_bwd(s)
        torch.cuda.synchronize()
    assert np.all(np.abs(lz.cpu().numpy() - lz_ref) <= 1e-5 * np.abs(lz_ref))
    valid = W.valid_mask(b.lengths, b.n1)
    assert np.max(np.abs(mu.cpu().numpy() - mu_ref)[valid]) <= 2.1e-4


def test_log_domain_rounds_a_sum_once():
    # a span's log-sum-exp is rounded at the chart's magnitude once, not once
    # per product of tiles and lane: 2-norm of the marginals' error 7.4e-6 of
    # their own (9.6e-6 with a log2 per product, 9.8e-6 on charts that take a
    # width a step; same inputs, same arithmetic, same bits every time)
    import torch

    b = W.custom([60] * 40, seed=140, sd=8.0)
    s = torch.from_numpy(b.scores).to("cuda:0")
    _, mu_ref = orc.marginals(b.scores, b.lengths, threads=16)
    with B.Plan(b.lengths, n1=b.n1, device=s.device) as plan:
        _, mu = plan.inside_fwd_bwd(s)
        torch.cuda.synchronize()
    valid = W.valid_mask(b.lengths, b.n1)
    err = (mu.cpu().numpy() - mu_ref)[valid]
    assert np.linalg.norm(err) <= 8.5e-6 * np.linalg.norm(mu_ref[valid])


@pytest.mark.parametrize("length,count,sd,seed", [(30, 60, 8.0, 110)])
def test_sums_lost_to_underflow(length, count, sd, seed):
    # sums that underflow on few spans, none of them on an inside tile's
    # diagonal: without the outside sums the bundle of one sentence here keeps
    # the linear domain, 8e-2 off
    import torch

    b = W.custom([length] * count, seed=seed, sd=sd)
    s = torch.from_numpy(b.scores).to("cuda:0")
    lz_ref, mu_ref = orc.marginals(b.scores, b.lengths, threads=16)
    with B.Plan(b.lengths, n1=b.n1, device=s.device) as plan:
        lz, mu = plan.inside_fwd_bwd(s)
        torch.cuda.synchronize()
    assert np.all(np.abs(lz.cpu().numpy() - lz_ref) <= 1e-5 * np.maximum(1.0, np.abs(lz_ref)))
    valid = W.valid_mask(b.lengths, b.n1)
    assert np.max(np.abs(mu.cpu().numpy() - mu_ref)[valid]) <= 1e-4


@pytest.mark.parametrize("length,sd,tol", [(20, 5.0, 8e-7), (30, 4.0, 8e-7), (40, 3.0, 7.3e-7), (40, 5.0, 1.2e-6)])
def test_short_sentences_of_wide_spread_stay_linear(length, sd, tol):
    # 16 to 43 words whose scores spread further than the seed of the shift
    # allows for are rescaled, not sent to the log domain: 2-norm of the
    # marginals' error relative to their own 4.5e-7 to 7.1e-7 (in the log
    # domain 7.8e-7 to 2.4e-6)
    import torch

    b = W.custom([length] * (2000 // length - 10), seed=length + int(10 * sd), sd=sd)
    s = torch.from_numpy(b.scores).to("cuda:0")
    _, mu_ref = orc.marginals(b.scores, b.lengths, threads=16)
    with B.Plan(b.lengths, n1=b.n1, device=s.device) as plan:
        _, mu = plan.inside_fwd_bwd(s)
        torch.cuda.synchronize()
    valid = W.valid_mask(b.lengths, b.n1)
    err = (mu.cpu().numpy() - mu_ref)[valid]
    assert np.linalg.norm(err) <= tol * np.linalg.norm(mu_ref[valid])


@pytest.mark.parametrize("length", [10, 20, 30, 40])
def test_marginals_of_short_sentences_keep_float32s_digits(length):
    # marginals are products of the chart's own values: 2-norm of the error
    # 0.7 to 1.1e-7 of their own at deviation 2, a few float32 roundings (1.9
    # to 3.6e-7 through the values' logarithms)
    import torch

    b = W.custom([length] * (2000 // length), seed=length + 20, sd=2.0)
    s = torch.from_numpy(b.scores).to("cuda:0")
    _, mu_ref = orc.marginals(b.scores, b.lengths, threads=16)
    with B.Plan(b.lengths, n1=b.n1, device=s.device) as plan:
        _, mu = plan.inside_fwd_bwd(s)
        torch.cuda.synchronize()
    valid = W.valid_mask(b.lengths, b.n1)
    err = (mu.cpu().numpy() - mu_ref)[valid]
    assert np.linalg.norm(err) <= 1.5e-7 * np.linalg.norm(mu_ref[valid])


@pytest.mark.parametrize("length,count,sd,forbid,seed,tol", [(200, 24, 4.0, 0.0, 1, 1.5e-6), (300, 8, 3.0, 0.05, 4, 1.7e-6)])
def test_low_sums_that_do_not_matter_stay_linear(length, count, sd, forbid, seed, tol):
    # sums below 2^-100 beside values far above 1, but not of the same span:
    # no redo in the log domain, whose rounding would show (2-norm of the
    # marginals' error 1.0e-6 and 1.4e-6 of their own; 3.0e-6 and 2.2e-6 after
    # one)
    import torch

    b = W.custom([length] * count, seed=seed, sd=sd, forbid=forbid)
    s = torch.from_numpy(b.scores).to("cuda:0")
    _, mu_ref = orc.marginals(b.scores, b.lengths, threads=16)
    with B.Plan(b.lengths, n1=b.n1, device=s.device) as plan:
        _, mu = plan.inside_fwd_bwd(s)
        torch.cuda.synchronize()
    valid = W.valid_mask(b.lengths, b.n1)
    err = (mu.cpu().numpy() - mu_ref)[valid]
    assert np.linalg.norm(err) <= tol * np.linalg.norm(mu_ref[valid])
