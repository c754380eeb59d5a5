"""The tree walk with a wave to a tree (which calls take it is decided in fast_infer.hip): every block shape and window, both
sides of the lines, tiles with one flow too many, every kind of last round, trees of one to three levels and of odd
depth, fewer trees than waves, classes the trees do not divide by, more classes than features, lists.  Votes, predictions, scores and kept
rows, and binary32 margins, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_few_trees import _model, _u16
from test_gpu_fused_tiles import test_tiles as _fused_tiles

pytestmark = pytest.mark.gpu

CU = 256                                  # compute units of the device


def _feat(rng, n, ld):
    x = rng.normal(0, 1, size=(n, ld)).astype(np.float32)
    x[:, ::3] = np.round(x[:, ::3] * 4)   # repeated values: splits that hit a threshold exactly
    x[rng.integers(0, n, 50), rng.integers(0, ld, 50)] = rng.choice(np.array([np.nan, np.inf, -np.inf], np.float32), 50)
    return x


SHAPES = [(24 * CU, 64, 100, 7, 10, 0), (24 * CU + 1, 64, 48, 7, 10, 0), (24 * CU + 65, 20, 97, 6, 33, 1), (64 * CU, 33, 63, 9, 4, 0),  # 64 flows a block
          (64 * CU + 1, 64, 49, 7, 10, 0), (64 * CU + 127, 96, 101, 9, 7, 0), (128 * CU, 64, 96, 8, 3, 0), (128 * CU + 1, 64, 96, 8, 3, 0),
          (192 * CU - 1, 64, 50, 10, 10, 0), (192 * CU, 64, 50, 10, 10, 4), (256 * CU, 32, 53, 12, 10, 0), (320 * CU, 64, 48, 13, 2, 0),
          (64 * CU + 2, 128, 300, 10, 32, 0), (64 * CU + 129, 127, 64, 7, 10, 2), (64 * CU + 3, 64, 95, 8, 10, 0), (64 * CU + 3, 70, 51, 5, 64, 2),
          (1200 * CU - 1, 32, 49, 11, 10, 0), (1200 * CU + 1, 32, 51, 12, 10, 0), (1200 * CU + 255, 64, 97, 8, 5, 0), (1200 * CU, 64, 52, 5, 10, 0),
          ] + [(64 * CU + 40 + d, 64, 192 + d, d, 10, 0) for d in (1, 2, 3, 4)] + [(64 * CU + T, 40, T, 7, 10, 0) for T in (55, 56, 57, 62)] + [
              # the lines of the models that gain little
              (1200 * CU + 40, 64, 193, 1, 10, 0), (1200 * CU - 1, 64, 193, 1, 10, 0), (1200 * CU, 65, 193, 1, 10, 0), (256 * CU, 65, 200, 2, 10, 0), (320 * CU, 65, 399, 2, 10, 0),
              (320 * CU + 1, 65, 400, 2, 10, 0), (384 * CU + 1, 64, 193, 4, 10, 0), (384 * CU, 64, 193, 4, 10, 0), (432 * CU, 64, 193, 4, 10, 0), (384 * CU + 1, 97, 49, 7, 10, 0),
              (432 * CU, 113, 63, 7, 10, 0), (432 * CU, 113, 64, 7, 10, 0), (384 * CU, 113, 63, 10, 10, 0), (384 * CU + 1, 113, 95, 9, 10, 0), (384 * CU + 1, 96, 127, 8, 10, 0)]


@pytest.mark.parametrize("n,F,T,d,C,pad", SHAPES)
def test_votes(n, F, T, d, C, pad):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + 7 * T + d)
    feat = _feat(rng, n, F + pad)
    m = _model(rng, T, d, C, F, np.nan_to_num(feat[:4096, :F]))
    votes, pred, top, _ = oracle.fast_infer(np.ascontiguousarray(feat[:, :F]), m, n_threads=8)
    dev = "cuda:0"
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    g = lambda *s: torch.full(s, -1, dtype=torch.int16, device=dev)
    g_pred, g_top, g_votes = g(n), g(n), g(n, C)
    d_feat, d_m = torch.from_numpy(feat).to(dev), sf.forest_to_device(m, dev)
    ctx.sf_fast_infer(d_feat, d_m, g_pred, g_top, votes=g_votes)
    torch.cuda.synchronize()
    assert np.array_equal(_u16(g_pred), pred) and np.array_equal(_u16(g_top), top) and np.array_equal(_u16(g_votes), votes)
    # the same rows from a list that is shorter than its capacity
    take = np.sort(rng.permutation(n)[:n - n // 3]).astype(np.uint32)
    idx = np.full(n, 0xFFFFFFFF, np.uint32)
    idx[:take.size] = take
    s_pred, s_top, lab = g(n), g(n), g(n)
    ctx.sf_fast_infer_subset(d_feat, torch.from_numpy(idx.view(np.int32)).to(dev), torch.tensor([take.size], dtype=torch.int32, device=dev), d_m,
                             s_pred, s_top, labels=lab)
    torch.cuda.synchronize()
    assert np.array_equal(_u16(s_pred)[:take.size], pred[take]) and np.array_equal(_u16(s_top)[:take.size], top[take])
    assert np.all(_u16(s_pred)[take.size:] == 0xFFFF)
    want = np.full(n, 0xFFFF, np.uint16)
    want[take] = pred[take]
    assert np.array_equal(_u16(lab), want)


@pytest.mark.parametrize("n,F,T,d,C", [(70 * CU, 64, 52, 9, 10), (320 * CU, 33, 97, 7, 40), (1200 * CU, 32, 51, 10, 10), (1200 * CU + 3, 30, 300, 5, 7)])
def test_short_lists(n, F, T, d, C):
    """Lists far shorter than their capacity, whose blocks then take 64 flows each: around that line, one row, tiles of one flow, none."""
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + T)
    feat = _feat(rng, n, F)
    m = _model(rng, T, d, C, F, np.nan_to_num(feat[:4096]))
    _, pred, top, _ = oracle.fast_infer(feat, m, n_threads=8)
    dev = "cuda:0"
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    d_feat, d_m = torch.from_numpy(feat).to(dev), sf.forest_to_device(m, dev)
    for rows in (0, 1, 63, 65, 8 * CU, 24 * CU + 1, n // 4, n // 4 + 1, 64 * CU, 64 * CU + 1, 128 * CU, 128 * CU + 1):
        rows = min(rows, n)
        take = np.sort(rng.permutation(n)[:rows]).astype(np.uint32)
        idx = np.full(n, 0xFFFFFFFF, np.uint32)
        idx[:rows] = take
        g_pred, g_top, lab = (torch.full((n,), -1, dtype=torch.int16, device=dev) for _ in range(3))
        ctx.sf_fast_infer_subset(d_feat, torch.from_numpy(idx.view(np.int32)).to(dev), torch.tensor([rows], dtype=torch.int32, device=dev), d_m, g_pred, g_top, labels=lab)
        torch.cuda.synchronize()
        assert np.array_equal(_u16(g_pred)[:rows], pred[take]) and np.array_equal(_u16(g_top)[:rows], top[take]), rows
        assert np.all(_u16(g_pred)[rows:] == 0xFFFF) and np.all(_u16(g_top)[rows:] == 0xFFFF), rows
        want = np.full(n, 0xFFFF, np.uint16)
        want[take] = pred[take]
        assert np.array_equal(_u16(lab), want), rows


@pytest.mark.parametrize("n,F,T,d,leaves", [
    (1700 * CU - 1, 32, 64, 13, True), (1700 * CU, 32, 64, 13, True), (1700 * CU + 255, 64, 65, 13, True), (1700 * CU + 1, 20, 63, 13, True), (1700 * CU + 1, 33, 64, 14, True),
    (3000 * CU - 1, 96, 49, 8, False), (3000 * CU, 96, 49, 8, False), (3000 * CU + 1, 64, 81, 8, False), (3000 * CU + 127, 96, 50, 6, False), (3000 * CU + 129, 127, 130, 4, False),
    (2000 * CU - 1, 64, 60, 10, True), (2000 * CU, 64, 60, 10, True), (2000 * CU + 127, 95, 48, 7, True)])
def test_large_batches_outside(n, F, T, d, leaves):
    """What that form does not take in large batches: leaf numbers, a medium number of shallow trees (128 x 8, and one lane per flow for deep
    trees with leaf numbers), at the lines and with a last tile of one flow."""
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + T)
    feat = _feat(rng, n, F)
    m = _model(rng, T, d, 10, F, np.nan_to_num(feat[:4096]))
    votes, pred, top, leaf = oracle.fast_infer(feat, m, want_leaves=leaves, n_threads=8)
    dev = "cuda:0"
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    g = lambda *s: torch.full(s, -1, dtype=torch.int16, device=dev)
    g_pred, g_top, g_votes, g_leaf = g(n), g(n), g(n, 10), g(n, T) if leaves else None
    ctx.sf_fast_infer(torch.from_numpy(feat).to(dev), sf.forest_to_device(m, dev), g_pred, g_top, votes=g_votes, leaf_idx=g_leaf)
    torch.cuda.synchronize()
    assert np.array_equal(_u16(g_pred), pred) and np.array_equal(_u16(g_top), top) and np.array_equal(_u16(g_votes), votes)
    if leaves:
        assert np.array_equal(_u16(g_leaf), leaf)


@pytest.mark.parametrize("n,F,T,d,C", [
    (24 * CU + 1, 32, 60, 6, 6), (24 * CU + 63, 64, 51, 8, 16), (24 * CU + 1, 64, 30, 5, 17), (128 * CU - 1, 96, 25, 7, 5), (128 * CU, 64, 61, 8, 10),
    (128 * CU + 129, 96, 33, 9, 6), (128 * CU + 1, 10, 70, 3, 16), (128 * CU + 2, 64, 4, 8, 7), (320 * CU + 5, 64, 41, 8, 10), (320 * CU + 255, 64, 48, 5, 16),
    (320 * CU, 32, 36, 13, 9), (320 * CU + 1, 4, 40, 1, 12), (320 * CU, 64, 35, 2, 8), (384 * CU, 64, 14, 8, 3), (384 * CU - 1, 64, 14, 8, 3), (384 * CU + 1, 32, 21, 9, 4),
    (384 * CU, 96, 12, 8, 4), (128 * CU, 128, 24, 6, 8), (128 * CU - 1, 128, 24, 6, 8), (192 * CU + 1, 128, 18, 6, 6), (192 * CU + 1, 112, 24, 6, 8)])
@pytest.mark.parametrize("based", [True, False])
def test_margins(n, F, T, d, C, based):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + 5 * T + d)
    feat = _feat(rng, n, F)
    m = _model(rng, T, d, C, F, np.nan_to_num(feat[:4096]))
    m.leaf_value = rng.normal(0, 0.5, size=(T, 1 << d)).astype(np.float32)
    m.base = rng.uniform(-0.5, 0.5, size=C).astype(np.float32) if based else None
    want, pred, lc, _ = oracle.gbdt_infer(feat, m, n_threads=8)
    dev = "cuda:0"
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    margins = torch.full((n, C), float("nan"), dtype=torch.float32, device=dev)
    g_pred = torch.full((n,), -1, dtype=torch.int16, device=dev)
    score = torch.full((n,), float("nan"), dtype=torch.float32, device=dev)
    ctx.sf_gbdt_infer(torch.from_numpy(feat).to(dev), sf.gbdt_to_device(m, dev), sf.SF_SCORE_LC, g_pred, score, margins=margins)
    torch.cuda.synchronize()
    assert np.array_equal(margins.cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert np.array_equal(_u16(g_pred), pred)
    # the two binary64 exponentials agree to 1e-13; rounding to binary32 adds half a unit
    assert np.all(np.abs(score.cpu().numpy() - lc) <= 0.5 * np.spacing(np.abs(lc).astype(np.float32)) + 1e-13)


@pytest.mark.parametrize("n,F,T,d", [(3000 * CU - 1, 32, 75, 5), (3000 * CU, 32, 75, 5), (3000 * CU + 1, 17, 80, 6), (3000 * CU + 255, 32, 74, 4)])
def test_five_classes_leaf_numbers(n, F, T, d):
    """Leaf numbers of boosted models with five classes: margins, scores' classes and leaf numbers on both sides of the lines."""
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + T)
    feat = _feat(rng, n, F)
    m = _model(rng, T, d, 5, F, np.nan_to_num(feat[:4096]))
    m.leaf_value = rng.normal(0, 0.5, size=(T, 1 << d)).astype(np.float32)
    m.base = rng.uniform(-0.5, 0.5, size=5).astype(np.float32)
    want, pred, _, _ = oracle.gbdt_infer(feat, m, n_threads=8)
    leaf = oracle.fast_infer(feat, m, want_leaves=True, n_threads=8)[3]
    dev = "cuda:0"
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    margins = torch.full((n, 5), float("nan"), dtype=torch.float32, device=dev)
    g_pred, g_leaf = torch.full((n,), -1, dtype=torch.int16, device=dev), torch.full((n, T), -1, dtype=torch.int16, device=dev)
    ctx.sf_gbdt_infer(torch.from_numpy(feat).to(dev), sf.gbdt_to_device(m, dev), sf.SF_SCORE_LC, g_pred, torch.empty(n, device=dev), margins=margins, leaf_idx=g_leaf)
    torch.cuda.synchronize()
    assert np.array_equal(margins.cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert np.array_equal(_u16(g_pred), pred) and np.array_equal(_u16(g_leaf), leaf)


@pytest.mark.parametrize("n,depths,longest,T,d,C,negative,shift,skew", [
    (64 * CU, (8, 16), 20, 50, 7, 10, False, 1, 0), (64 * CU + 1, (8, 16), 20, 50, 7, 10, True, 0, 0), (64 * CU + 127, (8,), 9, 48, 9, 33, False, 0, 1),
    (128 * CU, (1, 9), 12, 300, 5, 10, False, 0, 0), (128 * CU + 1, (2, 16), 18, 97, 8, 7, False, 0, 0), (192 * CU + 130, (6, 12), 14, 61, 10, 10, True, 3, 0),
    (64 * CU + 2, (5,), 7, 197, 2, 4, False, 0, 1), (320 * CU + 1, (16,), 16, 49, 11, 2, False, 0, 0), (64 * CU + 3, (5, 8), 9, 192, 5, 10, False, 0, 0),
    (192 * CU, (5, 8), 9, 48, 5, 10, False, 0, 0), (320 * CU, (5, 8), 9, 191, 5, 10, False, 0, 0), (320 * CU, (5, 8), 9, 192, 5, 10, False, 0, 0), (64 * CU + 5, (8,), 8, 300, 3, 10, False, 0, 0), (64 * CU + 3, (3, 9), 9, 197, 3, 10, False, 0, 0), (320 * CU, (4, 8), 8, 64, 9, 10, True, 0, 0),
    (320 * CU, (4, 8), 8, 63, 10, 10, False, 0, 0), (64 * CU + 4, (4, 8), 8, 48, 11, 10, False, 0, 0), (432 * CU, (8, 16), 16, 97, 6, 10, False, 0, 0), (432 * CU - 1, (8, 16), 16, 192, 6, 10, False, 0, 0), (3000 * CU + 1, (2, 9), 9, 256, 4, 10, False, 0, 0)])
def test_fused(n, depths, longest, T, d, C, negative, shift, skew):
    _fused_tiles(n, depths, longest, T, d, C, negative, shift, skew)
