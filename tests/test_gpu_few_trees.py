"""Forests of few trees, and of trees too deep for the caches, in batches large enough for one lane per flow: the walk alone and
the fused feature + forest kernel on both sides of the lines in fast_infer.hip, with a last block that is nearly empty; and
every length of a last round of trees where several lanes share a flow.  Votes, predictions, leaf numbers, scores and kept rows
bit for bit against the oracle."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CU = 256                                  # compute units of the device
SENTINEL = -777.0


def _model(rng, T, d, C, F, feat):
    n_int, n_leaf = (1 << d) - 1, 1 << d
    nf = rng.integers(0, F, size=(T, n_int), dtype=np.uint16)
    nt = feat[rng.integers(0, feat.shape[0], size=(T, n_int)), nf.astype(np.int64)].astype(np.float32)
    return SimpleNamespace(n_trees=T, depth=d, n_classes=C, n_features=F, node_feat=nf, node_thr=np.ascontiguousarray(nt),
                           leaf_label=rng.integers(0, C, size=(T, n_leaf), dtype=np.uint8))


def _u16(t):
    return t.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("n,F,T,d,C,pad", [
    (1400 * CU + 1, 32, 1, 8, 10, 0), (1400 * CU + 77, 32, 4, 9, 3, 0), (1400 * CU + 255, 29, 12, 7, 33, 0), (1400 * CU, 32, 47, 2, 10, 1),
    (1400 * CU - 1, 32, 3, 4, 10, 0), (1400 * CU + 3, 33, 3, 1, 2, 0), (384 * CU + 5, 64, 64, 13, 10, 0), (384 * CU, 20, 64, 14, 4, 3), (384 * CU - 1, 64, 64, 13, 10, 0), (750 * CU + 5, 32, 4, 7, 10, 0), (750 * CU - 1, 32, 4, 7, 10, 0),
    (384 * CU + 130, 128, 64, 13, 64, 0)] + [(24 * CU + 100 + T, 64, T, 5, 10, 0) for T in (2, 4, 6, 9, 12, 14, 16, 17, 20, 21, 25, 47)]
    + [(24 * CU + T, 64, T, 6, 10, 0) for T in (48, 56, 57, 64, 65, 72)] + [(384 * CU + T, 32, T, 6, 10, 0) for T in (64, 80, 81)])
def test_walk(n, F, T, d, C, pad):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + 7 * T + d)
    feat = rng.normal(0, 1, size=(n, F + pad)).astype(np.float32)
    feat[:, ::3] = np.round(feat[:, ::3] * 4)   # repeated values: splits that hit a threshold exactly
    m = _model(rng, T, d, C, F, feat[:4096, :F])
    want_leaf = n * T <= 2_000_000
    votes, pred, top, leaf = oracle.fast_infer(np.ascontiguousarray(feat[:, :F]), m, want_leaves=want_leaf, n_threads=8)
    dev = "cuda:0"
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    g = lambda *s: torch.full(s, -1, dtype=torch.int16, device=dev)
    g_pred, g_top, g_votes, g_leaf = g(n), g(n), g(n, C), (g(n, T) if want_leaf else None)
    ctx.sf_fast_infer(torch.from_numpy(feat).to(dev), sf.forest_to_device(m, dev), g_pred, g_top, votes=g_votes, leaf_idx=g_leaf)
    torch.cuda.synchronize()
    assert np.array_equal(_u16(g_pred), pred) and np.array_equal(_u16(g_top), top) and np.array_equal(_u16(g_votes), votes)
    if want_leaf:
        assert np.array_equal(_u16(g_leaf), leaf)


ROUND2, ROUND3 = 512 * CU, 768 * CU       # flows in one round of blocks, with two windows and with one


@pytest.mark.parametrize("n,depths,longest,T,d,C,negative,shift,skew,pad", [
    (150 * CU, (8, 16), 20, 6, 5, 10, False, 0, 0, 0), (150 * CU - 1, (8, 16), 20, 6, 5, 10, False, 0, 0, 0), (150 * CU + 1, (5, 12), 14, 1, 12, 4, True, 1, 0, 3),
    (ROUND2 * 6 // 10 + 300, (1, 16), 16, 47, 3, 33, True, 0, 1, 0), (ROUND2 + 77, (8, 16), 16, 6, 4, 10, False, 0, 0, 1), (ROUND2 + 77, (8, 16), 16, 7, 4, 10, False, 0, 0, 0),
    (2 * ROUND2 - 5, (9, 16), 18, 64, 2, 10, False, 0, 0, 0), (ROUND2 * 8 // 10, (3, 7), 9, 6, 6, 10, True, 0, 1, 0), (ROUND2 * 8 // 10, (3, 7), 9, 7, 6, 10, False, 3, 0, 0),
    (150 * CU + 9, (16,), 16, 6, 8, 10, True, 0, 0, 0), (ROUND3 // 2 + 1, (9,), 30, 12, 4, 5, False, 1, 0, 2), (ROUND3 * 7 // 10, (16,), 16, 32, 3, 10, False, 0, 1, 0),
    (ROUND3 - 100, (12,), 16, 64, 3, 10, True, 0, 0, 0), (ROUND3 // 2 + 33, (8,), 8, 6, 5, 10, True, 0, 0, 0), (ROUND3 // 2 + 33, (1,), 3, 5, 13, 10, False, 2, 1, 1),
    (2 * ROUND3 + 77, (4,), 6, 50, 2, 10, True, 0, 0, 0), (2 * ROUND3 + 1, (8,), 9, 20, 7, 10, False, 0, 0, 0)])
def test_fused(n, depths, longest, T, d, C, negative, shift, skew, pad):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + 31 * T + d)
    full = rng.random(n) < 0.5
    lens = np.where(full, min(longest, 16), rng.integers(0, longest + 1, size=n))
    off = np.zeros(n + 1, np.uint32)
    off[1:] = np.cumsum(lens)
    off += np.uint32(shift)                # (the first packets of the arrays belong to no flow)
    m = int(off[-1])
    iat = np.exp(rng.normal(-6, 2, size=m)).astype(np.float32)
    if negative:                           # some waves with, most without
        iat[rng.integers(0, m, size=300)] *= -1
    pk = SimpleNamespace(n_flows=n, flow_off=off, pkt_size=rng.integers(0, 65536, size=m, dtype=np.uint16), pkt_iat=iat,
                         pkt_dir=rng.integers(0, 2, size=m, dtype=np.uint8), pkt_hdr=None)
    feat, _ = oracle.featurize(pk.flow_off, pk.pkt_size, pk.pkt_iat, pk.pkt_dir, depths, n_threads=8)
    F = 32 * len(depths)
    model = _model(rng, T, d, C, F, feat[:4096])
    _, pred, top, _ = oracle.fast_infer(feat, model, want_votes=False, n_threads=8)
    vmin = rng.integers(int(np.median(top)), int(top.max()) + 2, size=C).astype(int).tolist()
    dev = "cuda:0"
    d_pk = sf.packets_to_device(pk, dev)
    if skew:                               # arrays one element off the alignment of the wide loads
        off_by = lambda t: torch.cat([t[:1], t])[1:]
        d_pk = sf.DevicePackets(d_pk.flow_off, off_by(d_pk.pkt_size), off_by(d_pk.pkt_iat), off_by(d_pk.pkt_dir))
    forest = sf.forest_to_device(model, dev)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    got = torch.full((n, F + pad), SENTINEL, dtype=torch.float32, device=dev)
    g = lambda: torch.full((n,), -1, dtype=torch.int16, device=dev)
    g_pred, g_top, g_lab = g(), g(), g()
    ctx.sf_featurize_fast_infer(d_pk, list(depths), forest, vmin, got, g_pred, g_top, labels=g_lab)
    torch.cuda.synchronize()
    assert np.array_equal(_u16(g_pred), pred) and np.array_equal(_u16(g_top), top) and np.array_equal(_u16(g_lab), pred)
    keep = top < np.asarray(vmin)[pred]
    got = got.cpu().numpy()
    assert np.array_equal(got[keep][:, :F].view(np.uint32), feat[keep].view(np.uint32))
    assert np.all(got[~keep] == SENTINEL) and np.all(got[:, F:] == SENTINEL)
    g_pred, g_top = g(), g()               # no rows wanted
    ctx.sf_featurize_fast_infer(d_pk, list(depths), forest, vmin, None, g_pred, g_top)
    torch.cuda.synchronize()
    assert np.array_equal(_u16(g_pred), pred) and np.array_equal(_u16(g_top), top)


@pytest.mark.parametrize("n,F,T,d,C", [(384 * CU + 5, 32, 9, 5, 3), (384 * CU, 20, 31, 4, 3), (384 * CU + 3, 64, 9, 4, 3), (384 * CU + 200, 64, 13, 3, 1),
                                       (384 * CU + 1, 128, 4, 6, 1), (256 * CU + 7, 32, 41, 4, 2), (256 * CU - 1, 64, 41, 3, 2), (9000, 40, 12, 5, 1),
                                       (7000, 128, 66, 2, 33), (384 * CU + 9, 128, 64, 2, 64),
                                       (384 * CU + 11, 32, 23, 4, 5), (384 * CU + 11, 64, 23, 4, 5), (384 * CU - 1, 32, 11, 3, 5)])
def test_margins(n, F, T, d, C):
    """The boosted form on both sides of its lines; sums of binary32 margins in tree order, bit for bit."""
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + 5 * T + d)
    feat = rng.normal(0, 1, size=(n, F)).astype(np.float32)
    m = _model(rng, T, d, C, F, feat[:4096])
    m.leaf_value = rng.normal(0, 0.5, size=(T, 1 << d)).astype(np.float32)
    m.base = rng.uniform(-0.5, 0.5, size=C).astype(np.float32)
    want, pred, lc, _ = oracle.gbdt_infer(feat, m, n_threads=8)
    dev = "cuda:0"
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    margins = torch.full((n, C), float("nan"), dtype=torch.float32, device=dev)
    g_pred = torch.full((n,), -1, dtype=torch.int16, device=dev)
    score = torch.full((n,), float("nan"), dtype=torch.float32, device=dev)
    ctx.sf_gbdt_infer(torch.from_numpy(feat).to(dev), sf.gbdt_to_device(m, dev), sf.SF_SCORE_LC, g_pred, score, margins=margins)
    torch.cuda.synchronize()
    assert np.array_equal(margins.cpu().numpy().view(np.uint32), want.view(np.uint32)) and np.array_equal(_u16(g_pred), pred)
    # the two binary64 exponentials agree to 1e-13; rounding to binary32 adds half a unit
    assert np.all(np.abs(score.cpu().numpy() - lc) <= 0.5 * np.spacing(np.abs(lc).astype(np.float32)) + 1e-13)


def _median_us(call):
    import torch
    times = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    return sorted(times)[4]


def test_walk_rate():
    """Four shallow trees on a million rows of 32 features take at most 1.13 of the time of copying the rows (0.95; with one
    request at a time in flight 1.31)."""
    import torch
    import paper_2402_03694_amd as sf
    n, dev = 1 << 20, "cuda:0"
    rng = np.random.default_rng(1)
    feat = torch.randn((n, 32), device=dev)
    model = sf.forest_to_device(_model(rng, 4, 3, 10, 32, feat[:4096].cpu().numpy()), dev)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 4, 3))
    ctx.sf_forest_pack(model)
    pred, top = (torch.empty(n, dtype=torch.int16, device=dev) for _ in range(2))
    copy = torch.empty_like(feat)
    assert _median_us(lambda: ctx.sf_fast_infer(feat, model, pred, top)) <= 1.13 * _median_us(lambda: copy.copy_(feat))


def test_fused_rate():
    """Features and five trees in one call take at most 1.32 of the time of the features alone (1.14; four lanes a flow 1.55)."""
    import torch
    import paper_2402_03694_amd as sf
    n, dev, depths = 1 << 20, "cuda:0", [8, 16]
    rng = np.random.default_rng(2)
    m = 16 * n
    pk = sf.DevicePackets(torch.arange(0, m + 1, 16, dtype=torch.int32, device=dev), torch.randint(40, 1500, (m,), dtype=torch.int16, device=dev),
                          torch.rand(m, device=dev), torch.randint(0, 2, (m,), dtype=torch.uint8, device=dev))
    feat = torch.empty((n, 64), device=dev)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 5, 4))
    ctx.sf_featurize(pk, depths, feat)
    model = sf.forest_to_device(_model(rng, 5, 4, 10, 64, feat[:4096].cpu().numpy()), dev)
    ctx.sf_forest_pack(model)
    pred, top = (torch.empty(n, dtype=torch.int16, device=dev) for _ in range(2))
    alone = _median_us(lambda: ctx.sf_featurize(pk, depths, feat))
    assert _median_us(lambda: ctx.sf_featurize_fast_infer(pk, depths, model, 1, feat, pred, top)) <= 1.32 * alone


def test_margins_rate():
    """Three classes, 150 trees of depth 6 on a million rows of 32 features take at most 8.9 of the time of copying the rows
    (7.9; with the general split of the classes among lanes 9.9)."""
    import torch
    import paper_2402_03694_amd as sf
    n, dev = 1 << 20, "cuda:0"
    rng = np.random.default_rng(3)
    feat = torch.randn((n, 32), device=dev)
    m = _model(rng, 150, 6, 3, 32, feat[:4096].cpu().numpy())
    m.leaf_value, m.base = rng.normal(0, 0.5, size=(150, 64)).astype(np.float32), np.zeros(3, np.float32)
    model = sf.gbdt_to_device(m, dev)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 150, 6))
    ctx.sf_gbdt_pack(model)
    pred, score = torch.empty(n, dtype=torch.int16, device=dev), torch.empty(n, device=dev)
    copy = torch.empty_like(feat)
    ratio = _median_us(lambda: ctx.sf_gbdt_infer(feat, model, sf.SF_SCORE_LC, pred, score)) / _median_us(lambda: copy.copy_(feat))
    assert ratio <= 8.9
