"""Which calls of the fused entry points leave feature rows unwritten is part of the interface: the forest decides, not
the batch.  Models on both sides of each edge of the rule (vote counters of one and of two bytes, number of trees, depth):
where the steps are fused only the rows of flows under the gate are written, elsewhere every row is, and the call is
refused without a feature matrix.  Rows bit for bit against the oracle."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SENTINEL = -777.0


@pytest.mark.parametrize("depths,T,d,C,fused", [
    ((8, 16), 255, 4, 32, True), ((8, 16), 256, 4, 32, False), ((8, 16), 256, 1, 32, True), ((8, 16), 300, 3, 33, False),
    ((8, 16), 60, 4, 64, False), ((8, 16), 32, 4, 60, True), ((8, 16), 33, 4, 60, False), ((5, 10), 2, 12, 64, False), ((5, 10), 2, 1, 64, True),
    ((8, 16), 672, 4, 10, True), ((8, 16), 673, 4, 10, False), ((8, 16), 704, 2, 10, True), ((8, 16), 705, 2, 10, False),
    ((8, 16), 5760, 2, 10, False), ((8, 16), 5761, 2, 10, True), ((16,), 2752, 4, 10, True), ((16,), 2753, 4, 10, False),
    ((8, 17), 10, 4, 4, False), ((4, 8, 16), 10, 4, 4, False)])
def test_rows(depths, T, d, C, fused):
    import torch
    import paper_2402_03694_amd as sf
    n = 130 if T > 500 else 6500
    rng = np.random.default_rng(n + 31 * T + d)
    off = np.zeros(n + 1, np.uint32)
    off[1:] = np.cumsum(rng.integers(0, 20, size=n))
    m = int(off[-1])
    pk = SimpleNamespace(n_flows=n, flow_off=off, pkt_size=rng.integers(40, 1501, size=m, dtype=np.uint16),
                         pkt_iat=np.exp(rng.normal(-6, 2, size=m)).astype(np.float32), pkt_dir=rng.integers(0, 2, size=m, dtype=np.uint8), pkt_hdr=None)
    feat, _ = oracle.featurize(pk.flow_off, pk.pkt_size, pk.pkt_iat, pk.pkt_dir, depths, n_threads=8)
    F, n_int = 32 * len(depths), (1 << d) - 1
    nf = rng.integers(0, F, size=(T, n_int), dtype=np.uint16)
    nt = feat[rng.integers(0, n, size=(T, n_int)), nf.astype(np.int64)].astype(np.float32)
    model = SimpleNamespace(n_trees=T, depth=d, n_classes=C, n_features=F, node_feat=nf, node_thr=np.ascontiguousarray(nt),
                            leaf_label=rng.integers(0, C, size=(T, 1 << d), dtype=np.uint8))
    _, pred, top, _ = oracle.fast_infer(feat, model, want_votes=False, n_threads=8)
    vmin = int(np.median(top)) + 1
    dev = "cuda:0"
    d_pk, forest = sf.packets_to_device(pk, dev), sf.forest_to_device(model, dev)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    got = torch.full((n, F), SENTINEL, dtype=torch.float32, device=dev)
    g_pred, g_top, g_lab = (torch.full((n,), -1, dtype=torch.int16, device=dev) for _ in range(3))
    ctx.sf_featurize_fast_infer(d_pk, list(depths), forest, vmin, got, g_pred, g_top, labels=g_lab)
    torch.cuda.synchronize()
    u16 = lambda t: t.cpu().numpy().view(np.uint16)
    assert np.array_equal(u16(g_pred), pred) and np.array_equal(u16(g_top), top) and np.array_equal(u16(g_lab), pred)
    written = top < vmin if fused else np.ones(n, bool)
    got = got.cpu().numpy()
    assert np.array_equal(got[written].view(np.uint32), feat[written].view(np.uint32))
    assert np.all(got[~written] == SENTINEL)
    if fused:
        ctx.sf_featurize_fast_infer(d_pk, list(depths), forest, vmin, None, g_pred, g_top)
    else:
        with pytest.raises(sf.ServeFlowError):
            ctx.sf_featurize_fast_infer(d_pk, list(depths), forest, vmin, None, g_pred, g_top)
    torch.cuda.synchronize()
    assert np.array_equal(u16(g_pred), pred) and np.array_equal(u16(g_top), top)
