"""The fused feature + forest kernel at the edges of its block shapes: one flow, a tile with a flow too many or too
few, the batch sizes where the shape changes, one window and two, windows up to 8 packets and up to 16, few trees,
two-byte vote counters, packet arrays off the alignment of the wide loads, times with their sign bit set.
Predictions, scores and the kept feature rows bit for bit against the oracle; rows that are not kept untouched."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CU = 256                                  # compute units of the device
FEW, MANY = 24 * CU, 3 * 128 * CU         # where the shape changes
SENTINEL = -777.0


def _packets(rng, n, longest, negative, shift):
    lens = rng.integers(0, longest + 1, size=n) if longest < 16 else np.where(rng.random(n) < 0.5, 16, rng.integers(0, longest + 1, size=n))
    off = np.zeros(n + 1, np.uint32)
    off[1:] = np.cumsum(lens)
    off += np.uint32(shift)                # (the first packets of the arrays belong to no flow)
    m = int(off[-1])
    iat = np.exp(rng.normal(-6, 2, size=m)).astype(np.float32)
    if negative:
        iat[rng.random(m) < 0.01] *= -1
    return SimpleNamespace(n_flows=n, flow_off=off, pkt_size=rng.integers(40, 1501, size=m, dtype=np.uint16), pkt_iat=iat,
                           pkt_dir=rng.integers(0, 2, size=m, dtype=np.uint8), pkt_hdr=None)


@pytest.mark.parametrize("n,depths,longest,T,d,C,negative,shift,skew", [
    (1, (8, 16), 20, 100, 4, 10, False, 0, 0), (17, (5,), 7, 33, 5, 4, True, 1, 0), (97, (3, 16), 64, 100, 6, 10, False, 0, 1),
    (FEW, (8, 16), 20, 50, 4, 10, False, 1, 0), (FEW + 1, (8, 16), 20, 50, 4, 10, True, 0, 0), (FEW + 65, (8,), 9, 48, 3, 33, False, 0, 1),
    (FEW + 129, (1, 9), 12, 300, 3, 10, False, 0, 0), (FEW + 130, (2, 16), 18, 47, 7, 7, True, 0, 0), (FEW + 1, (7,), 9, 5, 4, 2, False, 0, 0),
    (MANY, (8, 16), 16, 100, 8, 10, False, 0, 0), (MANY + 127, (6, 12), 14, 60, 8, 10, True, 3, 0), (MANY + 1, (4,), 8, 64, 8, 3, False, 0, 0)])
def test_tiles(n, depths, longest, T, d, C, negative, shift, skew):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + 31 * T + d)
    pk = _packets(rng, n, longest, negative, shift)
    feat, _ = oracle.featurize(pk.flow_off, pk.pkt_size, pk.pkt_iat, pk.pkt_dir, depths, n_threads=8)
    F = 32 * len(depths)
    n_int = (1 << d) - 1
    nf = rng.integers(0, F, size=(T, n_int), dtype=np.uint16)
    nt = feat[rng.integers(0, min(n, 4096), size=(T, n_int)), nf.astype(np.int64)].astype(np.float32)
    m = SimpleNamespace(n_trees=T, depth=d, n_classes=C, n_features=F, node_feat=nf, node_thr=np.ascontiguousarray(nt),
                        leaf_label=rng.integers(0, C, size=(T, 1 << d), dtype=np.uint8))
    _, pred, top, _ = oracle.fast_infer(feat, m, want_votes=False, n_threads=8)
    vmin = rng.integers(int(np.median(top)), int(top.max()) + 2, size=C).astype(int).tolist()
    dev = "cuda:0"
    d_pk = sf.packets_to_device(pk, dev)
    if skew:                               # arrays one element off the alignment of the wide loads
        off_by = lambda t: torch.cat([t[:1], t])[1:]
        d_pk = sf.DevicePackets(d_pk.flow_off, off_by(d_pk.pkt_size), off_by(d_pk.pkt_iat), off_by(d_pk.pkt_dir))
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, T, d))
    ld = F + (0 if n % 2 else 3)           # rows on and off the 16-byte grid
    g_feat = torch.full((n, ld), SENTINEL, dtype=torch.float32, device=dev)
    g_pred, g_top, g_lab = (torch.full((n,), -1, dtype=torch.int16, device=dev) for _ in range(3))
    ctx.sf_featurize_fast_infer(d_pk, list(depths), sf.forest_to_device(m, dev), vmin, g_feat, g_pred, g_top, labels=g_lab)
    torch.cuda.synchronize()
    u16 = lambda t: t.cpu().numpy().view(np.uint16)
    assert np.array_equal(u16(g_pred), pred) and np.array_equal(u16(g_top), top) and np.array_equal(u16(g_lab), pred)
    keep = top < np.asarray(vmin)[pred]
    got = g_feat.cpu().numpy()
    assert np.array_equal(got[keep][:, :F].view(np.uint32), feat[keep].view(np.uint32))
    assert np.all(got[~keep] == SENTINEL) and np.all(got[:, F:] == SENTINEL)
