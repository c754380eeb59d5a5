"""The fused kernel on batches whose blocks are all resident at once, on both sides of the lines (256 compute units: one block of 128
flows a unit for a wave to a tree, three of 64 or 128 flows for lanes that share a flow): the same bits as the separate calls."""
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("keep", [True, False])
@pytest.mark.parametrize("n,trees,depth", [(16384, 100, 10), (16385, 100, 10), (32768, 100, 6), (32769, 100, 6), (49152, 60, 2), (49153, 60, 2),
                                           (5003, 20, 9), (98304, 20, 9), (98305, 20, 9)])
def test_fused_few(n, trees, depth, keep):
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(n + trees)
    lens = torch.randint(0, 24, (n,), device=DEV, generator=g)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    off[1:] = lens.cumsum(0)
    m, windows, c, f = int(off[-1]), [5, 13], 6, 64
    pk = sf.DevicePackets(off.int(), torch.randint(40, 1500, (m,), device=DEV, generator=g).to(torch.int16),
                          torch.rand(m, device=DEV, generator=g), (torch.rand(m, device=DEV, generator=g) < 0.5).to(torch.uint8))
    forest = sf.DeviceForest(trees, depth, c, f, torch.randint(0, f, (trees, 2 ** depth - 1), device=DEV, generator=g).to(torch.int16),
                             torch.rand((trees, 2 ** depth - 1), device=DEV, generator=g) * 500,
                             torch.randint(0, c, (trees, 2 ** depth), device=DEV, generator=g).to(torch.uint8))
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, trees, depth, f))
    ctx.sf_forest_pack(forest)
    new = lambda: torch.full((n,), -1, dtype=torch.int16, device=DEV)
    pred, top, want_pred, want_top = new(), new(), new(), new()
    feat, want = torch.full((n, f), -3.0, device=DEV), torch.zeros((n, f), device=DEV)
    ctx.sf_featurize(pk, windows, want)
    ctx.sf_fast_infer(want, forest, want_pred, want_top)
    vmin = int(want_top.int().median()) + 1
    ctx.sf_featurize_fast_infer(pk, windows, forest, vmin, feat if keep else None, pred, top)
    assert torch.equal(pred, want_pred) and torch.equal(top, want_top)
    if keep:
        under = want_top.int() < vmin
        assert torch.equal(feat[under].view(torch.int32), want[under].view(torch.int32))
        assert bool((feat[~under] == -3.0).all())
