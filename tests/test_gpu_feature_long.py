"""Windows deeper than 32 packets on both sides of the line between one lane per flow and four waves per 64 flows (512 flows a
compute unit, 16 packets a flow on average): the same bits as the oracle on pieces of the batch, and for pieces as for the whole."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("n,mean,depths", [(131077, 8, (8, 64)), (131077, 30, (33,)), (40001, 12, (5, 40, 64)), (197, 60, (16, 34, 50, 64)), (64, 64, (63,)), (3, 33, (1, 33))])
def test_long_windows(n, mean, depths):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + mean)
    lens = np.clip(rng.geometric(1.0 / mean, n), 1, 70) if mean < 60 else rng.integers(mean - 30, 71, n)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint32)
    m = int(off[-1])
    size = rng.integers(40, 1501, m).astype(np.uint16)
    iat = np.exp(rng.standard_normal(m) * 2 - 6).astype(np.float32)
    way = rng.integers(0, 2, m).astype(np.uint8)
    up = lambda a, t: torch.from_numpy(np.ascontiguousarray(a).view(t)).to(DEV)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n))

    def run(a, b):
        p, q = int(off[a]), int(off[b])
        pk = sf.DevicePackets(up(off[a:b + 1] - off[a], np.int32), up(size[p:q], np.int16), up(iat[p:q], np.float32), up(way[p:q], np.uint8))
        feat = torch.full((b - a, 32 * len(depths)), -1.0, device=DEV)
        ctx.sf_featurize(pk, list(depths), feat)
        return feat.cpu().numpy().view(np.uint32)

    whole = run(0, n)
    for a in range(0, n, 30011):
        b = min(n, a + 30011)
        assert np.array_equal(run(a, b), whole[a:b]), a
    for a, b in ((0, min(n, 700)), (max(0, n - 700), n)):
        p, q = int(off[a]), int(off[b])
        want, _ = oracle.featurize(off[a:b + 1] - off[a], size[p:q], iat[p:q], way[p:q], depths)
        assert np.array_equal(whole[a:b], want.view(np.uint32)), a
