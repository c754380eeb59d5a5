"""Windows deeper than 32 packets on both sides of the lines between one lane per flow and four waves per 64 flows, for flows of one
length and ragged ones (256 compute units): a batch's rows are the bits of its pieces, which go in parts."""
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("n,mean,ragged", [(49151, 4, False), (49152, 4, False), (50001, 12, False), (81920, 32, False), (81919, 32, False), (196609, 16, False),
                                           (65537, 2, True), (98305, 7, True), (131073, 11, True), (98305, 33, False)])
def test_deep_windows(n, mean, ragged):
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(n + mean)
    off = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    lens = torch.full((n,), mean, device=DEV)
    if ragged:   # 0 to 2 mean - 1 packets, and some long flows where the mean leaves room
        lens = torch.randint(0, 2 * mean - 1, (n,), device=DEV, generator=g)
        lens[5::400] = 40 if mean > 2 else 3
    off[1:] = torch.cumsum(lens, 0)
    m = int(off[-1])
    size = torch.randint(40, 1500, (m,), device=DEV, generator=g).to(torch.int16)
    iat, way = torch.rand(m, device=DEV, generator=g), (torch.rand(m, device=DEV, generator=g) < 0.5).to(torch.uint8)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n))

    def run(a, b):
        p, q = int(off[a]), int(off[b])
        pk = sf.DevicePackets((off[a:b + 1] - off[a]).contiguous(), size[p:q].clone(), iat[p:q].clone(), way[p:q].clone())
        feat = torch.full((b - a, 64), -1.0, device=DEV)
        ctx.sf_featurize(pk, [5, 64], feat)
        return feat.view(torch.int32)

    whole = run(0, n)
    for a in range(0, n, 30011):
        b = min(n, a + 30011)
        assert torch.equal(run(a, b), whole[a:b]), a
