"""The one-lane form of the feature kernel on batches large enough for it (the rule is in featurize.hip), for each packet
capacity, with what the small batches of the other tests no longer bring to it: flows of every length from none up, in one
wave (so that its windows take different networks), times with their sign bit set, arrays off the alignment of the wide
loads, a last block that is nearly empty.  "even" batches are ragged too, but their mean length is the window's, which
is what the rule takes flows of one length for.  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CU = 256                                  # compute units of the device
TWO, SIX, EIGHT = 2 * 256 * CU, 6 * 256 * CU, 8 * 256 * CU  # flows for two, six, eight waves per SIMD: where the rule's lines lie


@pytest.mark.parametrize("n,depths,longest,even,negative,skew,pad", [
    (TWO + 37, (1, 4), 9, False, False, 0, 0), (TWO + 1, (3,), 5, False, True, 1, 1), (EIGHT + 5, (2, 6), 8, False, True, 0, 0),
    (TWO + 37, (3, 8), 8, True, True, 0, 0), (TWO + 63, (2, 4, 6, 8), 8, True, False, 1, 2), (TWO + 2, (8,), 8, True, False, 0, 0),
    (SIX + 37, (5, 10), 20, False, True, 0, 0), (SIX + 1, (7, 15), 16, False, False, 1, 0), (SIX + 9, (9,), 64, False, False, 0, 3),
    (TWO + 37, (8, 16), 16, True, True, 0, 0), (TWO + 1, (1, 5, 11, 16), 16, True, False, 1, 1),
    (TWO + 37, (5, 20), 40, False, True, 0, 0), (TWO + 1, (8, 16, 24, 32), 40, False, True, 1, 1), (TWO + 65, (32,), 32, True, False, 0, 0)])
def test_lanes(n, depths, longest, even, negative, skew, pad):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + 100 * depths[-1] + len(depths))
    lens = rng.integers(0, longest + 1, size=n)
    if even:                               # pairs of top + d and top - d packets: as many packets as n flows of top
        top = depths[-1]
        lens[1::2] = 2 * top - lens[0:n - 1:2]
        lens[n - n % 2:] = top
        assert lens.sum() == top * n and lens.min() == 0 and lens.max() == 2 * top
    off = np.zeros(n + 1, np.uint32)
    off[1:] = np.cumsum(lens)
    m = int(off[-1])
    size = rng.integers(0, 65536, size=m, dtype=np.uint16)
    iat = np.exp(rng.normal(-6, 2, size=m)).astype(np.float32)
    if negative:                           # some waves with, most without
        at = rng.integers(0, m, size=200)
        iat[at] *= -1
    direction = rng.integers(0, 2, size=m, dtype=np.uint8)
    want, _ = oracle.featurize(off, size, iat, direction, depths, n_threads=8)
    dev = "cuda:0"
    up = lambda a: torch.from_numpy(a).to(dev)
    arrays = [up(size.view(np.int16)), up(iat), up(direction)]
    if skew:                               # arrays one element off the alignment of the wide loads
        arrays = [torch.cat([t[:1], t])[1:] for t in arrays]
    F = 32 * len(depths)
    got = torch.full((n, F + pad), -777.0, dtype=torch.float32, device=dev)
    ctx = sf.ServeFlow(1 << 20)
    ctx.sf_featurize(sf.DevicePackets(up(off.view(np.int32)), *arrays), list(depths), got)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    assert np.array_equal(got[:, :F].view(np.uint32), want.view(np.uint32))
    assert np.all(got[:, F:] == -777.0)
