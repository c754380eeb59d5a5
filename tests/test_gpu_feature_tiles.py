"""The stand-alone feature kernel at the edges of its tiles of 64 flows, for each packet capacity (windows up to 8, 16
and 32 packets): a flow too many or too few, one to four windows on and off the capacity, empty flows, arrays off the
alignment of the wide loads, rows off the 16-byte grid, times with their sign bit set.  Bit for bit against the
oracle; columns past the features untouched."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SENTINEL = -777.0


@pytest.mark.parametrize("n,depths,longest,negative,shift,skew,pad", [
    (1, (8,), 9, False, 0, 0, 0), (63, (1, 7), 8, True, 1, 0, 4), (64, (3, 8), 8, False, 0, 1, 1), (65, (2, 4, 6, 8), 20, False, 0, 0, 0),
    (1, (9,), 9, True, 0, 0, 0), (127, (16,), 16, False, 1, 0, 3), (128, (8, 16), 64, False, 0, 0, 0), (129, (1, 8, 9, 16), 17, True, 0, 1, 0),
    (1, (32,), 64, False, 0, 0, 0), (191, (17,), 18, True, 1, 0, 0), (192, (16, 31), 33, False, 0, 1, 1), (193, (8, 16, 24, 32), 32, False, 0, 0, 0),
    (3 * 4 * 64 * 256, (8, 16), 16, False, 0, 0, 0), (3 * 4 * 64 * 256 + 1, (5, 8), 8, True, 0, 0, 1),
    (2 * 4 * 64 * 256, (5, 20), 32, False, 1, 0, 0), (20011, (3, 9, 20), 64, False, 3, 0, 0), (20011, (8, 16, 32), 40, True, 0, 0, 2)])
def test_tiles(n, depths, longest, negative, shift, skew, pad):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(1000 * n + depths[-1])
    top = depths[-1]
    full = n > 100000                      # (as many flows as one lane per flow is used for, on a whole device: every window full)
    lens = np.where(full | (rng.random(n) < 0.5), min(top, longest), rng.integers(0, longest + 1, size=n))
    off = np.zeros(n + 1, np.uint32)
    off[1:] = np.cumsum(lens)
    off += np.uint32(shift)                # (the first packets of the arrays belong to no flow)
    m = int(off[-1])
    size = rng.integers(0, 65536, size=m, dtype=np.uint16)
    iat = np.exp(rng.normal(-6, 2, size=m)).astype(np.float32)
    if negative:
        iat[rng.random(m) < 0.01] *= -1
    direction = rng.integers(0, 2, size=m, dtype=np.uint8)
    want, _ = oracle.featurize(off, size, iat, direction, depths, n_threads=8)
    dev = "cuda:0"
    up = lambda a: torch.from_numpy(a).to(dev)
    arrays = [up(size.view(np.int16)), up(iat), up(direction)]
    if skew:                               # arrays one element off the alignment of the wide loads
        arrays = [torch.cat([t[:1], t])[1:] for t in arrays]
    F = 32 * len(depths)
    got = torch.full((n, F + pad), SENTINEL, dtype=torch.float32, device=dev)
    ctx = sf.ServeFlow(1 << 20)
    ctx.sf_featurize(sf.DevicePackets(up(off.view(np.int32)), *arrays), list(depths), got)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    assert np.array_equal(got[:, :F].view(np.uint32), want.view(np.uint32))
    assert np.all(got[:, F:] == SENTINEL)
