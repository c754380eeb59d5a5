"""The binary32 slow model in one launch, eight rows per block: row counts around a block and past the grid, widths
around the pieces of 128 outputs x 32 inputs, weights off the 16-byte grid, header bits as input, a model too wide
for it and a list too long (one launch per layer).  Logits bit for bit: the sums run in order of the inputs, one multiply and one add per
term, each rounded."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("rows,dims,raw", [
    (1, (32, 8, 8, 2), 0), (7, (31, 33, 130, 64), 0), (9, (64, 128, 128, 4), 0), (200, (64, 129, 64, 33), 0), (77, (100, 255, 257, 7), 0),
    (8193, (32, 40, 36, 5), 0), (40, (3 * 21, 64, 127, 9), 21), (30, (96, 1000, 700, 6), 0), ((1 << 15) - 10, (8, 9, 10, 3), 0)])
def test_rows(rows, dims, raw):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(rows + dims[1])
    n = rows + 11
    idx = np.sort(rng.permutation(n)[:rows]).astype(np.int32)
    off1 = rows % 2                        # weights one element off the 16-byte grid
    dev = lambda a: torch.from_numpy(np.concatenate([a.reshape(-1)[:off1], a.reshape(-1)])).to(DEV)[off1:].reshape(a.shape)
    par = [(rng.standard_normal(s) / 8).astype(np.float32) for o, k in zip(dims[1:], dims[:-1]) for s in ((o, k), (o,))]
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    logits = torch.full((n, dims[3]), float("nan"), device=DEV)
    labels = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    kw, mu, inv = {}, None, None
    if raw:
        m = 3 * n
        hdr = rng.integers(-2 ** 31, 2 ** 31, size=(m, 1), dtype=np.int64).astype(np.int32)
        z = lambda t: torch.zeros(m, dtype=t, device=DEV)
        pk = sf.DevicePackets(torch.arange(0, m + 1, 3, dtype=torch.int32, device=DEV), z(torch.int16), z(torch.float32), z(torch.uint8),
                              torch.from_numpy(hdr).to(DEV))
        b = np.arange(raw)
        x = ((hdr.view(np.uint32) >> (b // 8 * 8 + 7 - b % 8).astype(np.uint32)) & 1).astype(np.float32).reshape(n, -1)
        kw = dict(raw_src=pk, raw_pkts=3, raw_bits=raw)
    else:
        x = rng.standard_normal((n, dims[0])).astype(np.float32)
        mu, inv = rng.standard_normal(dims[0]).astype(np.float32), (rng.random(dims[0]) + 0.5).astype(np.float32)
        kw = dict(feat=torch.from_numpy(x).to(DEV))
        x = np.clip((x - mu) * inv, np.float32(-8), np.float32(8))
        mu, inv = torch.from_numpy(mu).to(DEV), torch.from_numpy(inv).to(DEV)
    mlp = sf.DeviceMlp(dims, sf.SF_F32, *[dev(p) for p in par], mu=mu, inv_sigma=inv)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 0, 0, *dims[:3]))
    full = np.concatenate([idx, np.zeros(n - rows, np.int32)])
    ctx.sf_slow_infer(mlp, torch.from_numpy(full).to(DEV), count, labels, logits=logits, **kw)
    torch.cuda.synchronize()
    h = x[idx]
    for layer in range(3):
        w, bias = par[2 * layer], par[2 * layer + 1]
        acc = np.zeros((rows, w.shape[0]), np.float32)
        for k in range(w.shape[1]):
            acc = acc + h[:, k:k + 1] * w[:, k][None, :]
        h = acc + bias
        if layer < 2:
            h = np.where(h < 0, np.float32(0), h)
    got = logits.cpu().numpy()
    assert np.array_equal(got[:rows].view(np.uint32), h.view(np.uint32)) and np.isnan(got[rows:]).all()
    want = np.full(n, -1, np.int16)
    want[idx] = h.argmax(1)
    assert np.array_equal(labels.cpu().numpy(), want)
