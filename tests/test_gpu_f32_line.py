"""The binary32 slow model on both sides of the line between one launch for the whole model and one per layer (rows of the
list times terms of a row): the same bits, and a long list through a wide model at the rate of a longer one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _setup(rows, cap, dims, seed):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(seed)
    par = [(rng.standard_normal(s) / 16).astype(np.float32) for o, k in zip(dims[1:], dims[:-1]) for s in ((o, k), (o,))]
    x = rng.standard_normal((rows, dims[0])).astype(np.float32)
    up = lambda a: torch.from_numpy(a).to(DEV)
    feat = torch.zeros((cap, dims[0]), device=DEV)
    feat[cap - rows:] = up(x)
    idx = torch.zeros(cap, dtype=torch.int32, device=DEV)
    idx[:rows] = torch.arange(cap - rows, cap, dtype=torch.int32, device=DEV)
    mlp = sf.DeviceMlp(dims, sf.SF_F32, *[up(p) for p in par])
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(cap, 0, 0, *dims[:3]))
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    logits = torch.full((cap, dims[3]), float("nan"), device=DEV)
    labels = torch.full((cap,), -1, dtype=torch.int16, device=DEV)
    return x, par, lambda: ctx.sf_slow_infer(mlp, idx, count, labels, feat=feat, logits=logits), logits, labels


@pytest.mark.parametrize("dims", [(64, 700, 700, 3), (32, 650, 600, 64)])
@pytest.mark.parametrize("cap", [8000, 12000, 32768, 32769])
def test_bits(dims, cap):
    import torch
    rows = 50
    x, par, call, logits, labels = _setup(rows, cap, dims, cap + dims[1])
    call()
    torch.cuda.synchronize()
    h = x
    for layer in range(3):
        w, bias = par[2 * layer], par[2 * layer + 1]
        acc = np.zeros((rows, w.shape[0]), np.float32)
        for k in range(w.shape[1]):
            acc = acc + h[:, k:k + 1] * w[:, k][None, :]
        h = acc + bias
        if layer < 2:
            h = np.where(h < 0, np.float32(0), h)
    assert np.array_equal(logits[:rows].cpu().numpy().view(np.uint32), h.view(np.uint32)) and torch.isnan(logits[rows:]).all()
    want = np.full(cap, -1, np.int16)
    want[cap - rows:] = h.argmax(1)
    assert np.array_equal(labels.cpu().numpy(), want)


def test_rate():
    """A row of 32,768 takes at most 1.4 times a row of 100,000 (one launch for the whole model: 1.7 times)."""
    import torch
    per_row = []
    for rows in (100000, 32768):
        _, _, call, _, _ = _setup(rows, rows, (128, 650, 650, 10), rows)
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            call()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        per_row.append(sorted(times)[2] / rows)
    assert per_row[1] <= 1.4 * per_row[0], per_row
