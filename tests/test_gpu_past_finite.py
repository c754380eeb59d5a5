"""Infinite and missing values through the bfloat16 models' forms (wide ones: few rows, tiles, the last layer along with the second
hidden one, split over K, 256 rows a block; narrow ones: a row block a block, tiles, registers) and the binary32 model's in one launch
(4 and 16 rows a block): a row's logits follow from its own values whatever the form, against binary64 (binary32: the same sums), and
the label is the oracle's, class 0 first, then every class that is strictly larger than the best before it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
INF, NAN = float("inf"), float("nan")


def _labels(v):
    best, label = v[:, 0].copy(), np.zeros(len(v), np.int16)
    for c in range(1, v.shape[1]):
        take = v[:, c] > best   # (false beside a NaN)
        best[take], label[take] = v[take, c], c
    return label


def _same(a, b):
    return np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.nan_to_num(a, nan=0.0), np.nan_to_num(b, nan=0.0))


def _run(mlp, feat, rows):
    import torch
    import paper_2402_03694_amd as sf
    most = len(feat)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(most, 0, 0, *mlp.dims[:3]))
    idx = torch.arange(most, dtype=torch.int32, device=DEV)
    for r, cap in [(r, cap) for r in rows for cap in {r, most}]:
        logits = torch.full((cap, mlp.dims[3]), -7.0, device=DEV)
        labels = torch.full((most,), -1, dtype=torch.int16, device=DEV)
        ctx.sf_slow_infer(mlp, idx, torch.tensor([r], dtype=torch.int32, device=DEV), labels, feat=feat, logits=logits)
        got, lab = logits.cpu().numpy(), labels.cpu().numpy()
        assert (got[r:] == -7).all() and (lab[r:] == -1).all(), (r, cap)
        assert np.array_equal(lab[:r], _labels(got[:r])), (r, cap)
        yield (r, cap), got[:r]


def _special(par, x, case):
    """Weights, biases and inputs (numpy) with the case's values put in."""
    w1, b1, w2, b2, w3, b3 = par
    if case == "hidden":    # the last unit of each hidden layer is infinite; it makes one unit of the next one so and the others zero
        b1[-1] = INF
        w2[:, -1] = -np.abs(w2[:, -1]) - 0.01
        w2[5, -1] = 0.5
        w3[:, 5] = np.where(np.arange(len(b3)) % 3 == 1, 0.5, -0.5)
    elif case == "out":     # missing and infinite logits in both halves of a lane pair's classes
        b3[0::4], b3[1::5] = NAN, INF
        if len(b3) > 2:
            b3[2] = -INF
    else:                   # inputs
        x[5, 3], x[33, 0], x[1000, -1], x[len(x) - 2, 1] = INF, NAN, -INF, NAN


@pytest.mark.parametrize("case", ["hidden", "out", "in"])
@pytest.mark.parametrize("dims", [(40, 600, 500, 7), (64, 530, 577, 32), (32, 520, 96, 64), (33, 520, 520, 1), (64, 300, 1100, 33), (40, 100, 75, 6), (96, 300, 300, 32)])
def test_bfloat16(dims, case):
    import torch
    import paper_2402_03694_amd as sf
    most = 49999
    rng = np.random.default_rng(dims[1] + dims[2])
    bf = lambda a: torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16)
    par = [rng.standard_normal(s) * (k ** -0.5 if len(s) == 2 else 0.1) for o, k in zip(dims[1:], dims[:-1]) for s in ((o, k), (o,))]
    x = rng.standard_normal((most, dims[0])).astype(np.float32)
    _special(par, x, case)
    par = [bf(p) if p.ndim == 2 else torch.from_numpy(p.astype(np.float32)) for p in par]
    mlp = sf.DeviceMlp(dims, sf.SF_BF16, *[p.to(DEV) for p in par])
    rows = (most, 1, 33, 1023, 2049, 5000, 20000, 32769)
    out = dict(_run(mlp, torch.from_numpy(x).to(DEV), rows))
    for (r, cap), got in out.items():
        assert _same(got, out[most, most][:r]), (r, cap)
    at = np.r_[0:64, 1000, most - 2]   # (the bound is test_gpu_wide_last's)
    h = bf(x[at]).double()
    for layer in range(3):
        h = h @ par[2 * layer].double().T + par[2 * layer + 1].double()
        if layer < 2:
            h = torch.where(h > 0, h, torch.zeros_like(h)).to(torch.bfloat16).double()   # (a hidden NaN counts as zero)
    want, got = h.numpy(), out[most, most][at].astype(np.float64)
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), fin) and _same(got[~fin], want[~fin])
    assert (np.abs(got[fin] - want[fin]) < 1e-2).all()


@pytest.mark.parametrize("case", ["hidden", "out", "in"])
@pytest.mark.parametrize("dims", [(17, 130, 70, 5), (64, 300, 129, 33), (30, 9, 300, 64)])
def test_binary32(dims, case):
    import torch
    import paper_2402_03694_amd as sf
    most = 2100
    rng = np.random.default_rng(dims[1])
    par = [(rng.standard_normal(s) / 8).astype(np.float32) for o, k in zip(dims[1:], dims[:-1]) for s in ((o, k), (o,))]
    x = rng.standard_normal((most, dims[0])).astype(np.float32)
    _special(par, x, case)
    mlp = sf.DeviceMlp(dims, sf.SF_F32, *[torch.from_numpy(p).to(DEV) for p in par])
    out = dict(_run(mlp, torch.from_numpy(x).to(DEV), (most, 1, 40, 1500, 2048, 2049)))
    h = x
    with np.errstate(invalid="ignore"):
        for layer in range(3):
            acc = np.zeros((most, dims[layer + 1]), np.float32)
            for k in range(dims[layer]):
                acc = acc + h[:, k:k + 1] * par[2 * layer][:, k][None, :]
            h = acc + par[2 * layer + 1]
            if layer < 2:
                h = np.where(h < 0, np.float32(0), h)
    for r, got in out.items():
        assert _same(got, h[:len(got)]), r
