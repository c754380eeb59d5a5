"""The gate, each of its kernels: one launch for small batches, sizes around its tiles of 8,192 rows and around the lines to the two launches (40,960 rows for
gates that read two arrays, 65,536 for the others) and above, where blocks take several tiles, every gate, arrays off the alignment of the wide loads, lists shorter than their
capacity, NaN scores.  Lists and counts exactly as numpy gives them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [1, 7, 8, 9, 511, 8191, 8192, 8193, 16385, 24576 + 5, 40959, 40960, 40961, 49152 + 3, 65535, 65536, 65537, (1 << 20) + 5, (1 << 23) + 9]


def _case(n, off):
    import torch
    import paper_2402_03694_amd as sf
    rng = np.random.default_rng(n + off)
    dev = "cuda:0"
    put = lambda x: torch.from_numpy(np.concatenate([x[:1].repeat(off), x]).view(np.int16 if x.dtype == np.uint16 else x.dtype)).to(dev)[off:]
    return torch, sf, rng, dev, put, sf.ServeFlow(sf.sf_workspace_bytes(n, 1, 1))


def _check(torch, dev, n, call, want):
    idx, count = torch.full((n,), -1, dtype=torch.int32, device=dev), torch.full((1,), -1, dtype=torch.int32, device=dev)
    call(idx, count)
    torch.cuda.synchronize()
    assert int(count[0]) == want.size
    got = idx.cpu().numpy()
    assert np.array_equal(got[:want.size], want) and np.all(got[want.size:] == -1)


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("n", SIZES)
def test_gates(n, off):
    torch, sf, rng, dev, put, ctx = _case(n, off)
    top, pred = rng.integers(0, 100, n).astype(np.uint16), rng.integers(0, 12, n).astype(np.uint16)
    total = rng.integers(0, 130, n).astype(np.uint16)
    score = rng.random(n).astype(np.float32)
    score[rng.integers(0, n, 1 + n // 50)] = rng.choice(np.array([np.nan, np.inf, 0.75], np.float32), 1 + n // 50)
    vmin = rng.integers(0, 101, 10)
    d_top, d_pred, d_total, d_score = put(top), put(pred), put(total), put(score)
    for v in (0, 30, 101):
        _check(torch, dev, n, lambda i, c: ctx.sf_route(d_top, d_pred, v, i, c), np.flatnonzero(top < v))
    _check(torch, dev, n, lambda i, c: ctx.sf_route(d_top, d_pred, vmin.astype(int).tolist(), i, c),
           np.flatnonzero(top < vmin[np.minimum(pred, 9)]))  # (a class past the last threshold takes the last)
    _check(torch, dev, n, lambda i, c: ctx.sf_route_score(d_score, 0.75, i, c), np.flatnonzero(score > np.float32(0.75)))
    theta = np.float32(0.6)
    below = np.where(total == 0, True, top.astype(np.float64) < np.float64(theta) * total)
    _check(torch, dev, n, lambda i, c: ctx.sf_route_ratio(d_top, d_total, float(theta), i, c), np.flatnonzero(below))


@pytest.mark.parametrize("n,live", [(1, 0), (9, 8), (8193, 8192), (40000, 0), (40960, 8193), (40961, 40000), (65536, 16384), (65536, 65536), (65536, 65535)])
@pytest.mark.parametrize("per_class", [False, True])
def test_lists(n, live, per_class):
    torch, sf, rng, dev, put, ctx = _case(n, 0)
    src = np.sort(rng.permutation(4 * n)[:n]).astype(np.int32)
    top, pred = rng.integers(0, 100, n).astype(np.uint16), rng.integers(0, 10, n).astype(np.uint16)
    vmin = rng.integers(0, 101, 10) if per_class else np.full(10, 45)
    d_src, d_live = torch.from_numpy(src).to(dev), torch.tensor([live], dtype=torch.int32, device=dev)
    want = src[:live][top[:live] < vmin[pred[:live]]]
    _check(torch, dev, n, lambda i, c: ctx.sf_route_subset(put(top), put(pred), d_src, d_live, vmin.astype(int).tolist() if per_class else 45, i, c), want)
