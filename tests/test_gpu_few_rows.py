"""The bfloat16 slow model where a block has one row block of 32 rows: a row's logits and label are the same bits as in the tiles of a
longer list (16,400 rows: more than a row block a block on 256 compute units), for every count of k-steps and column blocks a wave,
inputs and outputs around whole blocks, rows off the 16-byte grid, with and without an input map, and through a separate label index."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
LONG = 16400


@pytest.mark.parametrize("dims,ld,has_map", [
    ((64, 512, 512, 10), 64, True), ((128, 512, 512, 32), 128, True), ((65, 256, 257, 7), 65, True), ((1, 257, 256, 1), 3, False), ((96, 300, 200, 31), 96, True),
    ((31, 33, 500, 4), 33, True), ((127, 288, 31, 2), 128, False), ((12, 30, 20, 5), 12, True)])
def test_same_bits(dims, ld, has_map):
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(dims[1] * 1000 + dims[2])
    rand = lambda *s: torch.randn(s, device=DEV, generator=g)
    par = []
    for o, k in zip(dims[1:], dims[:-1]):
        par += [(rand(o, k) / k ** 0.5).to(torch.bfloat16), rand(o) * 0.1]
    mu, inv = (rand(dims[0]), torch.rand(dims[0], device=DEV, generator=g) + 0.5) if has_map else (None, None)
    feat = rand(LONG, ld)
    mlp = sf.DeviceMlp(dims, sf.SF_BF16, *par, mu=mu, inv_sigma=inv)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(LONG, 0, 0, *dims[:3]))
    ctx.sf_mlp_order(mlp)

    def run(rows, cap, pairs):
        first = torch.arange(rows, dtype=torch.int32, device=DEV)
        idx = torch.cat([first, torch.full((cap - rows,), 2 ** 31 - 1, dtype=torch.int32, device=DEV)])
        count = torch.tensor([rows], dtype=torch.int32, device=DEV)
        logits = torch.full((cap, dims[3]), float("nan"), device=DEV)
        labels = torch.full((LONG,), -1, dtype=torch.int16, device=DEV)
        if pairs:
            ctx.sf_slow_infer_pairs(mlp, feat, idx, (LONG - 1 - idx.long()).clamp(0).to(torch.int32), count, labels, logits=logits)
            labels = labels.flip(0)
        else:
            ctx.sf_slow_infer(mlp, idx, count, labels, feat=feat, logits=logits)
        return logits, labels

    want, want_labels = run(LONG, LONG, False)
    assert not torch.isnan(want).any()
    for rows, cap in ((1, 1), (31, 31), (32, 97), (33, 33), (500, 9000), (8191, 8192), (8193, 30000)):
        for pairs in (False, True):
            got, labels = run(rows, min(cap, LONG), pairs)
            assert torch.equal(got[:rows].view(torch.int32), want[:rows].view(torch.int32)), (rows, cap, pairs)
            assert torch.isnan(got[rows:]).all()
            assert torch.equal(labels[:rows], want_labels[:rows]) and (labels[rows:] == -1).all(), (rows, cap, pairs)
