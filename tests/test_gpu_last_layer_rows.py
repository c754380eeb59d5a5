"""The last layer of a wide model in launches of its own: 32 rows a block or 256 (128 with more than 32 classes), dealt out so that a row
is read where the layer before wrote it.  Row counts around whole groups of blocks of either, past the grid, and lists that end inside a
group give every row the bits it has in the whole batch."""
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dims", [(16, 520, 36, 5), (16, 520, 40, 7), (8, 40, 1030, 3), (16, 520, 36, 40)])
def test_last_layer(dims):
    import torch
    import paper_2402_03694_amd as sf
    most = 264000 if dims[2] < 512 else 70000   # (256 rows a block on 1,024 blocks: 262,144)
    g = torch.Generator(device=DEV)
    g.manual_seed(dims[2] + dims[3])
    rand = lambda *s: torch.randn(s, device=DEV, generator=g)
    par = []
    for o, k in zip(dims[1:], dims[:-1]):
        par += [(rand(o, k) / k ** 0.5).to(torch.bfloat16), rand(o) * 0.1]
    mlp = sf.DeviceMlp(dims, sf.SF_BF16, *par)
    feat = rand(most, dims[0])
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(most, 0, 0, *dims[:3]))
    idx = torch.arange(most, dtype=torch.int32, device=DEV)

    def run(rows):
        logits = torch.full((most, dims[3]), float("nan"), device=DEV)
        labels = torch.full((most,), -1, dtype=torch.int16, device=DEV)
        ctx.sf_slow_infer(mlp, idx, torch.tensor([rows], dtype=torch.int32, device=DEV), labels, feat=feat, logits=logits)
        assert torch.isnan(logits[rows:]).all() and (labels[rows:] == -1).all(), rows
        return logits[:rows], labels[:rows]

    want, want_labels = run(most)
    assert not torch.isnan(want).any() and torch.equal(want_labels.long(), want.argmax(1))
    for rows in (31, 32, 993, 1024, 1025, 8193, 8320, 20480, 20481, 32768, 33793, 34816, 34817, 36865, 40961, 65537):
        got, labels = run(rows)
        assert torch.equal(got.view(torch.int32), want[:rows].view(torch.int32)), rows
        assert torch.equal(labels, want_labels[:rows]), rows


@pytest.mark.parametrize("dims", [(8, 40, 1100, 3), (8, 520, 500, 7), (8, 520, 200, 32), (8, 520, 1030, 40)])
def test_one_chain(dims):
    """A logit is one binary32 chain in order of K: behind 2^26 each step's 16 products of 1/4 are half a unit in the last place and go
    (halves round to the even 2^26), 64 of them summed apart would not.  Hidden units are all one."""
    import torch
    import paper_2402_03694_amd as sf
    most = 70000
    w3 = torch.full((dims[3], dims[2]), 0.25)
    w3[:, :16] = 2.0 ** 22
    zero = lambda o, k: torch.zeros((o, k), dtype=torch.bfloat16, device=DEV)
    par = (zero(dims[1], dims[0]), torch.ones(dims[1], device=DEV), zero(dims[2], dims[1]), torch.ones(dims[2], device=DEV), w3.to(torch.bfloat16).to(DEV),
           torch.zeros(dims[3], device=DEV))
    feat = torch.zeros((most, dims[0]), device=DEV)
    idx = torch.arange(most, dtype=torch.int32, device=DEV)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(most, 0, 0, *dims[:3]))
    for ordered in (False, True):
        mlp = sf.DeviceMlp(dims, sf.SF_BF16, *par)
        if ordered and dims[3] <= 32:
            ctx.sf_mlp_order(mlp)
        for rows in (1, 500, 5000, 16384, 32769, most):
            logits = torch.zeros((most, dims[3]), device=DEV)
            labels = torch.full((most,), -1, dtype=torch.int16, device=DEV)
            ctx.sf_slow_infer(mlp, idx, torch.tensor([rows], dtype=torch.int32, device=DEV), labels, feat=feat, logits=logits)
            assert (logits[:rows] == 2.0 ** 26).all() and (labels[:rows] == 0).all(), (ordered, rows)
