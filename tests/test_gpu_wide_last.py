"""The layers of a wide model in each of their forms.  The hidden layers: 32 rows x 256 columns a block while that gives a block one
tile (1,024 columns: 2,048 rows), 128 rows x 512 columns past it.  The last layer: along with the second hidden layer (all columns of a row in one block),
split by pieces of K over a block's waves (short lists), 256 rows a block (long ones).  A row's logits and label are the same bits in
all of them, with and without operand-ordered weights, and agree with binary64 on the same activations' layers."""
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dims", [(64, 1024, 1024, 16), (64, 150, 1000, 31), (40, 600, 500, 7), (64, 530, 577, 32), (33, 520, 520, 1),
                                  (64, 600, 1100, 33), (32, 520, 96, 64),
                                  (600, 1100, 64, 5), (40, 2100, 530, 9)])
def test_same_bits(dims):
    import torch
    import paper_2402_03694_amd as sf
    most = 65536 if dims[2] > 512 else 50000
    g = torch.Generator(device=DEV)
    g.manual_seed(dims[2])
    rand = lambda *s: torch.randn(s, device=DEV, generator=g)
    par = []
    for o, k in zip(dims[1:], dims[:-1]):
        par += [(rand(o, k) / k ** 0.5).to(torch.bfloat16), rand(o) * 0.1]
    feat = rand(most, dims[0])
    idx = torch.arange(most, dtype=torch.int32, device=DEV)
    out = []
    for ordered in (False, True):
        if ordered and dims[3] > 32:
            continue
        mlp = sf.DeviceMlp(dims, sf.SF_BF16, *par)
        ctx = sf.ServeFlow(sf.sf_workspace_bytes(most, 0, 0, *dims[:3]))
        if ordered:
            ctx.sf_mlp_order(mlp)
        for rows in (most, 1, 33, 1023, 2048, 2049, 5000, 32769, 49153, most - 31):   # (256 compute units: the second hidden layer takes the last one along for `most`)
            logits = torch.full((most, dims[3]), float("nan"), device=DEV)
            labels = torch.full((most,), -1, dtype=torch.int16, device=DEV)
            ctx.sf_slow_infer(mlp, idx, torch.tensor([rows], dtype=torch.int32, device=DEV), labels, feat=feat, logits=logits)
            assert torch.isnan(logits[rows:]).all() and (labels[rows:] == -1).all(), rows
            out.append((rows, logits[:rows].clone(), labels[:rows].clone()))
    want, want_labels = out[0][1:]
    for rows, logits, labels in out:
        assert torch.equal(logits.view(torch.int32), want[:rows].view(torch.int32)), rows
        assert torch.equal(labels, want_labels[:rows]) and torch.equal(labels.long(), logits.argmax(1)), rows
    # binary64 from the same bfloat16 weights, hidden activations rounded to bfloat16: binary32 sums of up to 1,024 terms are within
    # 1e-4, an activation on the other side of a rounding boundary adds 2^-8 of it times a weight (rms 1/32): 1e-2 in all
    x = feat[:64].to(torch.bfloat16).double()
    for layer in range(3):
        x = x @ par[2 * layer].double().T + par[2 * layer + 1].double()
        if layer < 2:
            x = x.clamp(min=0).to(torch.bfloat16).double()
    assert (x - want[:64].double()).abs().max() < 1e-2
