"""The slow model's register form where it can go wrong: runs of rows that end in a full pass, a low one or a tile of one or two
row blocks, widths around the column blocks (odd numbers of them, a width just past a multiple of 128), inputs that are not whole
k-steps, one class and all 32, label indices apart from the input rows, no input map, no logits.
Logits against the same model in 64 bits with the hidden activations rounded to bfloat16; labels: the arg-max of the logits."""
import pytest

from test_gpu_wide_tiles import DEV, _check, _model, _reference

pytestmark = pytest.mark.gpu

UNITS = 256          # compute units: a run is the rows divided by this
CAP = 128 * UNITS + 1  # the shortest list that takes this form (192 * UNITS + 1 for some with more than 64 inputs and 384 columns in the first layer)


def _run(rows, cap, dims, mapped, pairs, with_logits=True):
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + 7 * dims[1] + dims[0])
    n = cap + 77
    mlp = _model(g, dims, mapped)
    feat = torch.randn((n, dims[0] + 4), device=DEV, generator=g)
    idx = torch.randperm(n, device=DEV, generator=g)[:cap].to(torch.int32)
    dst = torch.randperm(n, device=DEV, generator=g)[:cap].to(torch.int32) if pairs else idx
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 0, 0, *dims[:3]))
    torch.cuda.synchronize()
    if rows % 2:
        ctx.sf_mlp_order(mlp)  # (else the call orders the weights in its workspace)
    logits = torch.full((cap, dims[3]), float("nan"), device=DEV) if with_logits else None
    labels = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    if pairs:
        ctx.sf_slow_infer_pairs(mlp, feat, idx, dst, count, labels, logits=logits)
    else:
        ctx.sf_slow_infer(mlp, idx, count, labels, feat=feat, logits=logits)
    torch.cuda.synchronize()
    return mlp, feat[idx[:rows].long(), :dims[0]], logits, labels, dst[:rows], n


@pytest.mark.parametrize("rows", [1, 31, 33, 32 * UNITS + 1, 64 * UNITS + 5, 96 * UNITS + 1, 128 * UNITS, 128 * UNITS + 1, 160 * UNITS + 3, 256 * UNITS,
                                  256 * UNITS + 1, 288 * UNITS + 40, 360 * UNITS + 9, 416 * UNITS + 31])
def test_runs(rows):
    out = _run(rows, max(rows, CAP), (64, 160, 96, 10), mapped=True, pairs=rows % 3 == 0)
    _check(out[0], _reference(out[0], out[1]), *out[2:])


@pytest.mark.parametrize("dims", [(64, 512, 512, 10), (128, 512, 512, 32), (128, 510, 500, 1), (4, 33, 64, 2), (64, 128, 256, 17), (100, 129, 31, 16),
                                  (32, 256, 225, 9), (96, 300, 200, 7), (68, 384, 384, 32), (64, 385, 481, 8), (124, 480, 1, 3), (60, 1, 40, 5)])
def test_widths(dims):
    rows = 290 * UNITS + 11 # one pass of 256 rows a block, then one or two row blocks
    out = _run(rows, rows, dims, mapped=dims[1] % 2 == 0, pairs=False)
    _check(out[0], _reference(out[0], out[1]), *out[2:])


@pytest.mark.parametrize("dims", [(128, 257, 200, 10), (64, 512, 448, 4)])
def test_low_pass(dims):
    rows = 100 * UNITS # three or four row blocks a block
    out = _run(rows, CAP, dims, mapped=True, pairs=True)
    _check(out[0], _reference(out[0], out[1]), *out[2:])


@pytest.mark.parametrize("dims", [(64, 512, 512, 10), (100, 130, 70, 32)])
def test_place_in_the_list(dims):
    """A row's logits are the same bits wherever in the list it stands: in a full pass, a low one or a tile."""
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    mlp = _model(g, dims, True)
    feat = torch.randn((512, dims[0]), device=DEV, generator=g)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(400 * UNITS, 0, 0, *dims[:3]))
    labels = torch.empty(512, dtype=torch.int16, device=DEV)
    first = None
    for rows in (256 * UNITS, 60 * UNITS, 30 * UNITS, 120 * UNITS, 290 * UNITS):
        idx = (torch.arange(max(rows, CAP), device=DEV) * 5 % 512).to(torch.int32)
        logits = torch.empty((len(idx), dims[3]), device=DEV)
        torch.cuda.synchronize()
        # (pairs: a list may be longer than there are input rows)
        ctx.sf_slow_infer_pairs(mlp, feat, idx, idx, torch.tensor([rows], dtype=torch.int32, device=DEV), labels, logits=logits)
        torch.cuda.synchronize()
        first = logits[:512].clone() if first is None else first
        assert torch.equal(logits[:rows], first[torch.arange(rows, device=DEV) % 512])


@pytest.mark.parametrize("dims", [(64, 512, 512, 10), (100, 130, 70, 32), (128, 300, 500, 7), (4, 40, 20, 1), (64, 384, 160, 17), (96, 400, 200, 9)])
@pytest.mark.parametrize("rows", [40, 20011, 128 * UNITS])
def test_forms_agree(dims, rows):
    """A row's logits are the same bits whatever decides between the forms: the list's capacity, the input's row stride, its alignment."""
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(dims[1] + rows)
    mlp = _model(g, dims, True)
    n = 192 * UNITS + 1
    x = torch.randn((n, dims[0]), device=DEV, generator=g)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 0, 0, *dims[:3]))
    outs = []
    for cap, ld, offset in ((rows, dims[0], 0), (128 * UNITS, dims[0], 0), (CAP, dims[0], 0), (n - 1, dims[0], 0), (n, dims[0], 0), (n, dims[0] + 1, 0), (n, dims[0], 1)):
        flat = torch.zeros(n * ld + 1, device=DEV)
        feat = flat[offset:offset + n * ld].view(n, ld)
        feat[:, :dims[0]] = x
        logits = torch.full((cap, dims[3]), float("nan"), device=DEV)
        labels = torch.full((n,), -1, dtype=torch.int16, device=DEV)
        idx = torch.arange(cap, device=DEV, dtype=torch.int32)
        torch.cuda.synchronize()
        ctx.sf_slow_infer(mlp, idx, torch.tensor([rows], dtype=torch.int32, device=DEV), labels, feat=feat, logits=logits)
        torch.cuda.synchronize()
        outs.append((logits[:rows], labels))
    for logits, labels in outs[1:]:
        assert torch.equal(logits, outs[0][0]) and torch.equal(labels, outs[0][1])


@pytest.mark.parametrize("n_in", [1, 3, 8, 30, 68, 70, 127, 132, 200, 510, 512])
@pytest.mark.parametrize("rows,cap", [(1, 1), (64, 70), (40 * UNITS, 40 * UNITS), (70 * UNITS + 5, 70 * UNITS + 5), (30 * UNITS + 3, CAP), (50 * UNITS, CAP)])
def test_input_rows(n_in, rows, cap):
    """Tiles whose input comes in whole 16-byte elements and not, held in registers for the next tile and not, rows missing at the end."""
    out = _run(rows, cap, (n_in, 70, 40, 6), mapped=n_in % 2 == 0, pairs=False)
    _check(out[0], _reference(out[0], out[1]), *out[2:])


def test_labels_alone():
    import torch
    rows = 260 * UNITS
    full = _run(rows, rows, (64, 256, 256, 10), True, False)
    alone = _run(rows, rows, (64, 256, 256, 10), True, False, with_logits=False)
    assert torch.equal(full[3], alone[3])


def _labels(logits):
    """The oracle's rule: class 0 first, then every class that is strictly larger than the best before it."""
    import numpy as np
    v = logits.cpu().numpy()
    best, label = v[:, 0].copy(), np.zeros(len(v), np.int16)
    for c in range(1, v.shape[1]):
        take = v[:, c] > best   # (false beside a NaN)
        best[take], label[take] = v[take, c], c
    return label


@pytest.mark.parametrize("classes,bad", [(10, {0: "nan"}), (10, {8: "nan"}), (10, {4: "nan"}), (10, {c: "nan" for c in range(10)}), (4, {0: "nan", 3: "nan"}),
                                         (32, {c: "nan" for c in (4, 8, 12, 16, 20)}), (32, {c: "nan" for c in range(8, 16)}), (17, {16: "nan"}),
                                         (10, {c: "-inf" for c in range(10)}), (10, {0: "-inf", 1: "nan", 8: "nan", 9: "inf"}), (9, {3: "inf", 8: "inf"})])
@pytest.mark.parametrize("rows,cap", [(416 * UNITS + 31, 416 * UNITS + 31), (100 * UNITS, CAP), (63 * UNITS, CAP), (20 * UNITS, CAP), (100 * UNITS, 128 * UNITS),
                                      (50, 60)])
def test_labels_of_missing_logits(rows, cap, classes, bad):
    """Logits that are NaN or infinite: the label does not follow from where the row stands (full pass and tile, low pass, tiles of two and
    one row blocks, the tiles of shorter lists), and neither half of the classes hides the other's."""
    import numpy as np
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(classes + len(bad))
    dims = (64, 160, 96, classes)
    mlp = _model(g, dims, True)
    for c, v in bad.items():
        mlp.b3[c] = float(v)
    feat = torch.randn((cap, 64), device=DEV, generator=g)
    idx = torch.arange(cap, device=DEV, dtype=torch.int32)
    logits = torch.empty((cap, classes), device=DEV)
    labels = torch.full((cap,), -1, dtype=torch.int16, device=DEV)
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(cap, 0, 0, *dims[:3]))
    torch.cuda.synchronize()
    ctx.sf_slow_infer(mlp, idx, count, labels, feat=feat, logits=logits)
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(logits[:rows]).all(0).cpu(), torch.tensor([bad.get(c) == "nan" for c in range(classes)]))
    assert np.array_equal(labels[:rows].cpu().numpy(), _labels(logits[:rows]))


def test_values_past_the_finite():
    """Infinite and missing inputs stay with their own rows, and a hidden NaN counts as zero (the input map keeps NaN, relu does not)."""
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    n, dims = CAP + 1000, (64, 256, 128, 10)
    mlp = _model(g, dims, True)
    feat = torch.randn((n, 64), device=DEV, generator=g)
    idx = torch.arange(n, device=DEV, dtype=torch.int32)
    count = torch.tensor([n], dtype=torch.int32, device=DEV)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 0, 0, *dims[:3]))
    outs = []
    for bad in (False, True):
        x = feat.clone()
        if bad:
            x[5, 3], x[64, 0], x[40000 % n, 63] = float("inf"), float("nan"), float("-inf")
        logits = torch.empty((n, 10), device=DEV)
        labels = torch.empty(n, dtype=torch.int16, device=DEV)
        torch.cuda.synchronize()
        ctx.sf_slow_infer(mlp, idx, count, labels, feat=x, logits=logits)
        torch.cuda.synchronize()
        outs.append(logits)
    same = torch.ones(n, dtype=torch.bool, device=DEV)
    same[[5, 64, 40000 % n]] = False
    assert torch.equal(outs[0][same], outs[1][same])
    # every hidden value of the first layer is NaN, so zero; the rest follows from the biases
    h = torch.relu(mlp.b2.double()).float().to(torch.bfloat16).double()
    want = h @ mlp.w3.double().t() + mlp.b3.double()
    assert float((outs[1][64].double() - want).abs().max()) < 1e-2
    assert torch.isfinite(outs[1]).all()
