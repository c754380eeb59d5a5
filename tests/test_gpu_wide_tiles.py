"""The slow model of any width (one kernel per layer) where its tiles end: rows around the tile height, more row
blocks than compute units, a last row block or column block that is nearly empty, input widths around the slabs of
64 that decide whether a row block stays in shared memory, header bits in whole bytes and not, several chunks of rows.
Logits against the same model in 64 bits with the hidden activations rounded to bfloat16; labels: the arg-max of the
logits that came out."""
import pytest

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _model(g, dims, mapped):
    import torch
    import paper_2402_03694_amd as sf
    p = []
    for n_out, k in zip(dims[1:], dims[:-1]):
        p.append(((torch.rand((n_out, k), device=DEV, generator=g) * 2 - 1) * (6.0 / (n_out + k)) ** 0.5).to(torch.bfloat16))
        p.append(torch.rand(n_out, device=DEV, generator=g) * 0.2 - 0.1)
    mu = torch.randn(dims[0], device=DEV, generator=g) if mapped else None
    inv = torch.rand(dims[0], device=DEV, generator=g) + 0.5 if mapped else None
    return sf.DeviceMlp(dims, sf.SF_BF16, *p, mu=mu, inv_sigma=inv)


def _reference(mlp, x):
    import torch
    bf = lambda t: t.to(torch.float32).to(torch.bfloat16).double()
    if mlp.mu is not None:
        x = ((x - mlp.mu) * mlp.inv_sigma).clamp(-mlp.clamp, mlp.clamp)
    h = bf(x)
    for w, b in ((mlp.w1, mlp.b1), (mlp.w2, mlp.b2)):
        h = bf(torch.relu(h @ w.double().t() + b.double()))
    return h @ mlp.w3.double().t() + mlp.b3.double()


def _check(mlp, ref, logits, labels, idx, n):
    import torch
    rows = ref.shape[0]
    diff = (logits[:rows].double() - ref).abs()
    # a sum in binary32 that falls on the other side of a bfloat16 rounding moves one hidden value by 2^-8 of itself;
    # of 1,000 such values with random signs a few do, far below 1 % of a logit's size
    assert float(diff.max()) <= 1e-2 * float(ref.abs().max()), float(diff.max())
    assert torch.isnan(logits[rows:]).all()               # rows past the count are not written
    want = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    want[idx.long()] = logits[:rows].argmax(1).to(torch.int16)
    assert torch.equal(labels, want)


@pytest.mark.parametrize("rows,dims,ordered,small_ws", [
    (1, (64, 520, 600, 3), True, False), (127, (63, 1056, 608, 10), True, False), (128, (65, 513, 1056, 33), False, False),
    (129, (128, 1024, 64, 10), True, False), (255, (192, 100, 1024, 32), True, False), (257, (193, 520, 130, 2), True, True),
    (1000, (256, 700, 190, 7), True, True), (1025, (40, 64, 2048, 10), True, False), (32768, (64, 1024, 576, 10), True, False),
    (32769, (128, 1030, 1024, 32), True, False), (70001, (96, 640, 1100, 5), True, False), (2000, (513, 40, 50, 4), False, False)])
def test_feature_rows(rows, dims, ordered, small_ws):
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + dims[1])
    n = rows + 77
    mlp = _model(g, dims, mapped=True)
    feat = torch.randn((n, dims[0] + dims[0] % 4), device=DEV, generator=g)
    idx = torch.randperm(n, device=DEV, generator=g)[:rows].sort().values.to(torch.int32)
    ws = sf.sf_workspace_bytes(256 if small_ws else n, 0, 0, *dims[:3])
    ctx = sf.ServeFlow(ws)
    if ordered and dims[3] <= 32:
        ctx.sf_mlp_order(mlp)
    logits = torch.full((n, dims[3]), float("nan"), device=DEV)
    labels = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    ctx.sf_slow_infer(mlp, torch.cat([idx, idx[:1].expand(n - rows)]).contiguous(), count, labels, feat=feat, logits=logits)
    torch.cuda.synchronize()
    _check(mlp, _reference(mlp, feat[idx.long(), :dims[0]]), logits, labels, idx, n)


@pytest.mark.parametrize("rows,raw_pkts,raw_bits,hidden", [
    (1, 1, 96, (64, 64)), (130, 2, 96, (520, 64)), (257, 3, 64, (64, 520)), (300, 10, 480, (1024, 512)), (999, 5, 31, (200, 100)),
    (513, 9, 12, (96, 40)), (33000, 4, 96, (600, 64))])
def test_header_bits(rows, raw_pkts, raw_bits, hidden):
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + raw_bits)
    n, words = rows + 33, (raw_bits + 31) // 32
    dims = (raw_pkts * raw_bits, *hidden, 10)
    mlp = _model(g, dims, mapped=False)
    lens = torch.randint(0, raw_pkts + 3, (n,), device=DEV, generator=g)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    off[1:] = lens.cumsum(0)
    m = int(off[-1])
    hdr = torch.randint(-2 ** 31, 2 ** 31, (max(m, 1), words), dtype=torch.int32, device=DEV, generator=g)
    z = lambda t: torch.zeros(max(m, 1), dtype=t, device=DEV)
    pk = sf.DevicePackets(off.to(torch.int32), z(torch.int16), z(torch.float32), z(torch.uint8), hdr)
    idx = torch.randperm(n, device=DEV, generator=g)[:rows].sort().values.to(torch.int32)
    # bit b of a packet is bit 7 - b % 8 of byte b / 8 of its little-endian words
    b = torch.arange(raw_bits, device=DEV)
    bits = (hdr[:, b // 32].long() >> (b % 32 // 8 * 8 + 7 - b % 8)) & 1
    at = off[idx.long()][:, None] + torch.arange(raw_pkts, device=DEV)
    have = torch.arange(raw_pkts, device=DEV) < lens[idx.long()][:, None]
    x = (bits[at.clamp(max=max(m, 1) - 1)] * have[:, :, None]).reshape(rows, -1).float()
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 0, 0, *dims[:3]))
    ctx.sf_mlp_order(mlp)
    logits = torch.full((n, 10), float("nan"), device=DEV)
    labels = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    ctx.sf_slow_infer(mlp, torch.cat([idx, idx[:1].expand(n - rows)]).contiguous(), count, labels, raw_src=pk, raw_pkts=raw_pkts,
                      raw_bits=raw_bits, logits=logits)
    torch.cuda.synchronize()
    _check(mlp, _reference(mlp, x), logits, labels, idx, n)
