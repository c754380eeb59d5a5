"""The wide layer where a block walks several row blocks, each through all its column blocks, with K streamed through the
slab buffers: feature rows and header bits (512 row blocks, so that no compute unit gets a tile more than in the other
order), with a last row block that is full, nearly empty and missing."""
import pytest

from test_gpu_wide_tiles import DEV, _check, _model, _reference

pytestmark = pytest.mark.gpu

FULL = 2 * 256 * 128                      # two row blocks for every compute unit


@pytest.mark.parametrize("rows,dims,raw_bits", [(FULL, (256, 1024, 64, 10), 0), (FULL - 127, (321, 600, 40, 7), 0), (FULL - 128, (200, 520, 64, 5), 0),
                                                (FULL, (4 * 96, 1024, 64, 10), 96), (FULL - 127, (7 * 40, 560, 40, 10), 40)])
def test_walk(rows, dims, raw_bits):
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + dims[0])
    n = rows + 50
    mlp = _model(g, dims, mapped=not raw_bits)
    idx = torch.randperm(n, device=DEV, generator=g)[:rows].sort().values.to(torch.int32)
    if raw_bits:
        pkts, words = dims[0] // raw_bits, (raw_bits + 31) // 32
        hdr = torch.randint(-2 ** 31, 2 ** 31, (n * pkts, words), dtype=torch.int32, device=DEV, generator=g)
        z = lambda t: torch.zeros(n * pkts, dtype=t, device=DEV)
        pk = sf.DevicePackets(torch.arange(0, n * pkts + 1, pkts, dtype=torch.int32, device=DEV), z(torch.int16), z(torch.float32), z(torch.uint8), hdr)
        b = torch.arange(raw_bits, device=DEV)
        x = ((hdr[:, b // 32] >> (b % 32 // 8 * 8 + 7 - b % 8).to(torch.int32)) & 1).reshape(n, -1)[idx.long()].float()
        kw = dict(raw_src=pk, raw_pkts=pkts, raw_bits=raw_bits)
    else:
        feat = torch.randn((n, dims[0] + dims[0] % 4), device=DEV, generator=g)
        x = feat[idx.long(), :dims[0]]
        kw = dict(feat=feat)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 0, 0, *dims[:3]))
    ctx.sf_mlp_order(mlp)
    logits = torch.full((n, dims[3]), float("nan"), device=DEV)
    labels = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    ctx.sf_slow_infer(mlp, torch.cat([idx, idx[:1].expand(n - rows)]).contiguous(), count, labels, logits=logits, **kw)
    torch.cuda.synchronize()
    _check(mlp, _reference(mlp, x), logits, labels, idx, n)
