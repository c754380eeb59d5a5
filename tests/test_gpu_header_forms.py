"""Header bits as the wide layer's input, for every way their bits can lie: whole bytes, 9 bits and more that end inside a byte
(features that straddle a byte, a word, the end of a packet, and a word and the end of a packet at once), 1 to 7 bits
(features of two to eight packets); more words than the bits need, more and fewer packets than the features take, K in
the slab buffers and streamed, several tiles.  Against the same model in 64 bits; the bits themselves are exact."""
import pytest

from test_gpu_wide_tiles import DEV, _check, _model, _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,pkts,rows,extra", [
    (1, 9, 130, 0), (1, 230, 300, 1), (2, 31, 129, 0), (2, 130, 257, 0), (3, 40, 140, 0), (3, 75, 300, 1), (4, 30, 130, 0), (5, 70, 40000, 0),
    (6, 45, 257, 0), (7, 25, 200, 2), (7, 30, 40000, 0), (8, 24, 130, 0), (9, 20, 129, 0), (15, 30, 257, 0), (25, 3, 130, 0), (31, 9, 300, 1),
    (33, 5, 130, 0), (34, 9, 40000, 0), (57, 3, 257, 0), (63, 7, 300, 0), (95, 2, 130, 1), (100, 1, 129, 0), (255, 2, 130, 0),
    (257, 3, 257, 0), (477, 10, 300, 0), (1023, 2, 200, 0), (1000, 1, 130, 1), (1070, 2, 130, 0)])
def test_forms(bits, pkts, rows, extra):
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(1000 * bits + pkts)
    n, words = rows + 13, (bits + 31) // 32 + extra
    dims = (pkts * bits, 1024 if rows > 1000 else 600, 64, 10)
    mlp = _model(g, dims, mapped=False)
    lens = torch.randint(0, pkts + 3, (n,), device=DEV, generator=g)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    off[1:] = lens.cumsum(0)
    m = int(off[-1])
    hdr = torch.randint(-2 ** 31, 2 ** 31, (max(m, 1), words), dtype=torch.int32, device=DEV, generator=g)
    z = lambda t: torch.zeros(max(m, 1), dtype=t, device=DEV)
    pk = sf.DevicePackets(off.to(torch.int32), z(torch.int16), z(torch.float32), z(torch.uint8), hdr)
    idx = torch.randperm(n, device=DEV, generator=g)[:rows].sort().values.to(torch.int32)
    # bit b of a packet is bit 7 - b % 8 of byte b / 8 of its little-endian words
    b = torch.arange(bits, device=DEV)
    value = (hdr[:, b // 32] >> (b % 32 // 8 * 8 + 7 - b % 8).to(torch.int32)) & 1
    at = off[idx.long()][:, None] + torch.arange(pkts, device=DEV)
    have = torch.arange(pkts, device=DEV) < lens[idx.long()][:, None]
    x = (value[at.clamp(max=max(m, 1) - 1)] * have[:, :, None]).reshape(rows, -1).float()
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(n, 0, 0, *dims[:3]))
    ctx.sf_mlp_order(mlp)
    logits = torch.full((n, 10), float("nan"), device=DEV)
    labels = torch.full((n,), -1, dtype=torch.int16, device=DEV)
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    ctx.sf_slow_infer(mlp, torch.cat([idx, idx[:1].expand(n - rows)]).contiguous(), count, labels, raw_src=pk, raw_pkts=pkts, raw_bits=bits,
                      logits=logits)
    torch.cuda.synchronize()
    _check(mlp, _reference(mlp, x), logits, labels, idx, n)


@pytest.mark.parametrize("bits", [1, 2, 3, 4, 5, 6, 7, 8, 9, 23, 33, 39, 64, 101])
def test_every_feature(bits):
    """A first layer that copies single input features: every feature of every packet comes out as it went in."""
    import torch
    import paper_2402_03694_amd as sf
    g = torch.Generator(device=DEV)
    g.manual_seed(bits)
    pkts = max(2, 300 // bits)
    k, rows, words = pkts * bits, 128, (bits + 31) // 32
    hdr = torch.randint(-2 ** 31, 2 ** 31, (rows * pkts, words), dtype=torch.int32, device=DEV, generator=g)
    z = lambda t: torch.zeros(rows * pkts, dtype=t, device=DEV)
    pk = sf.DevicePackets(torch.arange(0, rows * pkts + 1, pkts, dtype=torch.int32, device=DEV), z(torch.int16), z(torch.float32), z(torch.uint8), hdr)
    b = torch.arange(bits, device=DEV)
    x = ((hdr[:, b // 32] >> (b % 32 // 8 * 8 + 7 - b % 8).to(torch.int32)) & 1).reshape(rows, k)
    # the identity twice, then sums of eight features each with weights 1 .. 128: exact in bfloat16 and binary32
    bf = lambda t: t.to(torch.bfloat16).contiguous()
    eye = torch.eye(k, device=DEV)
    idx = torch.arange(rows, dtype=torch.int32, device=DEV)
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(rows, 0, 0, k, k, k))
    count = torch.tensor([rows], dtype=torch.int32, device=DEV)
    for first in range(0, k, 8 * 32):
        w3 = torch.zeros((32, k), device=DEV)
        for f in range(first, min(k, first + 8 * 32)):
            w3[(f - first) // 8, f] = 2.0 ** (f % 8)
        mlp = sf.DeviceMlp((k, k, k, 32), sf.SF_BF16, bf(eye), torch.zeros(k, device=DEV), bf(eye), torch.zeros(k, device=DEV), bf(w3),
                           torch.zeros(32, device=DEV))
        logits = torch.full((rows, 32), float("nan"), device=DEV)
        labels = torch.full((rows,), -1, dtype=torch.int16, device=DEV)
        ctx.sf_slow_infer(mlp, idx, count, labels, raw_src=pk, raw_pkts=pkts, raw_bits=bits, logits=logits)
        torch.cuda.synchronize()
        assert torch.equal(logits.double(), x.double() @ w3.double().t())
