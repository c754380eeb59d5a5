"""The work this library is measured on: whole passes through its public entry points, over the range of batch
sizes, flow lengths, models and gates that its workloads (synth/configs.py) and tests use.

A case is a dict of plain values.  `path` says which calls a pass makes:
  classify  sf_classify: features, forest, gate and slow model behind one call (flow statistics or header bits)
  steps     sf_featurize, sf_fast_infer, sf_route, sf_slow_infer one after the other, the feature matrix kept
  cascade   three tiers: features, a decision tree on every flow, the forest on the tree's uncertain flows, the
            slow model on the forest's
  boosted   features, boosted trees with a real-valued score, the gate on it, the slow model
  join      a few steps of the queue join, each followed by the slow model on the pairs it found

Sizes of a case: `flows` per batch; `packets` per flow (0: ragged, geometric with mean about ten); `windows`: packet
depths of the feature windows; `trees`, `depth`, `classes`; `hidden`: the slow model's two widths; `dtype`; `target`:
the share of flows the gate hands on (reached as closely as an integer score allows); `gate`: one threshold for all
classes or one per class; `raw`: the slow model reads this many header bits of each packet instead of the statistics.
"""
import math

import torch

import paper_2402_03694_amd as sf

DEV = "cuda:0"
CALIB = 4096           # flows whose features fix split thresholds and the input map (as the workloads do)
GATE_SAMPLE = 1 << 16  # flows the gate's thresholds are taken from
GEOM_P, MAX_PKTS = 0.1, 64
JOIN_STEPS, JOIN_TIMEOUT = 4, 1


def _case(name, path, flows, packets, windows, trees, depth, classes, hidden, dtype="bf16", target=0.25, gate="one", raw=0,
          tree0=0, score="lc"):
    c = {"path": path, "flows": flows, "packets": packets, "windows": windows, "trees": trees, "depth": depth,
         "classes": classes, "hidden": hidden, "dtype": dtype, "target": target, "gate": gate, "raw": raw, "tree0": tree0,
         "score": score}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a handful of flows as they come off the wire: what one call costs when the batch is next to nothing
        _case("burst", "classify", 97, 0, "8,16", 100, 12, 10, "512,512"),
        # the small binary32 workload: 4,096 flows of 8 packets, nearly all of them handed on
        _case("small", "classify", 4096, 8, "8", 16, 8, 4, "128,128", dtype="f32", target=1.0),
        # the main workload: a million flows of 16 packets, thresholds per class that hand on a quarter
        _case("main", "classify", 1 << 20, 16, "8,16", 100, 12, 10, "512,512", gate="class"),
        # the same models through the four calls, an odd number of ragged flows
        _case("steps", "steps", 250007, 0, "8,16", 100, 12, 10, "512,512"),
        # an ordinary batch with nothing on a round number: three windows, odd depths and widths
        _case("odd", "steps", 20011, 0, "3,9,20", 150, 9, 7, "300,200"),
        # the slow model on raw header bits: 10 packets x 480 bits
        _case("header", "classify", 1 << 20, 10, "5,10", 100, 10, 10, "1024,512", target=0.2, raw=480),
        # streaming micro-batches: ragged flows of 1 to 64 packets
        _case("stream", "classify", 65536, 0, "8,64", 200, 10, 16, "1024,1024", target=0.3),
        # the large workload: four million flows of 32 packets, 500 trees, wide slow model
        _case("sweep", "classify", 1 << 22, 32, "8,16,24,32", 500, 10, 32, "2048,2048"),
        # three tiers
        _case("cascade", "cascade", 1 << 20, 16, "8,16", 100, 12, 10, "512,512", target=0.18, tree0=10),
        # boosted trees, 20 rounds x 10 classes, gated by the entropy of their softmax
        _case("boosted", "boosted", 1 << 20, 16, "8,16", 200, 8, 10, "512,512", score="entropy"),
        # a smaller boosted model on a smaller, ragged batch, least-confidence score
        _case("boosted_small", "boosted", 10007, 0, "8", 60, 6, 6, "128,64"),
        # the two queues in front of the slow model, at the rate at which the main workload hands flows on
        _case("join", "join", 179427, 16, "8,16", 0, 0, 10, "512,512", target=1.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["classify", "classify", "classify", "steps", "steps", "cascade", "boosted", "join"])
    n_win = rng.choice([1, 2, 2, 2, 3, 4])
    top = rng.choice([5, 8, 10, 16, 16, 20, 32, 64])
    if path == "boosted":
        n_win = min(n_win, 3)
    n_win = min(n_win, top)
    windows = sorted(rng.sample(range(1, top), n_win - 1) + [top]) if rng.random() < 0.5 else [top * (k + 1) // n_win for k in range(n_win)]
    packets = rng.choice([0, 0, top, min(64, top + rng.randrange(8))])
    if path == "join":
        return _case(None, "join", _log(rng, 300, 300000), 16, "8,16", 0, 0, rng.randrange(2, 33), "%d,%d" % (_log(rng, 32, 1024), _log(rng, 32, 1024)),
                     target=1.0)
    raw = 0
    if path == "classify" and rng.random() < 0.25:
        raw, packets = rng.choice([96, 480, 352]), rng.choice([0, 10])
    flows = _log(rng, 1, 300000 if raw or top > 16 else 1000000)
    classes = rng.randrange(2, 33) if path != "boosted" else rng.randrange(2, 17)
    trees = _log(rng, 5, 300)
    if path == "boosted":
        trees = max(classes, trees // classes * classes)
    dtype = "f32" if not raw and flows <= 20000 and rng.random() < 0.3 else "bf16"
    widest = 256 if dtype == "f32" else 1024
    return _case(None, path, flows, packets, ",".join(str(w) for w in windows), trees, rng.randrange(4, 13), classes,
                 "%d,%d" % (_log(rng, 32, widest), _log(rng, 32, widest)), dtype=dtype, target=round(rng.uniform(0.03, 0.6), 3),
                 gate=rng.choice(["one", "class"]) if path in ("classify", "steps") else "one", raw=raw,
                 tree0=rng.randrange(4, 13) if path == "cascade" else 0, score=rng.choice(["lc", "entropy"]))


# ---- inputs ------------------------------------------------------------------------------------------------------


def _lens(case):
    windows = [int(w) for w in case["windows"].split(",")]
    hidden = [int(w) for w in case["hidden"].split(",")]
    return windows, hidden


def _packets(case, g, n):
    """Packet records with the workloads' distributions: sizes in three modes, log-normal times, fair directions."""
    if case["packets"]:
        lens = torch.full((n,), case["packets"], dtype=torch.int64, device=DEV)
    else:
        lens = torch.empty(n, device=DEV).geometric_(GEOM_P, generator=g).clamp_(1, MAX_PKTS).to(torch.int64)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=off[1:])
    m = int(off[-1])
    mode = torch.rand(m, device=DEV, generator=g)
    u = torch.rand(m, device=DEV, generator=g)
    size = torch.where(mode < 0.6, 40 + (u * 61).floor(), torch.where(mode < 0.85, 500 + (u * 501).floor(), torch.full_like(u, 1500.0)))
    iat = torch.exp(torch.randn(m, device=DEV, generator=g) * 2.0 - 6.0)
    direction = (torch.rand(m, device=DEV, generator=g) < 0.5).to(torch.uint8)
    hdr = None
    if case["raw"]:
        words = (case["raw"] + 31) // 32
        rand = lambda: torch.randint(-2 ** 31, 2 ** 31, (m, words), dtype=torch.int32, device=DEV, generator=g)
        hdr = rand()                                     # every bit set with probability 77 / 256 = 0.3008
        for bit in (0, 1, 1, 0, 0, 1, 0):                # binary 0.01001101, from its last digit up
            hdr = (hdr | rand()) if bit else (hdr & rand())
        pattern = torch.randint(-2 ** 31, 2 ** 31, (case["classes"], 2), dtype=torch.int32, device=DEV, generator=g)
        hidden_class = torch.randint(0, case["classes"], (n,), device=DEV, generator=g)
        hdr[:, :2] = pattern[torch.repeat_interleave(hidden_class, lens)]  # fields that are the same for a whole class
    return sf.DevicePackets(off.to(torch.int32), size.to(torch.int16), iat, direction, hdr)


def _splits(g, trees, depth, n_feat, sample):
    n_int = (1 << depth) - 1
    feat = torch.randint(0, n_feat, (trees, n_int), device=DEV, generator=g)
    row = torch.randint(0, sample.shape[0], (trees, n_int), device=DEV, generator=g)
    return feat.to(torch.int16), sample[row, feat].contiguous()


def _forest(case, g, n_feat, sample):
    nf, nt = _splits(g, case["trees"], case["depth"], n_feat, sample)
    leaf = torch.randint(0, case["classes"], (case["trees"], 1 << case["depth"]), device=DEV, generator=g).to(torch.uint8)
    return sf.DeviceForest(case["trees"], case["depth"], case["classes"], n_feat, nf, nt, leaf)


def _boosted(case, g, n_feat, sample):
    nf, nt = _splits(g, case["trees"], case["depth"], n_feat, sample)
    value = torch.randn((case["trees"], 1 << case["depth"]), device=DEV, generator=g) * 0.5
    base = torch.rand(case["classes"], device=DEV, generator=g) - 0.5
    return sf.DeviceGbdt(case["trees"], case["depth"], case["classes"], n_feat, nf, nt, value, base)


def _tree(case, g, n_feat, sample):
    """Leaves with a few dozen samples each, the majority class holding 15 to 100 % of them."""
    nf, nt = _splits(g, 1, case["tree0"], n_feat, sample)
    n_leaf, c = 1 << case["tree0"], case["classes"]
    total = 15 + torch.randint(20, 70, (n_leaf,), device=DEV, generator=g)
    share = 0.15 + 0.85 * torch.rand(n_leaf, device=DEV, generator=g)
    count = ((1 - share) * total / max(c - 1, 1)).floor()[:, None].repeat(1, c)
    major = torch.randint(0, c, (n_leaf, 1), device=DEV, generator=g)
    count.scatter_(1, major, (share * total).ceil()[:, None])
    return sf.DeviceTree(case["tree0"], c, n_feat, nf[0].contiguous(), nt[0].contiguous(), count.to(torch.int16))


def _mlp(case, g, n_in, sample):
    _, hidden = _lens(case)
    dims = (n_in, hidden[0], hidden[1], case["classes"])
    bf = case["dtype"] == "bf16"

    def layer(n_out, k):
        a = math.sqrt(6.0 / (n_out + k))
        w = (torch.rand((n_out, k), device=DEV, generator=g) * 2 - 1) * a
        return (w.to(torch.bfloat16) if bf else w), torch.rand(n_out, device=DEV, generator=g) * 0.2 - 0.1

    w = [x for k in range(3) for x in layer(dims[k + 1], dims[k])]
    mu = inv = None
    if sample is not None:
        mu, sd = sample.double().mean(0), sample.double().std(0, unbiased=False)
        mu, inv = mu.float(), torch.where(sd > 0, 1.0 / sd, torch.ones_like(sd)).float()
    return sf.DeviceMlp(dims, sf.SF_BF16 if bf else sf.SF_F32, *w, mu=mu, inv_sigma=inv)


def _gate(case, ctx, g, top, pred):
    """Thresholds for the target share: one for all classes, or one per class (Algorithm 2 on drawn true labels)."""
    t, c, n = case["trees"], case["classes"], int(top.shape[0])
    if case["gate"] == "one":
        if case["target"] >= 1.0:
            return sf.sf_vmin_from_theta(0.75, t)
        vmin, _ = sf.sf_vmin_for_target(ctx.sf_score_histogram(top, t), t, case["target"])
        return vmin
    a = torch.rand(c, device=DEV, generator=g) * 0.7 - 0.6
    b = torch.rand(c, device=DEV, generator=g) * 4 + 3
    p = pred.long()
    right = torch.rand(n, device=DEV, generator=g) < (a[p] + b[p] * top / t).clamp(0.02, 0.98)
    other = (p + 1 + torch.randint(0, max(c - 1, 1), (n,), device=DEV, generator=g)) % c
    truth = torch.where(right, p, other).to(torch.int16)
    vmin, _ = sf.sf_per_class_thresholds(ctx.sf_class_score_histogram(top, pred, truth, t, c), t, c, case["target"])
    return vmin


def _prepare_join(case, g):
    """Arrivals of JOIN_STEPS steps: of a flow's two records 70 % come in the same step, 20 % one step apart, 10 % alone."""
    n, c = case["flows"], case["classes"]
    cap = max(4, (4 * n - 1).bit_length())
    _, hidden = _lens(case)
    total = n * JOIN_STEPS
    feat = torch.randn((total, 64), device=DEV, generator=g)
    mlp = _mlp(case, g, 64, feat[:CALIB])
    ctx = sf.ServeFlow(max(sf.sf_join_workspace_bytes(cap), sf.sf_workspace_bytes(2 * n, 0, 0, 64, *hidden)))
    ctx.sf_mlp_order(mlp)
    ids = torch.randperm(total, device=DEV, generator=g) + 1
    ids = ids * 0x1E3779B97F4A7C15  # distinct 64-bit flow numbers (an odd multiplier), wrapped
    step3 = torch.arange(total, device=DEV) // n
    u = torch.rand(total, device=DEV, generator=g)
    step2 = torch.where(u < 0.7, step3, torch.where(u < 0.8, step3 + 1, torch.where(u < 0.9, step3 - 1, torch.full_like(step3, -1))))
    late_row = torch.randperm(total, device=DEV, generator=g).to(torch.int32)
    flow = torch.arange(total, device=DEV, dtype=torch.int32)
    batches = []
    for s in range(JOIN_STEPS):
        a, b = torch.nonzero(step3 == s)[:, 0], torch.nonzero(step2 == s)[:, 0]
        batches.append((ids[a].contiguous(), flow[a].contiguous(), ids[b].contiguous(), late_row[b].contiguous()))
    i32 = lambda m: torch.zeros(m, dtype=torch.int32, device=DEV)
    labels = torch.randint(0, c, (total,), device=DEV, generator=g).to(torch.int16)
    return {"case": case, "ctx": ctx, "mlp": mlp, "feat": feat, "table": sf.DeviceJoinTable(cap, DEV), "batches": batches, "now": 0,
            "pair_q3": i32(2 * n), "pair_q2": i32(2 * n), "n_pairs": [i32(1) for _ in range(JOIN_STEPS)], "stats": i32(4), "labels": labels}


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    if case["path"] == "join":
        return _prepare_join(case, g)
    windows, hidden = _lens(case)
    n, f, c, t = case["flows"], 32 * len(windows), case["classes"], case["trees"]
    n_in = 10 * case["raw"] if case["raw"] else f
    ctx = sf.ServeFlow(sf.sf_workspace_bytes(max(n, GATE_SAMPLE), t, case["depth"], n_in, *hidden))
    # the models come from a sample of flows drawn like the batch
    known = _packets(dict(case, raw=0), g, GATE_SAMPLE)
    feat_known = torch.empty((GATE_SAMPLE, f), dtype=torch.float32, device=DEV)
    ctx.sf_featurize(known, windows, feat_known)
    sample = feat_known[:CALIB]
    i16 = lambda m: torch.zeros(m, dtype=torch.int16, device=DEV)
    i32 = lambda m: torch.zeros(m, dtype=torch.int32, device=DEV)
    mlp = _mlp(case, g, n_in, None if case["raw"] else sample)
    ctx.sf_mlp_order(mlp)
    st = {"case": case, "ctx": ctx, "windows": windows, "mlp": mlp, "pred": i16(n), "labels": i16(n), "esc_idx": i32(n),
          "esc_count": i32(1), "logits": torch.zeros((n, c), dtype=torch.float32, device=DEV),
          "feat": torch.zeros((n, f), dtype=torch.float32, device=DEV)}
    pred, top = i16(GATE_SAMPLE), i16(GATE_SAMPLE)
    if case["path"] == "boosted":
        st["kind"] = sf.SF_SCORE_ENTROPY if case["score"] == "entropy" else sf.SF_SCORE_LC
        st["model"] = _boosted(case, g, f, sample)
        ctx.sf_gbdt_pack(st["model"])
        st["score"] = torch.zeros(n, dtype=torch.float32, device=DEV)
        score = torch.empty(GATE_SAMPLE, dtype=torch.float32, device=DEV)
        ctx.sf_gbdt_infer(feat_known, st["model"], st["kind"], pred, score)
        st["threshold"] = ctx.sf_score_quantiles(score, [1.0 - case["target"]])[0]
    else:
        n_feat = 32 if case["path"] == "cascade" else f  # a cascade's trees see the first window only
        st["model"] = _forest(case, g, n_feat, sample)
        ctx.sf_forest_pack(st["model"])
        ctx.sf_fast_infer(feat_known, st["model"], pred, top)
        st["vmin"] = _gate(case, ctx, g, top, pred)
        st["top"] = i16(n)
    if case["path"] == "cascade":
        st["tree"] = _tree(case, g, 32, sample)
        st.update(top0=i16(n), tot0=i16(n), idx0=i32(n), count0=i32(1))
    st["pk"] = _packets(case, g, n)
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    path = case["path"]
    if path == "join":
        now = st["now"]
        st["now"] = now + JOIN_STEPS + JOIN_TIMEOUT + 1  # by the next pass every record left waiting has timed out
        for s, (id3, row3, id2, row2) in enumerate(st["batches"]):
            ctx.sf_join_step(st["table"], now + s, JOIN_TIMEOUT, id3, row3, id2, row2, st["pair_q3"], st["pair_q2"], st["n_pairs"][s], st["stats"])
            ctx.sf_slow_infer_pairs(st["mlp"], st["feat"], st["pair_q2"], st["pair_q3"], st["n_pairs"][s], st["labels"])
        return {"labels": st["labels"], "n_pairs": st["n_pairs"], "stats": st["stats"]}
    pk, windows, feat, mlp, pred, labels = st["pk"], st["windows"], st["feat"], st["mlp"], st["pred"], st["labels"]
    esc_idx, esc_count, logits = st["esc_idx"], st["esc_count"], st["logits"]
    out = {"pred": pred, "labels": labels, "esc_idx": esc_idx, "esc_count": esc_count, "logits": logits}
    if path == "classify":
        raw = {"raw_pkts": 10, "raw_bits": case["raw"]} if case["raw"] else {}
        ctx.sf_classify(pk, windows, st["model"], st["vmin"], mlp, feat, pred, st["top"], esc_idx, esc_count, labels, logits=logits, **raw)
        out["top"] = st["top"]
        return out
    ctx.sf_featurize(pk, windows, feat)
    out["feat"] = feat
    if path == "steps":
        ctx.sf_fast_infer(feat, st["model"], pred, st["top"])
        ctx.sf_route(st["top"], pred, st["vmin"], esc_idx, esc_count)
        ctx.sf_slow_infer(mlp, esc_idx, esc_count, labels, feat=feat, logits=logits, pred=pred)
        out["top"] = st["top"]
    elif path == "boosted":
        ctx.sf_gbdt_infer(feat, st["model"], st["kind"], pred, st["score"])
        ctx.sf_route_score(st["score"], st["threshold"], esc_idx, esc_count)
        ctx.sf_slow_infer(mlp, esc_idx, esc_count, labels, feat=feat, logits=logits, pred=pred)
        out["score"] = st["score"]
    else:  # cascade: each tier's label stands until a later tier replaces it
        ctx.sf_fastest_infer(feat, st["tree"], labels, st["top0"], st["tot0"])
        ctx.sf_route_ratio(st["top0"], st["tot0"], 0.6, st["idx0"], st["count0"])
        ctx.sf_fast_infer_subset(feat, st["idx0"], st["count0"], st["model"], pred, st["top"], labels=labels)
        ctx.sf_route_subset(st["top"], pred, st["idx0"], st["count0"], st["vmin"], esc_idx, esc_count)
        ctx.sf_slow_infer(mlp, esc_idx, esc_count, labels, feat=feat, logits=logits)
        out.update(top=st["top"], top0=st["top0"], tot0=st["tot0"], idx0=st["idx0"], count0=st["count0"])
    return out


# ---- what a pass cannot do without ---------------------------------------------------------------------------------


def work(case):
    windows, hidden = _lens(case)
    n, f, c = case["flows"], 32 * len(windows), case["classes"]
    n_in = 10 * case["raw"] if case["raw"] else f
    el = 2 if case["dtype"] == "bf16" else 4
    dims = (n_in, hidden[0], hidden[1], c)
    per_row = sum(dims[k] * dims[k + 1] for k in range(3))
    if case["path"] == "join":
        # arrivals (12 bytes a record), one input row and one label for each pair
        records, pairs = 1.8 * JOIN_STEPS * n, 0.85 * JOIN_STEPS * n
        return {"bytes": 12 * records + (4 * 64 + 2) * pairs + el * per_row, "flops": 2.0 * per_row * pairs}
    mean_of = lambda most: case["packets"] and min(case["packets"], most) or (1 - (1 - GEOM_P) ** min(most, MAX_PKTS)) / GEOM_P
    nodes = case["trees"] * ((1 << case["depth"]) - 1)
    share = case["target"]
    out_esc = 4 + 4 * c                                    # list entry and logits of a flow handed on
    visits = float(n) * case["trees"] * case["depth"]
    per_flow = 7 * mean_of(windows[-1]) + 4 + 6            # packets and offset in; label, prediction and score out
    if case["path"] != "classify":
        per_flow += 4 * f                                  # the feature matrix is an output
    if case["path"] == "cascade":
        visits = float(n) * (case["tree0"] + 0.5 * case["trees"] * case["depth"])
        share = 0.5 * case["target"]
        per_flow += 6
    if case["path"] == "boosted":
        per_flow += 2
    if case["raw"]:
        out_esc += mean_of(10) * ((case["raw"] + 31) // 32) * 4
    model = nodes * 6 + case["trees"] * (1 << case["depth"]) + el * per_row
    return {"bytes": n * (per_flow + share * out_esc) + model, "flops": 2.0 * per_row * share * n + visits}


def tolerance(case):
    """Against the slow model in 64 bits on the same rows the logits are off by at most 2.6e-7 (largest 2.3e-6) for
    binary32 models, and for bfloat16 models, whose hidden activations are bfloat16, by 2.6e-3 (largest 4e-2) with
    0.4 % of the slow labels falling on the other side of a tie; about four times that is stated.  Everything else
    (features, votes, scores, lists) is far inside these."""
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5, "differ": 1e-4}
    return {"rel": 1e-2, "max": 0.15, "differ": 5e-3}
