"""What a user of absb runs, as cases that can be timed: the decode step in the sizes and modes it is
used in, a decode loop that keeps its store current, and the store build of the prefill side.

A case is a dict of plain values.  `prepare` makes on the GPU what a serving program holds before the
call (paged caches, queries, the centroid store, page table, workspace); `run` is one pass through the
binding's entry points.  Kinds:

  step      one absb_decode_fused call: a decode step of one layer
  generate  a decode loop: `tokens` new tokens through `layers` layers, absb_append_token and
            absb_decode_fused per token and layer, the context lengths growing on host and device
  build     one absb_build_centroids call: the store of a context, after prefill

Ranges that the cases stand for (`draw` spreads over them): contexts of 512 tokens to 512 Ki per
request, 1 to 16 requests of equal or mixed lengths, 2 to 16 KV heads in groups of 1 to 8, f16 and bf16,
pages of 16 to 128 tokens, per-head block sizes 8 to 128, budgets of 128 to 16384 tokens, of a few
percent of the context, or of all of it.
"""
import math
import random

import numpy as np
import torch

from paper_2605_12110_amd import absb

D = 128  # head dimension
SELECTION = {"group": absb.SELECT_GROUP, "per_query_head": absb.SELECT_PER_QUERY_HEAD, "group_max": absb.SELECT_GROUP_MAX}
REPR = {"mean": absb.REPR_MEAN, "minmax": absb.REPR_MINMAX}
DTYPE = {"f16": (absb.F16, torch.float16), "bf16": (absb.BF16, torch.bfloat16)}


def case(**kw):
    """A case with the defaults of a Llama-3.1-8B-shaped layer; lengths are drawn from [len_lo, len_hi] and
    block sizes per KV head from `sizes`, by `shape_seed` (shapes belong to the case, values to the seed)."""
    c = dict(kind="step", dtype="f16", batch=1, q_heads=32, kv_heads=8, page=64, len_lo=4096, len_hi=4096,
             sizes="8,16,32,64", shape_seed=1, budget=512, budget_pct=0, select="group", repr="mean", sink=0,
             recent=0, keys="zipf", list=False, tokens=0, layers=1)
    c.update(kw)
    return c


def listed():
    return [
        # a short chat turn: one request, 4K context; launch and hand-over latency is all there is
        case(name="step_4k_b1", keys="planted"),
        # the headline of this repository's benchmark: one request at 128K, 8B-shaped layer
        case(name="step_128k_b1", len_lo=131072, len_hi=131072, sizes="8,16,32,64,128", budget=4096),
        # a batch of equal 32K contexts whose keys are of low rank
        case(name="step_32k_b8", dtype="bf16", batch=8, len_lo=32768, len_hi=32768, sizes="16,32,64", budget=2048, keys="lowrank"),
        # a full serving batch of ragged contexts, 8K to 128K, five query heads per KV head, 3 % budget
        case(name="step_mixed_b16", dtype="bf16", batch=16, q_heads=40, len_lo=8192, len_hi=131072, sizes="16,32,64",
             budget=0, budget_pct=3, keys="planted"),
        # one very long document, of odd length; the caller wants the list of selected blocks as well
        case(name="step_256k_b1", len_lo=262143, len_hi=262143, sizes="8,16,32,64,128", budget=4096, list=True),
        # a budget that covers the context: the dense reference pass of a calibration
        case(name="step_dense_128k", len_lo=131072, len_hi=131072, sizes="8,16,32,64,128", budget=131072),
        # max-min pooling with sink and recent tokens always kept
        case(name="step_minmax_sink_b4", batch=4, len_lo=20000, len_hi=65536, sizes="16,32,64", budget=2048, repr="minmax",
             sink=64, recent=256),
        # every query head selects for itself
        case(name="step_perquery_b8", dtype="bf16", batch=8, len_lo=32768, len_hi=32768, sizes="16,32,64", budget=2048,
             select="per_query_head"),
        # ranking by the group's best head, uniform blocks of one small page, larger budget
        case(name="step_groupmax_b4", batch=4, len_lo=65536, len_hi=65536, page=16, sizes="16", budget=8192, select="group_max"),
        # a decode loop: four requests, eight tokens through four layers, the store kept current
        case(name="generate_b4", kind="generate", dtype="bf16", batch=4, len_lo=3000, len_hi=24000, sizes="16,32,64",
             budget=2048, tokens=8, layers=4),
        # the store of one 128K context, after its prefill
        case(name="build_128k_b1", kind="build", len_lo=131072, len_hi=131072, sizes="8,16,32,64,128"),
        # the stores of a ragged batch at once
        case(name="build_mixed_b16", kind="build", dtype="bf16", batch=16, q_heads=40, len_lo=8192, len_hi=131072,
             sizes="16,32,64", keys="planted"),
    ]


MOST_BYTES = 2.2e9  # no drawn case moves more than the largest listed one


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choices(("step", "generate", "build"), (8, 2, 2))[0]
        batch = _log(rng, 1, 16)
        hi = _log(rng, 512, min(524288, 1200000 // batch))
        lo = hi if batch == 1 or rng.random() < 0.4 else max(1, int(hi * rng.uniform(0.05, 0.9)))
        kv = rng.choices((2, 4, 8, 16), (1, 1, 6, 1))[0]
        group = rng.choice((1, 2, 4, 4, 5, 7, 8))
        c = case(kind=kind, dtype=rng.choice(("f16", "bf16")), batch=batch, q_heads=kv * group, kv_heads=kv,
                 page=rng.choice((16, 32, 64, 64, 128)), len_lo=lo, len_hi=hi, shape_seed=rng.randrange(1 << 20),
                 sizes=rng.choice(("8,16,32,64,128", "16,32,64", "8,16,32,64", "16", "32", "64")),
                 repr=rng.choices(("mean", "minmax"), (4, 1))[0], keys=rng.choice(("zipf", "planted", "lowrank")))
        if kind != "build":
            mode = rng.random()
            if mode < 0.7:
                c["budget"] = _log(rng, 128, 16384)
            elif mode < 0.9:
                c["budget"], c["budget_pct"] = 0, rng.randint(2, 10)
            else:
                c["budget"] = hi
            if c["repr"] == "mean":
                c["select"] = rng.choices(("group", "per_query_head", "group_max"), (6, 1, 1))[0]
            if rng.random() < 0.25:
                c["sink"], c["recent"] = rng.choice((4, 64)), rng.choice((64, 256))
            c["list"] = rng.random() < 0.25
        if kind == "generate":
            c["tokens"], c["layers"] = rng.randint(2, 12), rng.randint(1, 4)
            if lengths(c).sum() * kv * c["layers"] > 1 << 24:
                continue
        if batch * kv * hi * 2 * D > 6e9 or work(c)["bytes"] > MOST_BYTES:
            continue
        return c


# ------------------------------------------------------------------ shapes of a case
def lengths(c):
    r = random.Random(c["shape_seed"])
    return np.array([r.randint(c["len_lo"], c["len_hi"]) for _ in range(c["batch"])], np.int32)


def block_sizes(c, layer=0):
    r = random.Random(1000 * c["shape_seed"] + layer)
    sizes = [int(x) for x in c["sizes"].split(",")]
    return np.array([r.choice(sizes) for _ in range(c["kv_heads"])], np.int32)


def budgets(c, lens):
    if c["budget_pct"]:
        return ((c["budget_pct"] * lens.astype(np.int64) + 99) // 100).astype(np.int32)
    return np.full(len(lens), c["budget"], np.int32)


def work(c):
    """Of one pass: 4-bit codes, scales and queries in, the K and V rows of the selected tokens in, outputs
    out; for a build the keys in, codes, scales and offsets out.  Scores, lists and partial sums between the
    stages are not counted.  Query heads that select for themselves read a list each (never more than the
    context)."""
    lens, R, G = lengths(c), 1 + (c["repr"] == "minmax"), c["q_heads"] // c["kv_heads"]
    nseg = c["batch"] * c["kv_heads"]
    nbytes = flops = 0.0
    for layer in range(c["layers"]):
        B = block_sizes(c, layer).astype(np.int64)
        N = -(-lens[:, None].astype(np.int64) // B)
        store = N.sum() * 64 * R + nseg * 128 * 4 * R
        if c["kind"] == "build":
            keys = lens.astype(np.int64).sum() * c["kv_heads"]
            nbytes += keys * 2 * D + store + nseg * 128 * 4 * R
            flops += keys * D * R
            continue
        T = budgets(c, lens).astype(np.int64)[:, None]
        chosen = np.minimum(-(-T // B) * B, lens[:, None]).sum()
        if c["select"] == "per_query_head":
            rows = np.minimum(G * (-(-T // B) * B), lens[:, None]).sum()
        else:
            rows = chosen
        ranked = 1 if c["select"] == "group" else G  # dot products per block
        steps = max(1, c["tokens"])
        nbytes += steps * (store + rows * 2 * 2 * D + c["batch"] * c["q_heads"] * D * 2 * 2)
        flops += steps * (N.sum() * 2 * D * R * ranked + chosen * G * 4 * D)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(c):
    # integers (selected blocks, codes) and the build's binary32 scales have one right value; the output is a
    # softmax average whose weights and result are rounded to the K/V type
    if c["kind"] == "build":
        return "exact"
    return {"rel": 1e-3 if c["dtype"] == "f16" else 8e-3}


# ------------------------------------------------------------------ what a program has in hand before the call
def _heavy_keys(c, g, k, q, page_table, lens):
    """Keys that a query meets in earnest, per (request, KV head): `planted` = 16 tokens well above the rest;
    `zipf` = up to 4096 tokens of falling weight, in runs of 1 to 64 (drawn per head)."""
    dev, P, G = k.device, c["page"], c["q_heads"] // c["kv_heads"]
    r = random.Random(c["shape_seed"] + 7)
    run_of_head = [r.choice((1, 4, 16, 64)) for _ in range(c["kv_heads"])]
    for b, L in enumerate(int(x) for x in lens):
        for h in range(c["kv_heads"]):
            if c["keys"] == "planted":
                u = torch.randn(D, generator=g, device=dev)
                u *= math.sqrt(D) / u.norm()
                pos = torch.randperm(L, generator=g, device=dev)[:16]
                rows = (4.0 * u).expand(len(pos), D)
                q[b, h * G:(h + 1) * G] += u.to(q.dtype)
            else:
                rho = run_of_head[h]
                runs = min(4096, L // 2) // rho
                if runs == 0:
                    continue
                slot = torch.randperm(L // rho, generator=g, device=dev)[:runs]
                pos = (slot[:, None] * rho + torch.arange(rho, device=dev)[None]).reshape(-1)
                pos = pos[torch.randperm(len(pos), generator=g, device=dev)]
                qbar = q[b, h * G:(h + 1) * G].float().mean(0)
                z = 16.0 - 1.1 * torch.log(torch.arange(1, len(pos) + 1, device=dev))
                rows = torch.randn(len(pos), D, generator=g, device=dev)
                rows += (z * math.sqrt(D) / qbar.norm())[:, None] * (qbar / qbar.norm())[None]
            k[page_table[b, pos // P].long(), h, pos % P] = rows.to(k.dtype)


def _keys_and_values(c, g, dev, tdt, q, page_table, lens, pages, need_v):
    shape = (pages, c["kv_heads"], c["page"], D)
    k = torch.empty(shape, dtype=tdt, device=dev)
    if c["keys"] == "lowrank":  # rank 8 per head, plus noise
        for h in range(c["kv_heads"]):
            basis = torch.randn(8, D, generator=g, device=dev) / math.sqrt(8)
            coef = torch.randn(pages * c["page"], 8, generator=g, device=dev)
            noise = torch.randn(pages * c["page"], D, generator=g, device=dev)
            k[:, h] = (coef @ basis + 0.1 * noise).to(tdt).view(pages, c["page"], D)
    else:
        k.normal_(generator=g)
        _heavy_keys(c, g, k, q, page_table, lens)
    v = torch.empty(shape, dtype=tdt, device=dev).normal_(generator=g) if need_v else None
    return k, v


def prepare(c, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    dt, tdt = DTYPE[c["dtype"]]
    P, Hkv, Hq = c["page"], c["kv_heads"], c["q_heads"]
    lens = lengths(c)
    end = lens + c["tokens"]  # what the contexts grow to
    npages = [-(-int(L) // P) for L in end]
    pages = sum(npages)
    perm = torch.randperm(pages, generator=g, device=dev).int()
    page_table = torch.zeros((c["batch"], max(npages)), dtype=torch.int32, device=dev)
    at = 0
    for b, n in enumerate(npages):
        page_table[b, :n] = perm[at:at + n]
        at += n
    T = budgets(c, lens)
    s = {"case": c, "lens": lens, "seq_lens0": torch.from_numpy(lens).to(dev), "layers": []}
    s["seq_lens"] = s["seq_lens0"].clone()
    # host lengths of every step of the loop, as the program's scheduler has them
    s["lens_at"] = [lens + i + 1 for i in range(c["tokens"])]
    budget = torch.from_numpy(T).to(dev)
    R = 1 + (c["repr"] == "minmax")
    nseg = c["batch"] * Hkv
    nsel = c["batch"] * (Hq if c["select"] == "per_query_head" else Hkv)
    for i in range(c["layers"]):
        q = torch.randn((max(1, c["tokens"]), c["batch"], Hq, D), generator=g, device=dev).to(tdt)
        k, v = _keys_and_values(c, g, dev, tdt, q[0], page_table, end, pages, c["kind"] != "build")
        layer = absb.Layer(Hq, Hkv, D, P, dt, block_sizes(c, i), (Hkv * P * D, P * D, D), block_repr=REPR[c["repr"]],
                           sink_tokens=c["sink"], recent_tokens=c["recent"], selection=SELECTION[c["select"]])
        batch = absb.Batch(seq_lens_host=lens, budget_host=None if c["kind"] == "build" else T, seq_lens=s["seq_lens"],
                           page_table=page_table, budget=budget)
        if c["tokens"]:
            batch.cap_lens_host = end
            batch.seq_lens_host = end  # buffers are sized for the longest contexts
        plan = absb.absb_plan(layer, batch)
        batch.seq_lens_host = lens
        batch.cent_off = torch.from_numpy(plan.cent_off).to(dev)
        # zero-filled: counters start at zero, and rows beyond the current lengths are defined
        x = dict(layer=layer, batch=batch, q=q, k=k, v=v,
                 codes=torch.zeros((plan.total_centroids, 64 * R), dtype=torch.uint8, device=dev),
                 qscale=torch.zeros((nseg, D * R), dtype=torch.float32, device=dev),
                 qmin=torch.zeros((nseg, D * R), dtype=torch.float32, device=dev),
                 workspace=torch.zeros(plan.workspace_bytes, dtype=torch.uint8, device=dev))
        batch.qmin = x["qmin"]
        if c["kind"] != "build":
            n = max(1, c["tokens"])
            x["out"] = torch.zeros((n, c["batch"], Hq, D), dtype=tdt, device=dev)
            x["lse"] = torch.zeros((n, c["batch"], Hq), dtype=torch.float32, device=dev)
            x["sel_idx"] = x["sel_cnt"] = None
            if c["list"] and not c["tokens"]:
                x["sel_idx"] = torch.zeros((nsel, plan.sel_stride), dtype=torch.int32, device=dev)
                x["sel_cnt"] = torch.zeros((nsel,), dtype=torch.int32, device=dev)
            x["tail"] = torch.zeros((nseg, D * R), dtype=torch.float32, device=dev)
            absb.absb_build_centroids(layer, batch, k, x["codes"], x["qscale"], x["qmin"], x["workspace"])
            absb.absb_workspace_init(layer, batch, x["workspace"])
        s["layers"].append(x)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    c = s["case"]
    if c["kind"] == "generate":
        return _generate(s, c)
    x = s["layers"][0]
    if c["kind"] == "build":
        absb.absb_build_centroids(x["layer"], x["batch"], x["k"], x["codes"], x["qscale"], x["qmin"], x["workspace"])
        return {"codes": x["codes"], "qscale": x["qscale"], "qmin": x["qmin"]}
    absb.absb_decode_fused(x["layer"], x["batch"], x["q"], x["codes"], x["qscale"], x["k"], x["v"], x["out"], x["lse"],
                           x["sel_idx"], x["sel_cnt"], x["workspace"])
    return {"out": x["out"], "lse": x["lse"], "sel_idx": x["sel_idx"], "sel_cnt": x["sel_cnt"]}


def _generate(s, c):
    seq_lens, got = s["seq_lens"], {}
    # the requests enter the decode batch: their lengths, and the state of their last blocks
    seq_lens.copy_(s["seq_lens0"])
    for x in s["layers"]:
        x["batch"].seq_lens_host = s["lens"]
        absb.absb_tail_init(x["layer"], x["batch"], x["k"], x["tail"])
    for i in range(c["tokens"]):
        seq_lens.add_(1)
        for x in s["layers"]:
            batch = x["batch"]
            batch.seq_lens_host = s["lens_at"][i]
            absb.absb_append_token(x["layer"], batch, x["k"], x["codes"], x["qscale"], x["qmin"], x["tail"])
            absb.absb_decode_fused(x["layer"], batch, x["q"][i], x["codes"], x["qscale"], x["k"], x["v"], x["out"][i],
                                   x["lse"][i], None, None, x["workspace"])
    for n, x in enumerate(s["layers"]):
        got["layer%d" % n] = {"out": x["out"], "lse": x["lse"], "codes": x["codes"], "tail": x["tail"]}
    return got
