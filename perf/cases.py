"""Performance cases: the calls that a prefill program makes of this library.

A case is one layer's attention pass (Triangle, dense causal, block-sparse)
or one layer's region probe, through the binding's public entry points, on
inputs, schedule and workspace that a program holds before the call.  Shapes
are the attention shapes of the workload table, of the tests and generic ones
between them; values follow the workload table's draws (N(0, 1), with
per-head factors in [0.5, 2] or with one key of eight times the norm, as an
attention sink has).

Fields of a case
  pass     triangle | causal | blocksparse | probe | region_grad
  lens     sequence lengths of the packed batch, comma separated
  hq, hkv, d, tile
  sink, window, last   the sections (0 where the pass has none)
  out      bf16 | f32 (attention passes)
  lse      whether the row normaliser is returned too
  entry    plan (Plan.run) | noalloc (triangle_attn_fwd_noalloc)
  density  block-sparse: share of the earlier k-tiles that a q-tile lists
  values   heads | sink (see above)
"""
import math

import numpy as np
import torch

from paper_2507_21526_amd import binding

DEVICE = "cuda"


def _case(name, kind, lens, hq, hkv, d, tile, sink=0, window=1, last=0, out="bf16", lse=False,
          entry="plan", density=0.0, values="sink"):
    c = {"pass": kind, "lens": ",".join(str(n) for n in lens), "hq": hq, "hkv": hkv, "d": d,
         "tile": tile, "sink": sink, "window": window, "last": last, "out": out, "lse": lse,
         "entry": entry, "density": density, "values": values}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one kv head, a 1024-token prompt (launch and
        # latency count)
        _case("tri_tiny_1k_d64", "triangle", [1024], 4, 1, 64, 64, 64, 256, 64),
        # a short odd prompt at the paper's own sink and window, with the
        # row normaliser, through the entry point of programs that may not
        # allocate
        _case("tri_prompt_3001", "triangle", [3001], 32, 8, 128, 128, 8, 512, 128, lse=True,
              entry="noalloc"),
        # a long document: 32K tokens, per-head scales
        _case("tri_32k", "triangle", [32768], 32, 8, 128, 128, 128, 2048, 128, values="heads"),
        # the largest call: one layer of the 128K-token prefill
        _case("tri_128k", "triangle", [131072], 32, 8, 128, 128, 128, 2048, 128),
        # long context at the paper's sink 8 / window 512: short work items
        _case("tri_64k_s8_w512", "triangle", [65536], 32, 8, 128, 128, 8, 512, 128),
        # a packed batch of ragged requests
        _case("tri_packed", "triangle", [8191, 317, 24001, 1, 15360, 2990], 32, 8, 128, 128,
              128, 2048, 128, lse=True, values="heads"),
        # seven query heads to a kv head, the wider window
        _case("tri_48k_g7", "triangle", [49152], 28, 4, 128, 128, 128, 4096, 256),
        # multi-head attention (one query head to a kv head)
        _case("tri_32k_mha", "triangle", [32768], 32, 32, 128, 128, 128, 2048, 128),
        # a dense layer over a packed batch of short requests, head dimension
        # 64, eight query heads to a kv head, fp32 output
        _case("causal_packed_d64", "causal", [4096, 77, 1500, 2048, 640, 3333, 129], 32, 4, 64,
              64, out="f32", lse=True, values="heads"),
        # a dense layer of the mixed stack
        _case("causal_16k", "causal", [16384], 32, 8, 128, 128),
        # a dense layer handed to a dynamic sparse method: a tenth of the
        # k-tiles
        _case("blocksparse_64k", "blocksparse", [65536], 32, 8, 128, 128, density=0.1),
        # one layer of the layer choice: the region probe of a 2K prompt, the
        # whole call (plan, causal pass, probe, means)
        _case("region_grad_2k", "region_grad", [2048], 32, 8, 128, 128, 64, 128, 128),
    ]


_LARGEST = 4.0e12  # flops of the largest drawn case (the largest listed one has 4.9e12)


def draw(rng):
    """One more case of the same ranges."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    while True:
        kind = rng.choices(["triangle", "causal", "blocksparse", "probe", "region_grad"],
                           [10, 4, 3, 1, 2])[0]
        d = rng.choice([128, 128, 128, 64])
        group = rng.choice([1, 2, 3, 4, 4, 4, 5, 6, 7, 8])
        hkv = rng.choice([1, 2, 4, 8, 8]) if group > 1 else rng.choice([4, 8, 16, 32])
        tile = rng.choice([128, 128, 128, 64])
        top = {"triangle": 131072, "causal": 32768, "blocksparse": 98304, "probe": 32768,
               "region_grad": 8192}[kind]
        total = log(700, top)
        lens = [total]
        if kind != "region_grad" and rng.random() < 0.4:  # a packed batch
            cuts = sorted(rng.randrange(total + 1) for _ in range(rng.randrange(1, 8)))
            lens = [b - a for a, b in zip([0] + cuts, cuts + [total])]
        sink = window = last = 0
        if kind in ("triangle", "probe", "region_grad"):
            sink = rng.choice([0, 4, 8, 64, 128, 128, rng.randrange(1, 257)])
            window = rng.choice([512, 2048, 2048, 4096, log(64, 4096)])
            last = rng.choice([0, 64, 128, 128, 256, rng.randrange(1, 257)])
        entry = "plan"
        if kind == "triangle" and total <= 16384 and rng.random() < 0.2:
            entry = "noalloc"
        c = _case(None, kind, lens, group * hkv, hkv, d, tile, sink, max(window, 1), last,
                  out=rng.choice(["bf16", "bf16", "bf16", "f32"]), lse=rng.random() < 0.3,
                  entry=entry,
                  density=round(rng.uniform(0.03, 0.3), 3) if kind == "blocksparse" else 0.0,
                  values=rng.choice(["heads", "sink"]))
        if work(c)["flops"] <= _LARGEST:
            return c


def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def _cu(case):
    return [0] + [int(x) for x in np.cumsum(_lens(case))]


def _lists(case, seed):
    """Block-sparse lists in CSR form: q-tile t of a sequence lists
    round(density t) of its earlier k-tiles, drawn without replacement, and
    its diagonal tile, as a block estimator does."""
    rng = np.random.default_rng(int(seed))
    ptr, idx = [0], []
    for n in _lens(case):
        for t in range(-(-n // case["tile"])):
            keep = rng.permutation(t)[:int(round(case["density"] * t))]
            idx.extend(int(x) for x in np.sort(keep))
            idx.append(t)
            ptr.append(len(idx))
    return ptr, idx


def _inputs(case, seed):
    g = torch.Generator(device=DEVICE).manual_seed(int(seed))
    total, hq, hkv, d = sum(_lens(case)), case["hq"], case["hkv"], case["d"]

    def normal(heads):
        x = torch.randn(total, heads, d, generator=g, device=DEVICE)
        if case["values"] == "heads":
            x *= 0.5 + 1.5 * torch.rand(1, heads, 1, generator=g, device=DEVICE)
        return x

    q, k, v = normal(hq).bfloat16(), normal(hkv), normal(hkv).bfloat16()
    if case["values"] == "sink":
        first = [b for b, n in zip(_cu(case), _lens(case)) if n]
        k[first] *= 8.0
    dout = None
    if case["pass"] in ("probe", "region_grad"):
        dout = torch.randn(total, hq, d, generator=g, device=DEVICE).bfloat16()
    return q, k.bfloat16(), v, dout


def prepare(case, seed):
    kind, cu = case["pass"], _cu(case)
    q, k, v, dout = _inputs(case, seed)
    hq, d = case["hq"], case["d"]
    s = {"case": case, "cu": cu, "q": q, "k": k, "v": v, "dout": dout, "scale": d ** -0.5}
    if kind == "region_grad":
        return s
    if kind == "blocksparse":
        plan = binding.Plan("blocksparse", cu, 0, 1, 0, case["tile"], hq, d,
                            blocks=_lists(case, seed))
    elif kind == "triangle":
        plan = binding.Plan("triangle", cu, case["sink"], case["window"], case["last"],
                            case["tile"], hq, d)
    else:
        plan = binding.Plan("causal", cu, 0, 1, 0, case["tile"], hq, d)
    s["plan"] = plan
    if kind == "probe":
        # the probe takes the causal normaliser, which the dense pass wrote
        o = torch.empty_like(q)
        s["lse"] = torch.empty(hq, q.shape[0], dtype=torch.float32, device=DEVICE)
        plan.run(q, k, v, o, s["lse"])
        s["sums"] = torch.empty(hq, 3, dtype=torch.float64, device=DEVICE)
        n = binding.ta_probe_workspace_bytes(plan.info, hq)
        s["ws"] = torch.empty(n, dtype=torch.uint8, device=DEVICE) if n else None
        return s
    s["o"] = torch.empty(q.shape, device=DEVICE,
                         dtype=torch.bfloat16 if case["out"] == "bf16" else torch.float32)
    s["lse"] = (torch.empty(hq, q.shape[0], dtype=torch.float32, device=DEVICE)
                if case["lse"] else None)
    return s


def run(state):
    s, case = state, state["case"]
    if case["pass"] == "region_grad":
        grad, sums = binding.region_grad(s["q"], s["k"], s["v"], s["dout"], s["cu"], case["sink"],
                                         case["window"], case["last"], case["tile"])
        return {"grad": grad, "sums": sums}
    plan = s["plan"]
    if case["pass"] == "probe":
        binding.region_grad_probe(s["q"], s["k"], s["v"], s["dout"], s["lse"], plan.sched,
                                  plan.info, s["scale"], case["sink"], case["window"],
                                  case["last"], s["sums"], s["ws"])
        return {"sums": s["sums"]}
    if case["entry"] == "noalloc":
        binding.triangle_attn_fwd_noalloc(s["q"], s["k"], s["v"], s["o"], s["lse"], plan.sched,
                                          plan.info, s["scale"])
    else:
        plan.run(s["q"], s["k"], s["v"], s["o"], s["lse"])
    return {"o": s["o"], "lse": s["lse"]}


def _pairs(case):
    """Kept (row, key) pairs of one query head."""
    kept = 0
    for n in _lens(case):
        i = np.arange(n, dtype=np.int64)
        if case["pass"] == "triangle":
            win = np.minimum(i + 1, case["window"])
            row = win + np.minimum(case["sink"], i + 1 - win)
            row[n - min(case["last"], n):] = i[n - min(case["last"], n):] + 1
        elif case["pass"] == "blocksparse":
            t = i // case["tile"]
            row = np.rint(case["density"] * t) * case["tile"] + i % case["tile"] + 1
        else:
            row = i + 1
        kept += int(row.sum())
    return kept


def work(case):
    """Two contractions per kept pair; every operand read and every result
    written once.  The probe's two are q.k and dO.v (its normaliser comes
    with them in one sweep)."""
    total, hq, hkv, d = sum(_lens(case)), case["hq"], case["hkv"], case["d"]
    nbytes = 2 * total * (hq + 2 * hkv) * d
    if case["pass"] in ("probe", "region_grad"):
        nbytes += 2 * total * hq * d + hq * 3 * 8
        nbytes += 4 * total * hq if case["pass"] == "probe" else 0
    else:
        nbytes += total * hq * d * (2 if case["out"] == "bf16" else 4)
        nbytes += 4 * total * hq if case["lse"] else 0
    return {"bytes": nbytes, "flops": 4 * d * hq * _pairs(case)}


def tolerance(case):
    if case["pass"] in ("probe", "region_grad"):
        # fp32 products under fp64 sums, 5e-7 against 64 bits; a section's
        # sum may be a small difference of large terms
        return {"rel": 2e-5, "max": 1e-3}
    # probabilities rounded to bf16 for the PV product (and the output, in
    # bf16): against 64 bits 1.3e-3 to 2.2e-3 is seen.  One value of a short
    # row, whose few terms do not average out, may be off by 2^-8 of |v| ~ 1,
    # where the rows of thousands of keys make the root mean square ~ 0.03.
    return {"rel": 8e-3, "max": 0.3}


def exact(case, seed):
    """The pass in 64 bits from its definition, a block of rows at a time."""
    q, k, v, dout = _inputs(case, seed)
    total, hq, hkv, d = q.shape[0], case["hq"], case["hkv"], case["d"]
    group, kind, tile = hq // hkv, case["pass"], case["tile"]
    scale = d ** -0.5
    probe = kind in ("probe", "region_grad")
    o = None if probe else torch.empty(total, hq, d, dtype=torch.float64, device=DEVICE)
    lse = torch.empty(hq, total, dtype=torch.float64, device=DEVICE) if case["lse"] else None
    sums = torch.zeros(hq, 3, dtype=torch.float64, device=DEVICE)
    pairs = [0, 0, 0]
    ptr, idx = _lists(case, seed) if kind == "blocksparse" else (None, None)
    qtile = 0

    def heads_first(x, a, b):  # [heads, rows, d] in 64 bits
        return x[a:b].to(torch.float64).transpose(0, 1).contiguous()

    for off, n in zip(_cu(case), _lens(case)):
        r0 = 0
        first_last = n - min(case["last"], n)
        while r0 < n:
            streaming = kind == "triangle" and r0 < first_last
            # rows whose scores take at most about 1 GB, a q-tile at least
            step = (1 << 27) // (hq * (r0 + 1)) // tile * tile
            step = 1024 if streaming else min(1024, max(tile, step))
            r1 = min(r0 + step, first_last if streaming else n)
            if streaming:
                lo = max(0, r0 - case["window"] + 1)
                s = min(case["sink"], lo)
                keys = torch.cat([torch.arange(s, device=DEVICE),
                                  torch.arange(lo, r1, device=DEVICE)])
            else:
                keys = torch.arange(r1, device=DEVICE)
            rows = torch.arange(r0, r1, device=DEVICE)[:, None]
            keep = keys[None, :] <= rows
            stream = (keys[None, :] < case["sink"]) | (rows - keys[None, :] < case["window"])
            if streaming:
                keep = keep & stream
            if kind == "blocksparse":
                # q-tiles r0 / tile .. of this sequence
                on = torch.zeros(r1 - r0, -(-n // tile), dtype=torch.bool)
                for t in range(r0 // tile, -(-r1 // tile)):
                    a, b = max(t * tile, r0) - r0, min((t + 1) * tile, r1) - r0
                    cols = torch.tensor(idx[ptr[qtile + t]:ptr[qtile + t + 1]])
                    on[a:b, cols] = True
                keep = keep & on.to(DEVICE)[:, keys // tile]
            R = r1 - r0
            qs = heads_first(q, off + r0, off + r1).reshape(hkv, group * R, d)
            ks = k[off + keys].to(torch.float64).permute(1, 2, 0).contiguous()  # [hkv, d, keys]
            sc = torch.bmm(qs, ks).mul_(scale).reshape(hq, R, -1)
            sc.masked_fill_(~keep, -math.inf)
            top = sc.amax(-1, keepdim=True)
            p = sc.sub_(top).exp_()
            den = p.sum(-1, keepdim=True)
            p /= den
            if lse is not None:
                lse[:, off + r0:off + r1] = (top + den.log())[..., 0]
            vs = v[off + keys].to(torch.float64).transpose(0, 1).contiguous()  # [hkv, keys, d]
            if not probe:
                o[off + r0:off + r1] = torch.bmm(p.reshape(hkv, group * R, -1), vs) \
                    .reshape(hq, R, d).transpose(0, 1)
            else:
                g = heads_first(dout, off + r0, off + r1).reshape(hkv, group * R, d)
                p *= torch.bmm(g, vs.transpose(1, 2).contiguous()).reshape(hq, R, -1)
                in_last = (rows >= first_last).expand(R, keys.numel())
                for i, m in enumerate((keep & stream, keep & ~stream & ~in_last,
                                       keep & ~stream & in_last)):
                    sums[:, i] += (p * m).sum((1, 2))
                    pairs[i] += int(m.sum())
            r0 = r1
        qtile += -(-n // tile)
    if kind == "probe":
        return {"sums": sums}
    if kind == "region_grad":
        s = sums.cpu().numpy()
        # entry order as run() gives it: numpy arrays on the host
        return {"grad": np.array([s[:, i].sum() / (hq * pairs[i]) if pairs[i] else 0.0
                                  for i in range(3)]), "sums": s}
    return {"o": o, "lse": lse}
