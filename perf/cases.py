"""The work that users of this library have it do, as cases that a timing or comparison harness can run.

A case is a dict of plain values.  `listed()` names the standing ones, `draw(rng)` gives more of the same
ranges, `prepare(case, seed)` makes what a program holds before the call (inputs, buffers, the prepared
plan), `run(state)` is one pass through the public entry points, `work(case)` the bytes and operations the
pass cannot do without, `tolerance(case)` how far two correct implementations may be apart.

Kinds of case
  compress  the whole path on a prefilled cache: score, allocate, select and gather (`Compressor.run`).
            With fresh = True the plan is made inside the pass: prompts have lengths of their own, so a
            server that meets a new length builds buffers and tables for it before it can compress.
  layers    the cache handed over layer by layer, as prefill produces it (`score_layer`), then one
            allocation and the gather into a paged cache.
  select    the stages behind the scores: budgets from given energies, selection and gather from given
            scores (a program that scores some other way, or keeps scores and changes the budget).
  decode    one decode step of attention over a compacted cache, packed or paged.

What comes back: selection is a step function of the scores.  One pair of tokens whose scores agree to
the last bits of fp32 may change places between two correct implementations, and every later row of that
unit then sits one place further on, so packed indices and rows of a large cache cannot be compared place
by place after a changed rounding.  Large `compress` and `layers` cases therefore return the scores and
energies, from which everything after them follows exactly; `select` returns budgets, offsets, indices and
rows, which have to agree to the bit; the smallest caches, where such a pair is practically never met,
return everything.
"""
import math

import torch

import kvsynth
import paper_2511_16786_amd as fc

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_PAGE = 64
# Caches up to this many (token, head, layer) entries return their indices and rows as well.
_WHOLE_ROWS = 4096


def _cache(name, kind="compress", config=None, **over):
    """A case with the shape of one of the repository's workloads, some fields replaced."""
    c = kvsynth.get_config(config or name)
    case = {"name": name, "kind": kind, "dtype": c.dtype, "batch": c.batch, "layers": c.layers,
            "kv_heads": c.kv_heads, "tokens": c.n_tokens, "head_dim": c.head_dim, "gamma": c.gamma,
            "rho": c.rho, "shared": False, "fresh": False}
    case.update(over)
    return case


def listed():
    return [
        # the smallest call: one fp32 layer of a short prompt, where launches and host time count
        _cache("tiny"),
        # a few layers of a 4K prompt
        _cache("mid"),
        # a multi-image prompt of a 28-layer model
        _cache("qwen_8k"),
        # the same model on a prompt as it comes: an odd number of tokens, a length met for the first time
        _cache("prompt_7321", config="qwen_8k", tokens=7321, fresh=True),
        # long multi-image / video context: the headline workload
        _cache("long_32k"),
        # the upper end of the cut-off range that works best (0.1 to 0.2)
        _cache("long_32k_wide", config="long_32k", gamma=0.2),
        # long context of arbitrary length, the whole layer sharing one index set
        _cache("long_30011", config="long_32k", tokens=30011, gamma=0.1, shared=True),
        # a batch of eight sequences, the most a pass is given here
        _cache("batch8_16k"),
        # prefill hands its layers over one by one; the kept rows go into a paged cache
        _cache("layers_16k", kind="layers", config="batch8_16k", batch=1),
        # budgets, selection and gather for given scores
        _cache("select_32k", kind="select", config="long_32k"),
        # a decode step over the compacted 32K cache, 7 query heads for each KV head
        _cache("decode_32k", kind="decode", config="long_32k", group=7, paged=False),
        # a decode step of eight sequences through block tables
        _cache("decode_paged", kind="decode", config="batch8_16k", group=7, paged=True),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["compress", "compress", "compress", "compress", "layers", "select", "decode", "decode"])
    case = {"kind": kind, "dtype": "f32" if rng.random() < 0.15 else "bf16",
            "batch": rng.choice([1, 1, 1, 2, 3, 8]), "layers": int(round(_log_uniform(rng, 1, 36))),
            "kv_heads": rng.choice([2, 4, 4, 8]), "head_dim": rng.choice([64, 128, 128]),
            "tokens": int(_log_uniform(rng, 512, 66000)), "gamma": round(_log_uniform(rng, 0.03, 0.5), 4),
            "rho": round(_log_uniform(rng, 0.05, 0.4), 4), "shared": rng.random() < 0.2, "fresh": False}
    # half of the caches are padded to a round length by their program, the others come as they are
    if rng.random() < 0.5:
        case["tokens"] = max(512, case["tokens"] // 256 * 256)
    if kind == "layers":
        case["layers"] = max(4, case["layers"])
    if kind == "compress":
        case["fresh"] = rng.random() < 0.25
    if kind == "decode":
        case["group"] = rng.choice([1, 4, 7, 8])
        case["paged"] = rng.random() < 0.5
    # no more than the largest listed cases: rows of the batch of eight, and for scoring also the
    # rows times kept modes of the long prompt of arbitrary length
    while True:
        c = case
        rows = c["batch"] * c["layers"] * c["kv_heads"] * c["tokens"] * c["head_dim"] * (2 if c["dtype"] == "f32" else 1)
        if rows <= 8 * 28 * 4 * 16384 * 128 and (
                kind in ("select", "decode") or rows * c["gamma"] * c["tokens"] <= 28 * 4 * 30011 * 128 * 0.1 * 30011):
            return case
        if case["batch"] > 1:
            case["batch"] = 1
        elif case["layers"] > 4:
            case["layers"] //= 2
        else:
            case["tokens"] = case["tokens"] * 3 // 4


def _total(case):
    return fc.total_budget(case["layers"], case["tokens"], case["rho"])


def _kv(case, gen):
    """K and V [B, L, H, N, d]: text around image blocks whose tokens follow a few smooth modes with
    noise, and a small share of strongly deviating pairs, as kvsynth describes them; made on the GPU."""
    B, L, H, N, d = (case[k] for k in ("batch", "layers", "kv_heads", "tokens", "head_dim"))
    dt = _DTYPES[case["dtype"]]
    dev = gen.device
    blocks = max(1, N // 1024)
    length = (N - N // 64) // blocks
    start = (N - blocks * length) // 2
    u = (torch.arange(length, device=dev, dtype=torch.float32) + 0.5) / length
    modes = torch.cos(math.pi * u[:, None] * torch.arange(8, device=dev, dtype=torch.float32))
    scale = (1.0 / torch.arange(1, 9, device=dev, dtype=torch.float32)).sqrt()[:, None]
    K = torch.empty((B, L, H, N, d), dtype=dt, device=dev)
    V = torch.empty_like(K)
    outliers = max(1, N // 50)
    for b in range(B):
        for l in range(L):
            # layers differ in how many pairs deviate: 0.5 % to 5 %
            share = torch.rand((), generator=gen, device=dev) * 2.25 + 0.25
            pos = torch.randperm(N, generator=gen, device=dev)[:outliers]
            strength = 3.0 * share * torch.rand((outliers, 1), generator=gen, device=dev).add_(0.2)
            for out in (K, V):
                x = torch.randn((H, N, d), generator=gen, device=dev)
                w = torch.randn((H, blocks, 8, d), generator=gen, device=dev) * scale
                image = x[:, start:start + blocks * length]
                image.mul_(0.1)
                image.add_(torch.matmul(modes, w).view(H, blocks * length, d))
                x.index_add_(1, pos, strength * torch.randn((H, outliers, d), generator=gen, device=dev))
                out[b, l] = x
    return K, V


def _budgets(case, gen):
    """Per-layer budgets that differ as the allocation makes them differ, and their offsets."""
    B, L, H, N = (case[k] for k in ("batch", "layers", "kv_heads", "tokens"))
    total = _total(case)
    w = 0.5 + torch.rand((B, L), generator=gen, device=gen.device, dtype=torch.float64).cpu()
    share = (total - L) * w / w.sum(1, keepdim=True)
    b = share.floor().clamp(max=N - 1).to(torch.int64) + 1
    for row in b:
        short = total - int(row.sum())
        l = 0
        while short > 0:
            give = min(short, N - int(row[l]))
            row[l] += give
            short -= give
            l += 1
    off = torch.zeros((B, L + 1), dtype=torch.int64)
    off[:, 1:] = torch.cumsum(H * b, 1)
    return b.to(torch.int32).to(gen.device), off.to(gen.device), H * total


def _table(case, gen, most):
    """Block table [B, L, H, pages] over a shuffled pool that holds every unit's `most` rows."""
    B, L, H = (case[k] for k in ("batch", "layers", "kv_heads"))
    pages = -(-most // _PAGE)
    table = torch.randperm(B * L * H * pages, generator=gen, device=gen.device).to(torch.int32)
    return table.view(B, L, H, pages), B * L * H * pages


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    B, L, H, N, d = (case[k] for k in ("batch", "layers", "kv_heads", "tokens", "head_dim"))
    dt = _DTYPES[case["dtype"]]
    s = {"case": case, "r": fc.cutoff_r(N, case["gamma"]), "total": _total(case)}
    kind = case["kind"]
    if kind in ("compress", "layers"):
        s["K"], s["V"] = _kv(case, gen)
    if kind == "compress" and not case["fresh"]:
        s["plan"] = fc.Compressor(s["K"], s["r"], s["total"], shared=case["shared"])
    elif kind == "layers":
        s["layers"] = [(s["K"][:, l:l + 1], s["V"][:, l:l + 1]) for l in range(L)]
        s["desc"] = fc.describe(s["layers"][0][0])
        s["path"] = fc.resolve_path(s["desc"], s["r"])
        s["workspace"] = torch.empty(fc.workspace_bytes(s["desc"], s["r"], s["path"]), dtype=torch.uint8, device=dev)
        fc.prepare(s["desc"], s["r"], s["path"], s["workspace"])
        s["scores"] = torch.empty((B, L, H, N), dtype=torch.float32, device=dev)
        s["energy"] = torch.empty((B, L, H, 4), dtype=torch.float64, device=dev)
    elif kind == "select":
        s["K"] = torch.randn((B, L, H, N, d), generator=gen, device=dev, dtype=dt)
        s["V"] = torch.randn((B, L, H, N, d), generator=gen, device=dev, dtype=dt)
        # mean squared deviations of noise over 2d values, with the long tail of the deviating pairs
        x = torch.randn((B, L, H, N), generator=gen, device=dev)
        tail = torch.rand((B, L, H, N), generator=gen, device=dev)
        s["scores"] = 0.02 * (1.0 + x / math.sqrt(d)).clamp_(min=0.05) * (1.0 + 200.0 * (tail - 0.97).clamp_(min=0.0))
        total = N * d * (0.5 + torch.rand((B, L, H, 2), generator=gen, device=dev, dtype=torch.float64))
        part = 0.01 + 0.1 * torch.rand((B, L, H, 2), generator=gen, device=dev, dtype=torch.float64)
        s["energy"] = torch.cat((total * part, total), 3)
    if kind in ("layers", "select"):
        s["budgets"] = torch.empty((B, L), dtype=torch.int32, device=dev)
        s["offsets"] = torch.empty((B, L + 1), dtype=torch.int64, device=dev)
        s["idx"] = torch.empty((B, H * s["total"]), dtype=torch.int32, device=dev)
    if kind == "layers":
        # pages for up to four times the mean budget, at most the whole layer
        s["table"], pages = _table(case, gen, min(N, 4 * s["total"] // L + 1))
        s["K_out"] = torch.empty((pages, _PAGE, d), dtype=dt, device=dev)
        s["V_out"] = torch.empty_like(s["K_out"])
        s["full"] = fc.describe(s["K"])
    elif kind == "select":
        s["desc"] = fc.describe(s["K"])
        s["K_out"] = torch.empty((B, H * s["total"], d), dtype=dt, device=dev)
        s["V_out"] = torch.empty_like(s["K_out"])
    elif kind == "decode":
        s["Q"] = torch.randn((B, L, H * case["group"], d), generator=gen, device=dev, dtype=dt)
        s["budgets"], s["offsets"], s["rows"] = _budgets(case, gen)
        s["out"] = torch.empty((B, L, H * case["group"], d), dtype=torch.float32, device=dev)
        if case["paged"]:
            s["table"], pages = _table(case, gen, int(s["budgets"].max()))
            shape = (pages, _PAGE, d)
        else:
            shape = (B, s["rows"], d)
        s["K"] = torch.randn(shape, generator=gen, device=dev, dtype=dt)
        s["V"] = torch.randn(shape, generator=gen, device=dev, dtype=dt)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "compress":
        plan = s.get("plan")
        if plan is None:
            plan = fc.Compressor(s["K"], s["r"], s["total"], shared=case["shared"])
        plan.run(s["K"], s["V"])
        out = {"scores": plan.scores, "energy": plan.energy}
        if _all_outputs(case):
            out.update(budgets=plan.budgets, offsets=plan.layer_offsets, idx=plan.idx, K=plan.K_out, V=plan.V_out)
        return out
    if kind == "decode":
        scale = 1.0 / math.sqrt(case["head_dim"])
        if case["paged"]:
            return fc.decode_attention_paged(s["Q"], s["K"], s["V"], case["kv_heads"], s["budgets"], s["table"],
                                             scale, out=s["out"])
        return fc.decode_attention(s["Q"], s["K"], s["V"], case["kv_heads"], s["budgets"], s["offsets"], s["rows"],
                                   scale, out=s["out"])
    B, L, H, N = (case[k] for k in ("batch", "layers", "kv_heads", "tokens"))
    rows = H * s["total"]
    if kind == "layers":
        for l, (K, V) in enumerate(s["layers"]):
            fc.score_layer(K, V, s["desc"], l, L, s["r"], s["path"], s["scores"], s["energy"], s["workspace"])
    fc.allocate(s["energy"], B, L, H, N, s["total"], 1, N, s["budgets"], s["offsets"])
    if kind == "layers":
        fc.select_gather_paged(s["K"], s["V"], s["full"], s["scores"], s["budgets"], s["offsets"], rows, s["idx"],
                               s["table"], _PAGE, s["K_out"], s["V_out"], shared=case["shared"])
        return {"scores": s["scores"], "energy": s["energy"]}
    fc.binding.select_gather(s["K"], s["V"], s["desc"], s["scores"], s["budgets"], s["offsets"], rows, s["idx"],
                             s["K_out"], s["V_out"], shared=case["shared"])
    return {"budgets": s["budgets"], "offsets": s["offsets"], "idx": s["idx"], "K": s["K_out"], "V": s["V_out"]}


def _all_outputs(case):
    return (case["kind"] == "compress"
            and case["batch"] * case["layers"] * case["kv_heads"] * case["tokens"] <= _WHOLE_ROWS)


def work(case):
    B, L, H, N, d = (case[k] for k in ("batch", "layers", "kv_heads", "tokens", "head_dim"))
    e = 2 if case["dtype"] == "bf16" else 4
    units, kept = B * L * H, B * H * _total(case)
    kind = case["kind"]
    if kind == "decode":
        q = B * L * H * case["group"] * d
        return {"bytes": 2 * kept * d * e + q * (e + 4), "flops": 4 * kept * case["group"] * d}
    if kind == "select":     # scores, the kept rows in, indices and rows out
        return {"bytes": units * (4 * N + 32) + kept * (4 * d * e + 4), "flops": 0}
    # K and V once, scores and energies out, indices and rows out; a cosine transform there and back
    return {"bytes": units * (2 * N * d * e + 4 * N + 32) + kept * (2 * d * e + 4),
            "flops": units * d * N * (10 * math.log2(N) + 6)}


def tolerance(case):
    if case["kind"] == "select":
        return "exact"
    if case["kind"] == "decode":
        # sums of thousands of rows in fp32, weights from exp2 of fp32 logits
        return {"rel": 2e-5, "max": 1e-3}
    # fp32 transforms of inputs up to tens of times the residual whose square is the score
    return {"rel": 1e-5, "max": 4e-4}
