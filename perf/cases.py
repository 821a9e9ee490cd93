"""The calls whose speed this repository is measured by.

Every case is one pass through the public entry points as a serving stack makes
it for one attention layer of a prompt: the whole sparse-prefill path, or one of
its stages where programs call the stage by itself.  Shapes are those of the
layers the paper's models have (32 query / 4 KV heads and 64 / 8, d = 128), of
their tensor-parallel shards, and of the small smoke workload.

Inputs follow the recipe of the repository's synthetic layers: keys around a
mean per KV head with a lognormal noise scale per key block, queries and values
around small offsets, RoPE on queries and keys, everything rounded once to bf16.
"""

import math

import torch

import paper_2609_20971_amd as rbs

D = 128
TAU_BASE, TAU_RESCUE = 0.9, 0.95  # the thresholds of the repository's workloads
N_SINK, N_LOCAL, N_RECENT = 1, 2, 0
BOX_BUDGET = 0.1                  # budget fraction of the Quest-style selector
#: Work of the largest listed case (in executed query-key pairs times heads): what a drawn one may cost.
MOST_PAIRS = 0.29 * 32 * 131072**2 / 2
#: exact() stops here (heads times tokens squared): the 64-bit attention of a larger case takes too long.
MOST_EXACT = 1.1 * 64 * 65536**2


def listed():
    def c(name, kind, n, hq, hkv, b, layout="heads", **more):
        return dict(name=name, kind=kind, n=n, hq=hq, hkv=hkv, b=b, layout=layout, **more)

    return [
        # The smoke workload: one small layer end to end, where launches and latency count.
        c("layer-2k-2heads-b64", "layer", 2048, 2, 1, 64),
        # A short prompt of odd length, taken in place from a fused QKV projection (token-major rows).
        c("layer-3001-qkv", "layer", 3001, 32, 4, 128, "qkv"),
        # A document-length prompt: selection still keeps about half the blocks.
        c("layer-32k", "layer", 32768, 32, 4, 128),
        # The headline layer: 128K tokens, Qwen3-30B-A3B heads, B = 128.
        c("layer-128k", "layer", 131072, 32, 4, 128),
        # The same prompt at the finest block size: the selector's share is largest here.
        c("layer-128k-b64", "layer", 131072, 32, 4, 64),
        # The 64-head layer through the one-pass entry point.
        c("fused-64k-64heads", "fused", 65536, 64, 8, 128),
        # A batch of ragged chat prompts, one launch per stage.
        c("varlen-16-chats", "varlen", 0, 32, 4, 128, "qkv",
          seqs="37,5210,813,129,2900,1024,412,7001,256,1777,95,3333,640,4500,1,2211"),
        # A layer kept dense (a model's first layers), with the log-sum-exp that a merge of partial results needs; B = 256.
        c("dense-16k-b256-lse", "attend", 16384, 32, 4, 256, "tokens", dense=True, lse=True),
        # FP8 attention of an FP8 model: the E4M3 copies of new Q, K and V, then attention at the paper's densities.
        c("fp8-40k", "fp8", 40961, 32, 4, 128, dense=False),
        # Block statistics alone: written when a prefix goes into a cache.
        c("stats-128k", "stats", 131072, 32, 4, 128),
        # Selection alone, on statistics kept with the prefix.
        c("select-48k-64heads", "select", 49000, 64, 8, 128, "tokens"),
        # The Quest-style selector of the paper's comparison: its boxes and its lists.
        c("box-select-32k", "variant", 32768, 32, 4, 128, selector="box"),
    ]


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "varlen", "varlen", "fused", "attend", "attend", "fp8", "fp8",
                       "stats", "select", "variant"])
    hq, hkv = rng.choice([(2, 1), (8, 1), (8, 8), (16, 2), (28, 4), (32, 4), (32, 4), (64, 8)])
    b = rng.choice([64, 128, 128, 256])
    layout = rng.choice(["heads", "tokens", "qkv"])
    if kind == "varlen":
        count = rng.randint(2, 24)
        seqs = [int(round(math.exp(rng.uniform(math.log(16), math.log(9000))))) for _ in range(count)]
        return dict(kind=kind, n=0, hq=hq, hkv=hkv, b=b, layout=layout, seqs=",".join(str(x) for x in seqs))
    # Full density bounds what a drawn case may cost.
    top = min(131072, int(math.sqrt(2 * MOST_PAIRS / hq)))
    n = min(top, int(round(math.exp(rng.uniform(math.log(300), math.log(top))))))
    case = dict(kind=kind, n=n, hq=hq, hkv=hkv, b=b, layout=layout)
    if kind in ("attend", "fp8"):
        case["dense"] = rng.random() < 0.3
    if kind == "attend":
        case["lse"] = rng.random() < 0.5
    if kind == "variant":
        case["selector"] = rng.choice(["box", "centroid", "full_l2"])
    return case


# ------------------------------------------------------------------ inputs

def _lengths(case):
    return [int(x) for x in case["seqs"].split(",")] if case["kind"] == "varlen" else [int(case["n"])]


def _rope(x, start=0):
    n, half = x.shape[-2], D // 2
    inv = 1.0e6 ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / D)
    ang = torch.arange(start, start + n, device=x.device, dtype=torch.float64)[:, None] * inv[None, :]
    cos, sin = ang.cos().float(), ang.sin().float()
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * cos - x2 * sin, x2 * cos + x1 * sin], dim=-1)


def _one_prompt(n, hq, hkv, b, gen):
    """Q, K, V of one prompt, fp32 [heads][n][d]."""
    def randn(*s):
        return torch.randn(*s, generator=gen, device="cuda")

    z = randn(hkv, 1, D)
    mu = 4.0 * z / z.norm(dim=-1, keepdim=True)
    m = -(-n // b)
    scale = (0.5 * randn(hkv, m)).exp().repeat_interleave(b, dim=1)[:, :n, None]
    k = _rope(randn(hkv, n, D) * scale + mu)
    q = _rope(randn(hq, n, D) + 0.1 * randn(hq, 1, D))
    v = randn(hkv, n, D) + 0.1 * randn(hkv, 1, D)
    return q, k, v


def _qkv(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    hq, hkv = case["hq"], case["hkv"]
    parts = [_one_prompt(n, hq, hkv, case["b"], gen) for n in _lengths(case)]
    q, k, v = (torch.cat([p[j] for p in parts], dim=1).to(torch.bfloat16) for j in range(3))
    del parts
    if case["layout"] == "tokens":  # [n][heads][d], as a projection's reshape leaves it
        q, k, v = (x.transpose(0, 1).contiguous().transpose(0, 1) for x in (q, k, v))
    elif case["layout"] == "qkv":   # one [n][(hq + 2 hkv) d] projection output
        buf = torch.cat([q, k, v], dim=0).transpose(0, 1).contiguous().transpose(0, 1)
        q, k, v = buf[:hq], buf[hq:hq + hkv], buf[hq + hkv:]
    return q, k, v


def _list_mask(case, seed):
    """Block lists of the kind that selection leaves, as a mask [hq][m][m]: every
    causal block (dense), or the sink, the local window and blocks that the
    heads of a group partly share, at densities that differ by head and fall
    with the prompt's length to about 5% at 128K."""
    n, hq, hkv, b = case["n"], case["hq"], case["hkv"], case["b"]
    m = -(-n // b)
    causal = torch.ones(m, m, dtype=torch.bool, device="cuda").tril()
    if case.get("dense"):
        return causal.expand(hq, m, m)
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    median = min(0.9, 0.05 * (131072 / n) ** 0.85)
    rho = (median * (0.8 * torch.randn(hq, 1, 1, generator=gen, device="cuda")).exp()).clamp(0.005, 0.95)
    shared = torch.randn(hkv, 1, m, generator=gen, device="cuda").repeat_interleave(hq // hkv, dim=0)
    score = (shared + torch.randn(hq, m, m, generator=gen, device="cuda")) / math.sqrt(2.0)
    mask = score > torch.special.ndtri(1.0 - rho.double()).float()
    i, j = torch.arange(m, device="cuda")[:, None], torch.arange(m, device="cuda")[None, :]
    return (mask | (j < N_SINK) | (j > i - N_LOCAL)) & causal


def _lists(shape, mask):
    """The mask as counts and ascending index rows (row i of a head at i (i + 1) / 2)."""
    hq, m, _ = mask.shape
    counts, indices = rbs.allocate_lists(shape)
    counts.copy_(mask.sum(dim=2, dtype=torch.int32))
    indices.fill_(-1)
    for h in range(hq):
        i, j = mask[h].nonzero(as_tuple=True)
        rank = mask[h].cumsum(dim=1)[i, j] - 1
        indices[h][i * (i + 1) // 2 + rank] = j.to(torch.int32)
    return counts, indices


def prepare(case, seed):
    q, k, v = _qkv(case, seed)
    kind, s = case["kind"], {"kind": case["kind"], "q": q, "k": k, "v": v}
    if kind == "varlen":
        s["batch"] = rbs.Batch(_lengths(case))
        s["shape"] = rbs.varlen_shape(s["batch"], case["hq"], case["hkv"], case["b"])
        s["stats"] = rbs.allocate_stats_varlen(s["shape"], s["batch"])
        s["counts"], s["indices"] = rbs.allocate_lists_varlen(s["shape"], s["batch"])
    else:
        s["shape"] = shape = rbs.make_shape(case["n"], case["hq"], case["hkv"], case["b"])
        s["stats"] = rbs.BlockStats.allocate(shape)
        if kind == "variant" and case["selector"] == "box":
            s["box"] = rbs.BoxStats.allocate(shape)
        if kind in ("attend", "fp8"):
            s["counts"], s["indices"] = _lists(shape, _list_mask(case, seed))
        else:
            s["counts"], s["indices"] = rbs.allocate_lists(shape)
    if kind not in ("attend", "fp8"):
        s["indices"].fill_(-1)  # slots past a row's count are left as they are
    if kind in ("select", "variant"):
        rbs.rbs_block_stats(s["shape"], k, s["stats"])
    if kind == "variant":
        s["selector"] = case["selector"]
        s["param"] = BOX_BUDGET if case["selector"] == "box" else TAU_BASE
    if kind == "fp8":
        s["f8"] = rbs.allocate_fp8(s["shape"])
    if kind in ("layer", "fused", "varlen", "attend", "fp8"):
        s["o"] = torch.empty_strided(tuple(q.shape), q.stride(), dtype=torch.bfloat16, device="cuda")
    s["lse"] = torch.empty(tuple(q.shape[:2]), device="cuda") if case.get("lse") else None
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    kind, shape, q, k, v = s["kind"], s["shape"], s["q"], s["k"], s["v"]
    counts, indices, stats = s["counts"], s["indices"], s["stats"]
    if kind == "layer":
        rbs.rbs_block_stats(shape, k, stats)
        rbs.rbs_select(shape, q, stats, TAU_BASE, TAU_RESCUE, N_SINK, N_LOCAL, N_RECENT, counts, indices)
        rbs.rbs_sparse_prefill(shape, q, k, v, counts, indices, O=s["o"])
        return {"o": s["o"], "counts": counts, "indices": indices}
    if kind == "fused":
        rbs.rbs_block_stats(shape, k, stats)
        rbs.rbs_select_attend(shape, q, k, v, stats, TAU_BASE, TAU_RESCUE, N_SINK, N_LOCAL, N_RECENT, counts=counts,
                              indices=indices, O=s["o"])
        return {"o": s["o"], "counts": counts, "indices": indices}
    if kind == "varlen":
        batch = s["batch"]
        rbs.rbs_block_stats_varlen(shape, batch, k, stats)
        rbs.rbs_select_varlen(shape, batch, q, stats, TAU_BASE, TAU_RESCUE, N_SINK, N_LOCAL, N_RECENT, counts,
                              indices)
        rbs.rbs_sparse_prefill_varlen(shape, batch, q, k, v, counts, indices, O=s["o"])
        return {"o": s["o"], "counts": counts, "indices": indices}
    if kind == "attend":
        rbs.rbs_sparse_prefill(shape, q, k, v, counts, indices, O=s["o"], lse=s["lse"])
        return {"o": s["o"]} if s["lse"] is None else {"o": s["o"], "lse": s["lse"]}
    if kind == "fp8":
        f8 = rbs.rbs_fp8_prepare(shape, q, k, v, s["f8"])
        rbs.rbs_sparse_prefill_fp8(shape, f8, counts, indices, O=s["o"])
        return {"o": s["o"], "amax": f8.amax, "q8": f8.Q8, "k8": f8.K8, "v8t": f8.V8t}
    if kind == "stats":
        rbs.rbs_block_stats(shape, k, stats)
        return {"centroids": stats.centroids, "radii": stats.radii, "beta": stats.beta, "quantiles": stats.quantiles}
    if kind == "select":
        rbs.rbs_select(shape, q, stats, TAU_BASE, TAU_RESCUE, N_SINK, N_LOCAL, N_RECENT, counts, indices)
        return {"counts": counts, "indices": indices}
    if kind == "variant":
        box = rbs.rbs_block_box(shape, k, s["box"]) if s["selector"] == "box" else None
        rbs.rbs_select_variant(shape, q, stats, s["selector"], s["param"], N_SINK, N_LOCAL, N_RECENT, box, counts,
                               indices)
        out = {"counts": counts, "indices": indices}
        if box is not None:
            out.update(center=box.center, half=box.half)
        return out
    raise ValueError(kind)


# ------------------------------------------------------------------ what a pass cannot do without

def _density(kind, n, b, dense):
    """Share of the causal block pairs that are executed, as measured on these inputs (rough)."""
    if dense:
        return 1.0
    if kind in ("attend", "fp8"):
        return min(0.9, 0.07 * (131072 / n) ** 0.85)
    if kind == "variant":
        return BOX_BUDGET
    at_128k, halvings = {64: (0.018, 6.5), 128: (0.29, 3.5), 256: (0.75, 3.5)}[b]
    return at_128k ** (1.0 - min(1.0, math.log2(max(1.0, 131072 / n)) / halvings))


def work(case):
    kind, hq, hkv, b = case["kind"], case["hq"], case["hkv"], case["b"]
    byt = flops = 0.0
    for n in _lengths(case):
        m = -(-n // b)
        pairs = m * (m + 1) / 2.0
        q, kv, st = 2.0 * hq * n * D, 2.0 * hkv * n * D, hkv * m * (4 * D + 8.0)
        dens = _density(kind, n, b, case.get("dense", False))
        lists = 4.0 * hq * (m + dens * pairs)
        scoring = 2.0 * hq * b * D * pairs
        attention = 4.0 * hq * b * b * D * pairs * dens
        if kind in ("layer", "varlen", "fused"):
            byt += 2 * q + 2 * kv + st + lists
            flops += scoring + attention
        elif kind == "attend":
            byt += 2 * q + 2 * kv + lists + (4.0 * hq * n if case.get("lse") else 0.0)
            flops += attention
        elif kind == "fp8":
            # The E4M3 copies are half a bf16 tensor each; the matrix core runs them at twice the bf16 rate.
            byt += 1.5 * (q + 2 * kv) + q + lists
            flops += attention / 2
        elif kind == "stats":
            byt += kv + st
        else:
            byt += q + hkv * m * D * 2.0 + lists + (kv + 2 * st if case.get("selector") == "box" else 0.0)
            flops += scoring * (2 if case.get("selector") == "box" else 1)
    return {"bytes": byt, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "stats":
        # fp32 sums of up to 256 bf16 values; beta divides a difference of two close radii.
        return {"rel": 2e-5, "max": 1e-3}
    if kind == "select":
        return {"rel": 0.0, "differ": 0.01}
    if kind == "variant":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}
    if kind == "fp8":
        # P in E4M3 (3 mantissa bits): the path is 1.0 to 1.5% from the 64-bit attention of the same E4M3 inputs.
        return {"rel": 0.03, "max": 0.5, "differ": 0.0}
    if kind == "attend":
        # bf16 P and output: 0.19% (at most 0.027 of a value) from the 64-bit attention.
        return {"rel": 0.008, "max": 0.11, "differ": 0.0}
    # Blocks near a threshold flip with the rounding of their scores (against
    # 64-bit scores 0.5 to 0.8% of the list slots and 1.3 to 2.3% of the counts
    # differ on the long prompts, where the output is 0.6% off); the same f16
    # operands summed in another order flip far fewer.
    return {"rel": 0.01, "max": 0.5, "differ": 0.01}


# ------------------------------------------------------------------ 64-bit reference

def _blocks64(k, b):
    """fp64 centroids [h][m][d] and radii [h][m] of k [h][n][d]."""
    h, n, _ = k.shape
    m = -(-n // b)
    cent = torch.empty(h, m, D, dtype=torch.float64, device=k.device)
    rad = torch.empty(h, m, dtype=torch.float64, device=k.device)
    for j in range(m):
        x = k[:, j * b:(j + 1) * b].double()
        cent[:, j] = x.mean(dim=1)
        rad[:, j] = (x - cent[:, j:j + 1]).norm(dim=2).amax(dim=1)
    return cent, rad


def _beta64(rad):
    quant = torch.stack([torch.quantile(rad, p, dim=1) for p in (0.5, 0.9)], dim=1)
    lo, hi = quant[:, :1], quant[:, 1:]
    return torch.where(hi > lo, ((rad - lo) / (hi - lo)).clamp(0, 1), (rad > lo).double()), quant


def _select64(q, cent, rad, beta, b):
    """The dual-branch selection of one prompt, as a mask [hq][m][m]."""
    hq, n, _ = q.shape
    hkv, m, _ = cent.shape
    i, j = torch.arange(m, device=q.device)[:, None], torch.arange(m, device=q.device)[None, :]
    forced = (j < N_SINK) | (j > i - N_LOCAL) | (i >= m - N_RECENT)
    masks = []
    for h in range(hq):
        g = h // (hq // hkv)
        x = q[h].double()
        logit = x @ cent[g].T / math.sqrt(D)
        up = x.norm(dim=1)[:, None] * (rad[g] * beta[g])[None, :] / math.sqrt(D)
        keep = forced
        for lg, tau in ((logit, TAU_BASE), (logit + up, TAU_RESCUE)):
            pad = torch.full((m * b - n, m), -math.inf, dtype=torch.float64, device=q.device)
            score = torch.cat([lg, pad]).view(m, b, m).logsumexp(dim=1)
            score = score.masked_fill(j > i, -math.inf)
            keep = keep | (score >= score.amax(dim=1, keepdim=True) + math.log(tau))
        masks.append(keep & (j <= i))
    return torch.stack(masks)


def _attend64(q, k, v, mask, b, want_lse=False):
    """Causal attention over the blocks of mask [hq][m][m], in fp64."""
    hq, n, _ = q.shape
    group = hq // k.shape[0]
    out = torch.empty(hq, n, D, dtype=torch.float64, device=q.device)
    lse = torch.empty(hq, n, dtype=torch.float64, device=q.device) if want_lse else None
    step = max(b, 2048 // b * b)
    pos = torch.arange(n, device=q.device)
    for h in range(hq):
        kk, vv = k[h // group].double(), v[h // group].double()
        for r0 in range(0, n, step):
            r1 = min(n, r0 + step)
            s = q[h, r0:r1].double() @ kk[:r1].T / math.sqrt(D)
            keep = mask[h, r0 // b:-(-r1 // b), :-(-r1 // b)]
            keep = keep.repeat_interleave(b, dim=0).repeat_interleave(b, dim=1)[:r1 - r0, :r1]
            s.masked_fill_(~(keep & (pos[None, :r1] <= pos[r0:r1, None])), -math.inf)
            top = s.amax(dim=1, keepdim=True)
            p = s.sub_(top).exp_()
            total = p.sum(dim=1, keepdim=True)
            out[h, r0:r1] = p @ vv[:r1] / total
            if want_lse:
                lse[h, r0:r1] = (top + total.log())[:, 0]
    return out, lse


def _e4m3_64(x, amax):
    """x quantised to E4M3 with its head's scale, and back, in fp64."""
    scale = torch.where(amax > 0, 448.0 / amax, torch.ones_like(amax))
    y = (x.float() * scale[:, None, None]).to(torch.float8_e4m3fn)
    return y.double() / scale.double()[:, None, None]


def exact(case, seed):
    kind, b = case["kind"], case["b"]
    if kind == "select" or case["hq"] * sum(x * x for x in _lengths(case)) > MOST_EXACT and kind not in ("stats", "variant"):
        return None
    if kind == "variant" and case["selector"] != "box":
        return None
    q, k, v = _qkv(case, seed)
    if kind == "stats":
        cent, rad = _blocks64(k, b)
        beta, quant = _beta64(rad)
        return {"centroids": cent, "radii": rad, "beta": beta, "quantiles": quant}
    if kind == "variant":
        n, m = case["n"], -(-case["n"] // b)
        lo = torch.stack([k[:, j * b:(j + 1) * b].double().amin(dim=1) for j in range(m)], dim=1)
        hi = torch.stack([k[:, j * b:(j + 1) * b].double().amax(dim=1) for j in range(m)], dim=1)
        return {"counts": None, "indices": None, "center": (lo + hi) / 2, "half": (hi - lo) / 2}
    if kind == "attend":
        o, lse = _attend64(q, k, v, _list_mask(case, seed), b, bool(case.get("lse")))
        return {"o": o} if lse is None else {"o": o, "lse": lse}
    if kind == "fp8":
        amax = [x.abs().float().amax(dim=(1, 2)) for x in (q, k, v)]
        q, k, v = (_e4m3_64(x, a) for x, a in zip((q, k, v), amax))
        return {"o": _attend64(q, k, v, _list_mask(case, seed), b)[0], "amax": torch.cat(amax).double(), "q8": None,
                "k8": None, "v8t": None}
    parts, t = [], 0
    for n in _lengths(case):
        qs, ks, vs = (x[:, t:t + n] for x in (q, k, v))
        cent, rad = _blocks64(ks, b)
        beta, _ = _beta64(rad)
        parts.append(_attend64(qs, ks, vs, _select64(qs, cent, rad, beta, b), b)[0])
        t += n
    return {"o": torch.cat(parts, dim=1), "counts": None, "indices": None}
