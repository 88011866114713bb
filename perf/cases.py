"""Performance cases of the compressed-KV path: what a program that serves a
model with this cache calls, over the sizes it meets.

Kinds of cases, each a pass through the package's public entry points:

* ``decode``   - one decode step: every layer's attention over the compressed
                 cache of a batch (``CompressedCache.decode``).  Layers run in
                 the order even, then odd, so that the planes a block's layers
                 share are not still in the last-level cache: in a model the
                 weights of a layer pass through it between two layers.
* ``generate`` - one decode step while a sequence grows: every layer's append
                 to the exact tail and its attention over the prefix, the
                 refreshed spans and the tail (``Generation``).
* ``probe``    - the routing losses of a prompt (``probe``).
* ``compress`` - a prompt's cache written for given modes
                 (``CompressedCache.compress``).
* ``prefill``  - a prompt as a whole, up to its first step of attention: probe, routing under
                 a byte budget, allocation, compress, every layer's decode.
"""
import math
import random

import numpy as np
import torch

from paper_2607_06519_amd import binding as B
from paper_2607_06519_amd.cache import CompressedCache, Generation, probe

SHARED, RESIDUAL, EXACT = 0, 1, 2
MIX = (0.50, 0.35, 0.15)          # shares of shared, residual and exact heads
NEEDLES, NEEDLE_AMP, NEEDLE_CHANNELS = 16, 5.0, 16
MOST = 8_400_000                  # tokens x layers x KV heads of a drawn case

# Shapes of the 8B model (32 query heads on 8 KV heads of 128 channels) and of
# the 70B one (64 on 8).  A case may take fewer layers than its model, a
# pipeline stage's share; its cache is still several times the last-level cache.
M8B = dict(layers=32, kv=8, group=4, d=128, topk=16, dtype="bf16", schedule=0, res_ppm=-1, batch=1, probes=256, graph=False)


def listed():
    def case(name, kind, **over):
        c = dict(M8B, name=name, kind=kind, tmin=32768, tmax=32768)
        c.update(over)
        return c

    return [
        # the smallest call: a small fp32 cache, bound by latency and launches
        case("decode_tiny_f32", "decode", layers=2, kv=4, group=1, d=64, topk=8, dtype="f32", tmin=512, tmax=512),
        # a short chat turn, one sequence, odd length, the step captured in a graph as a server does
        case("decode_8b_1k", "decode", tmin=1001, tmax=1001, graph=True),
        # the long-context step that the benchmark quotes
        case("decode_8b_32k", "decode"),
        # the same with FP8 coefficients
        case("decode_8b_fp8_32k", "decode", dtype="bf16_e4m3", layers=16),
        # the paper's block setting: pairs at both ends, blocks of four between
        case("decode_8b_mixed_32k", "decode", schedule=1, layers=16),
        # a batch of sequences of unlike lengths
        case("decode_8b_batch16", "decode", layers=8, batch=16, tmin=4096, tmax=16384),
        # the longest context, eight query heads to a KV head
        case("decode_70b_131k", "decode", layers=8, group=8, tmin=131072, tmax=131072),
        # a step of a chat that has outgrown its prompt: two refreshed spans and a tail
        case("generate_8b_4k", "generate", tmin=4096, tmax=4096, cap=512, tail=257, spans=2),
        # the parts of prefill: losses, then the cache (reusing the probe's selections)
        case("probe_8b_32k", "probe"),
        case("compress_8b_32k", "compress", layers=16, reuse=True),
        # prefill as a whole: the paper's block setting on a ragged prompt; token-level sets
        case("prefill_8b_mixed_12k", "prefill", schedule=1, tmin=12345, tmax=12345),
        case("prefill_8b_tokset_32k", "prefill", layers=16, topk=0, res_ppm=50000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["generate", "probe", "compress", "prefill", "prefill"])
    c = dict(M8B, kind=kind)
    c["schedule"] = rng.choice([0, 0, 0, 1, 2])
    c["layers"] = rng.choice({0: [2, 4, 8, 16, 32], 1: [12, 16, 32], 2: [4, 8, 16, 32]}[c["schedule"]])
    c["kv"] = rng.choice([2, 4, 8, 8, 8])
    c["group"] = rng.choice([1, 2, 4, 4, 8])
    c["d"] = rng.choice([64, 128, 128, 128])
    c["topk"] = rng.choice([c["d"] // 8] * 4 + [5, 24])
    c["dtype"] = rng.choice(["bf16"] * 4 + ["bf16_e4m3"] * 2 + ["f32"])
    if rng.random() < 0.2:
        c["topk"], c["res_ppm"] = 0, rng.choice([10000, 50000, 100000])
    cap = MOST // (8 if c["dtype"] == "f32" or c["topk"] in (5, 24) else 1) // (c["layers"] * c["kv"])
    if kind == "decode":
        c["batch"] = rng.choice([1, 1, 1, 2, 4, 16])
        c["graph"] = rng.random() < 0.5
    elif kind == "generate":
        c["batch"] = rng.choice([1, 1, 2])
        c["cap"] = rng.choice([128, 256, 512])
        c["tail"] = rng.randint(0, c["cap"] - 1)
        c["spans"] = rng.choice([0, 1, 2, 4])
    elif kind == "compress":
        c["reuse"] = rng.random() < 0.7
        cap //= 2
    elif kind == "prefill":
        cap //= 3
    if kind in ("probe", "prefill") and c["res_ppm"] >= 0:
        cap //= 2
    if kind in ("probe", "compress", "prefill"):
        c["probes"] = rng.choice([32, 100, 256])
    c["tmax"] = _log_int(rng, 100, max(200, min(131072, cap // c["batch"])))
    c["tmin"] = max(1, c["tmax"] // 4) if c["batch"] > 1 else c["tmax"]
    return c


# ---------------------------------------------------------------- what a case holds
def _dims(c):
    tok = c["res_ppm"] >= 0
    return B.dims(c["layers"], c["kv"], c["kv"] * c["group"], c["d"], c["topk"], c["dtype"], c["schedule"],
                  B.RES_TOKENS if tok else B.RES_CHANNELS, c["res_ppm"] if tok else 0)


def _sizes(c):
    n = c["layers"]
    return {0: [2] * (n // 2), 1: [2, 2] + [4] * ((n - 8) // 4) + [2, 2], 2: [4] * (n // 4)}[c["schedule"]]


def _blocks(c):
    first, out = 0, []
    for b in _sizes(c):
        out.append((first, b))
        first += b
    return out


def _lens(c, seed):
    r = random.Random("lens %d" % seed)
    return [r.randint(c["tmin"], c["tmax"]) for _ in range(c["batch"])]


def _mix_modes(c, n, seed):
    """Seeded modes of ``n`` sequences [n][blocks][kv] in the shares of MIX."""
    r, sizes = random.Random("modes %d" % seed), np.array(_sizes(c))
    out = np.empty((n, len(sizes), c["kv"]), dtype=np.uint8)
    for i in range(n):
        for size in (2, 4):           # the shares in each block size: the cache's bytes are the same for every seed
            units = int((sizes == size).sum()) * c["kv"]
            s, e = round(MIX[0] * units), round(MIX[2] * units)
            m = [SHARED] * s + [EXACT] * e + [RESIDUAL] * (units - s - e)
            r.shuffle(m)
            out[i, sizes == size] = np.array(m, dtype=np.uint8).reshape(-1, c["kv"])
    return out


def _gen(seed, *tags):
    return torch.Generator("cuda").manual_seed(random.Random("%d %s" % (seed, tags)).getrandbits(62))


def _in_type(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _block_inputs(c, seed, T, tag, size, b):
    """K and V of the layers of block ``b``, each [size][kv][T][d]: along depth a
    first-order autoregression, one correlation per head, with needle tokens
    whose channels spike in one of the layers."""
    g = _gen(seed, tag, b)
    d, kv = c["d"], c["kv"]
    rho = (0.75 + 0.20 * torch.rand(kv, 1, 1, generator=g, device="cuda"))
    x = torch.empty(2, size, kv, T, d, dtype=_in_type(c), device="cuda")
    y = torch.randn(2, kv, T, d, generator=g, device="cuda")
    x[:, 0] = y
    for n in range(1, size):
        y = rho * y + (1 - rho * rho).sqrt() * torch.randn(2, kv, T, d, generator=g, device="cuda")
        x[:, n] = y
    m = min(NEEDLES, T)
    pos = torch.randperm(T, generator=g, device="cuda")[:m].view(1, m, 1)
    chan = torch.rand(kv, m, d, generator=g, device="cuda").argsort(-1)[..., :NEEDLE_CHANNELS]
    layer = torch.randint(size, (kv, m, 1), generator=g, device="cuda")
    x[:, layer, torch.arange(kv, device="cuda").view(kv, 1, 1), pos, chan] += NEEDLE_AMP
    return x


def _inputs(c, seed, T, tag):
    """Per-layer lists of K and V, each [kv][T][d]."""
    k, v = [], []
    for b, size in enumerate(_sizes(c)):
        x = _block_inputs(c, seed, T, tag, size, b)
        k += list(x[0])
        v += list(x[1])
    return k, v


def _rows(c, seed, n, tag, scale=1.0):
    """[layers][n][kv * group][d] query rows."""
    g = _gen(seed, tag)
    x = torch.randn(c["layers"], n, c["kv"] * c["group"], c["d"], generator=g, device="cuda") * scale
    return x.to(_in_type(c))


def _probe_rows(c, seed, n, tag="probe"):
    """Per layer [heads][n][d] probe rows."""
    g = _gen(seed, tag)
    x = torch.randn(c["layers"], c["kv"] * c["group"], n, c["d"], generator=g, device="cuda") / math.sqrt(c["d"])
    return list(x.to(_in_type(c)))


def _budget(c, T, seed):
    """The byte budget of a sequence of T tokens: what the shares of MIX take."""
    return B.layout(_dims(c), [T], _mix_modes(c, 1, seed))[1]


def _order(c):
    return list(range(0, c["layers"], 2)) + list(range(1, c["layers"], 2))


def _filled_cache(c, seed, lens, modes, dims):
    """A cache of the sequences, compressed as after their prefill."""
    cache = CompressedCache(dims, lens, modes)
    for s, T in enumerate(lens):
        k, v = _inputs(c, seed, T, s)
        extra = None
        if c["res_ppm"] >= 0:
            _, extra = probe(dims, T, k, _probe_rows(c, seed, 32, ("set", s)), 32)
        cache.compress(s, k, v, token_scores=extra)
    return cache


def prepare(case, seed):
    c = case
    dims = _dims(c)
    lens = _lens(c, seed)
    st = dict(case=c, dims=dims, lens=lens)
    if c["kind"] in ("decode", "generate"):
        modes = _mix_modes(c, c["batch"], seed)
        st["cache"] = _filled_cache(c, seed, lens, modes, dims)
        st["q"] = _rows(c, seed, c["batch"], "q")
        st["out"] = torch.empty_like(st["q"])
    if c["graph"]:
        _decode_step(st)
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            _decode_step(st)
    if c["kind"] == "generate":
        gen = Generation(dims, st["cache"], c["cap"])
        for i in range(c["spans"] + 1):
            n = c["cap"] if i < c["spans"] else c["tail"]
            for l, (k, v) in enumerate(_tail_rows(c, seed, i, n)):
                gen.tail_k[l][:, :, :n] = k
                gen.tail_v[l][:, :, :n] = v
            if i < c["spans"]:
                gen.n_tail = n
                rows = [torch.stack(r) for r in zip(*(_probe_rows(c, seed, 32, ("span", i, s)) for s in range(c["batch"])))]
                gen.refresh(rows, 32, budget_bytes=_budget(c, n, seed + i))
            else:
                for _ in range(n):
                    gen.advance()
        st["gen"] = gen
        st["new"] = [t.view(c["layers"], c["batch"], c["kv"], c["d"]) for t in _new_rows(c, seed)]
    if c["kind"] in ("probe", "compress", "prefill"):
        st["k"], st["v"] = _inputs(c, seed, lens[0], 0)
        st["rows"] = _probe_rows(c, seed, c["probes"])
    if c["kind"] == "probe":
        st["v"] = None
    if c["kind"] == "compress":
        st["extra"] = None
        if c["reuse"] or c["res_ppm"] >= 0:
            _, st["extra"] = probe(dims, lens[0], st["k"], st["rows"], c["probes"])
        st["cache"] = CompressedCache(dims, lens, _mix_modes(c, 1, seed))
        st["cache"].buf.zero_()          # the padding between planes comes back with the rest
    if c["kind"] == "prefill":
        st["budget"] = _budget(c, lens[0], seed)
        st["q"] = _rows(c, seed, 1, "q")
        st["out"] = torch.empty_like(st["q"])
    return st


def _tail_rows(c, seed, i, n):
    """Per layer the K and V rows [batch][kv][n][d] that the i-th tail holds."""
    if n == 0:
        return []
    per = [_inputs(c, seed, n, ("tail", i, s)) for s in range(c["batch"])]
    return [(torch.stack([k[l] for k, _ in per]), torch.stack([v[l] for _, v in per])) for l in range(c["layers"])]


def _new_rows(c, seed):
    g = _gen(seed, "new")
    return torch.randn(2, c["layers"], c["batch"], c["kv"], c["d"], generator=g, device="cuda").to(_in_type(c))


def _decode_step(state):
    for l in _order(state["case"]):
        state["cache"].decode(l, state["q"][l], out=state["out"][l])


def run(state):
    c, dims = state["case"], state["dims"]
    if c["kind"] == "decode":
        if c["graph"]:
            state["graph"].replay()
        else:
            _decode_step(state)
        return state["out"]
    if c["kind"] == "generate":
        gen, (k, v) = state["gen"], state["new"]
        for l in range(c["layers"]):
            gen.append(l, k[l], v[l])
            gen.decode(l, state["q"][l], out=state["out"][l])
        return state["out"]
    if c["kind"] == "probe":
        errors, extra = probe(dims, state["lens"][0], state["k"], state["rows"], c["probes"])
        return {"errors": errors, "scores": extra} if c["res_ppm"] >= 0 else {"errors": errors}
    tok = c["res_ppm"] >= 0
    if c["kind"] == "compress":
        cache, extra = state["cache"], state["extra"]
        cache.compress(0, state["k"], state["v"], token_scores=extra if tok else None, k_select=None if tok else extra)
        return cache.buf[: cache.total_bytes]
    T = state["lens"][0]
    errors, extra = probe(dims, T, state["k"], state["rows"], c["probes"])
    modes, _, _ = B.route(dims, T, errors.cpu().numpy(), budget_bytes=state["budget"], allow_infeasible=True)
    cache = CompressedCache(dims, [T], modes)
    cache.compress(0, state["k"], state["v"], token_scores=extra if tok else None, k_select=None if tok else extra)
    for l in range(c["layers"]):
        cache.decode(l, state["q"][l], out=state["out"][l])
    return {"errors": errors, "modes": modes, "out": state["out"]}


# ---------------------------------------------------------------- the work of a pass
def _coef(c):
    return {"f32": 4, "bf16": 2, "bf16_e4m3": 1}[c["dtype"]]


def _elem(c):
    return 4 if c["dtype"] == "f32" else 2


def _mix_bytes(c, size):
    """Per token and KV head: bytes that a layer's decode reads, and bytes of the block's cache, in the shares of MIX."""
    d, e, f, k = c["d"], _elem(c), _coef(c), c["topk"]
    ent = 2 * k * (f + (1 if size == 2 else 2))
    if c["res_ppm"] >= 0:
        ent = 2 * (size - 1) * d * f * c["res_ppm"] / 1e6
    read = MIX[0] * 2 * d * f + MIX[1] * (2 * d * f + ent) + MIX[2] * 2 * d * e
    held = MIX[0] * 2 * d * f + MIX[1] * (2 * d * f + ent) + MIX[2] * 2 * d * e * size
    return read, held


def work(case):
    c = case
    d, e, kv, layers, G = c["d"], _elem(c), c["kv"], c["layers"], c["group"]
    tokens = c["batch"] * (c["tmin"] + c["tmax"]) / 2
    if c["kind"] == "generate":
        tokens += c["batch"] * c["spans"] * c["cap"]
    dec = sum(size * kv * tokens * _mix_bytes(c, size)[0] for size in _sizes(c)) + 2 * layers * c["batch"] * kv * G * d * e
    dec_flops = 4 * layers * kv * G * d * tokens
    if c["kind"] == "decode":
        return {"bytes": int(dec), "flops": int(dec_flops)}
    if c["kind"] == "generate":
        tail = layers * kv * c["batch"] * (c["tail"] + 1)
        return {"bytes": int(dec + tail * 2 * d * e), "flops": int(dec_flops + 4 * tail * G * d)}
    keys = layers * kv * tokens * d * e
    rows = layers * kv * G * c["probes"] * d * e
    if c["res_ppm"] >= 0:
        look = 2 * layers * kv * G * c["probes"] * tokens * d       # a maximum over the rows: every logit
    else:
        # the Gram matrices of the deviations: half of d x d, shared and residual, one a pair, four a block of four
        look = sum(kv * tokens * 2 * d * d * (1 if size == 2 else 4) for size in _sizes(c))
    wrote = sum(kv * tokens * _mix_bytes(c, size)[1] for size in _sizes(c))
    if c["kind"] == "probe":
        return {"bytes": int(keys + rows), "flops": int(look)}
    if c["kind"] == "compress":
        return {"bytes": int(2 * keys + wrote), "flops": int(2 * layers * kv * tokens * d)}
    return {"bytes": int(3 * keys + rows + wrote + dec), "flops": int(look + dec_flops)}


def tolerance(case):
    if case["kind"] == "compress":
        return "exact"                # bytes
    tok = case["res_ppm"] >= 0        # its scores are of deviations rounded to bf16, in fp32 caches too
    if tok and (case["dtype"] == "f32" or case["kind"] == "probe"):
        return {"rel": 5e-3, "max": 0.1}
    if case["dtype"] == "f32" or case["kind"] == "probe":
        return {"rel": 1e-5, "max": 4e-4}
    return {"rel": 1e-2, "max": 0.1}  # outputs in bf16, of probabilities in bf16


# ---------------------------------------------------------------- the same in 64 bits
def _dct4():
    n = torch.arange(4, dtype=torch.float64, device="cuda")
    return torch.stack([torch.cos(math.pi * (2 * n + 1) * j / 8) / math.sqrt(2) for j in range(4)])


def _stored(c, x):
    """A coefficient as the cache holds it."""
    if c["dtype"] == "f32":
        return x.float().double()
    if c["dtype"] == "bf16":
        return x.to(torch.bfloat16).double()
    return x.float().clamp(-448, 448).to(torch.float8_e4m3fn).double()


def _top(key, k):
    """Mask of the k largest along the last axis, ties to the lower index."""
    at = key.sort(dim=-1, descending=True, stable=True)[1][..., :k]
    return torch.zeros_like(key, dtype=torch.bool).scatter_(-1, at, True)


def _high(c, x):
    """Of one tensor [B][T][d] (64 bits): the high-frequency coefficients [T][d][B-1], the mask of those that a
    token keeps, and each layer's weights [B][B-1]."""
    if len(x) == 2:
        z = ((x[0] - x[1]) / 2).unsqueeze(-1)
        key = (x[0].float() - x[1].float()).abs()
        w = torch.tensor([[1.0], [-1.0]], dtype=torch.float64, device="cuda")
    else:
        f = _dct4()
        z = torch.stack([sum(f[j][n] * x[n] for n in range(4)) for j in (1, 2, 3)], -1)
        key = z.abs().flatten(1)
        w = f[1:].T
    return z, _top(key, c["topk"]).view(z.shape), w


def _rebuild(c, x, mode, kept=None):
    """The layers of one head's tensor [B][T][d] as decode sees them; ``kept``: mask [T] of a token-level set."""
    if mode == EXACT:
        return x
    y = _stored(c, x.mean(0)).expand_as(x)
    if mode == SHARED:
        return y
    if kept is None:
        z, keep, w = _high(c, x)
    else:
        z, _, w = _high(dict(c, topk=0), x)
        keep = kept.view(-1, 1, 1)
    z = _stored(c, z) * keep
    return y + torch.stack([(z * w[p]).sum(-1) for p in range(len(x))])


def _loss(c, k, q):
    """Eq. (2) of one head's keys [B][T][d] and probe rows [B][R][d]: shared, residual, and the token set's mask."""
    size, T, d = k.shape
    dev = k.mean(0) - k
    norm = size * q.shape[1] * d

    def gram(dv):
        return float(sum(((dv[p].T @ dv[p]) * (q[p].T @ q[p])).sum() for p in range(size))) / norm

    if c["res_ppm"] < 0:
        z, keep, w = _high(c, k)
        return gram(dev), gram(dev + torch.stack([(z * keep * w[p]).sum(-1) for p in range(size)])), None, None
    score = torch.zeros(T, dtype=torch.float64, device="cuda")
    share = torch.zeros_like(score)
    for p in range(size):
        for t in range(0, T, 8192):
            a = dev[p][t:t + 8192] @ q[p].T.contiguous()
            score[t:t + 8192] = torch.maximum(score[t:t + 8192], a.abs().amax(1))
            share[t:t + 8192] += (a * a).sum(1)
    kept = _top(score, -(-T * c["res_ppm"] // 1000000))
    return float(share.sum()) / norm, float(share[~kept].sum()) / norm, score, kept


def _plane(n):
    return -(-n // 256) * 256


def _unit_bytes(c, T, size):
    d, e, f = c["d"], _elem(c), _coef(c)
    coef = _plane(-(-T * d // 1024) * 1024) if f == 1 else _plane(T * d * f)
    if c["res_ppm"] >= 0:
        n = -(-T * c["res_ppm"] // 1000000)
        ent = _plane(-(-T // 32) * 4) + _plane((-(-T // 128) + 1) * 4) + 2 * _plane(n * (size - 1) * d * f)
    else:
        ent = 2 * _plane(T * c["topk"] * (1 if size == 2 else 2)) + 2 * _plane(T * c["topk"] * f)
    return [2 * coef, 2 * coef + ent, 2 * size * _plane(T * d * e)]


def _omega(c, size):
    d, e, f, k = c["d"], _elem(c), _coef(c), c["topk"]
    ent = 2 * k * (f + (1 if size == 2 else 2))
    if c["res_ppm"] >= 0:
        ent = 2 * (size - 1) * d * f * c["res_ppm"] / 1e6 + 1 / 8 + 4 / 128
    full = 2 * size * d * e
    return [2 * d * f / full, (2 * d * f + ent) / full, 1.0]


def _route(c, T, errors, budget):
    """Modes [blocks][kv] at the smallest penalty that fits the budget."""
    sizes = np.repeat(_sizes(c), c["kv"])
    E = np.concatenate([errors.reshape(-1, 2), np.zeros((len(sizes), 1))], 1)
    om = np.array([_omega(c, s) for s in sizes])
    held = np.array([_unit_bytes(c, T, s) for s in sizes])
    cuts = {0.0, math.inf}
    pairs = [(0, 1), (0, 2), (1, 2)]
    at = {}
    for a, b in pairs:
        lo = om[:, a] <= om[:, b]
        with np.errstate(divide="ignore", invalid="ignore"):
            cut = (np.where(lo, E[:, a], E[:, b]) - np.where(lo, E[:, b], E[:, a])) / np.abs(om[:, b] - om[:, a])
        at[a, b] = (lo, cut)
        cuts |= {float(x) for x in cut if x > 0 and math.isfinite(x)}
    rows = np.arange(len(sizes))

    def better(x, y, lam):
        out = np.empty(len(sizes), dtype=int)
        for a, b in pairs:
            here = (x == a) & (y == b)
            lo, cut = at[a, b]
            out[here] = np.where((lam >= cut) == lo, a, b)[here]
        return out

    for lam in sorted(cuts):
        best = better(better(np.full(len(sizes), 0), np.full(len(sizes), 1), lam), np.full(len(sizes), 2), lam)
        if held[rows, best].sum() <= budget:
            return best.reshape(-1, c["kv"])
    return np.zeros((len(_sizes(c)), c["kv"]), dtype=int)


def _attend(q, ks, vs):
    """softmax(q K^T / sqrt(d)) V of one head: q [G][d], lists of rows."""
    k, v = torch.cat(ks), torch.cat(vs)
    p = torch.softmax(k @ q.T.contiguous() / math.sqrt(q.shape[1]), 0)
    return p.T.contiguous() @ v


def _heads(x, h, G):
    return x[h * G:(h + 1) * G].double()


def exact(case, seed):
    c = case
    if c["kind"] == "compress":
        return None
    lens, kv, G = _lens(c, seed), c["kv"], c["group"]
    blocks, sizes = _blocks(c), _sizes(c)
    if c["kind"] in ("probe", "prefill"):
        rows = _probe_rows(c, seed, c["probes"])
        T = lens[0]
        E = np.zeros((len(blocks), kv, 2))
        score, sets = [], {}
        for b, (first, size) in enumerate(blocks):
            x = _block_inputs(c, seed, T, 0, size, b)[0]
            for h in range(kv):
                q = torch.stack([_heads(rows[first + p], h, G).flatten(0, 1) for p in range(size)])
                es, er, s, kept = _loss(c, x[:, h].double(), q)
                E[b, h] = es, er
                score.append(s)
                sets[b, h] = kept
        if c["kind"] == "probe":
            if c["res_ppm"] < 0:
                return {"errors": E}
            return {"errors": E, "scores": torch.stack(score).view(len(blocks), kv, T)}
        modes = [_route(c, T, E, _budget(c, T, seed))]
        q = _rows(c, seed, 1, "q")
    else:
        modes, q = _mix_modes(c, c["batch"], seed), _rows(c, seed, c["batch"], "q")
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    for s, T in enumerate(lens):
        if c["kind"] != "prefill":
            sets = _set_masks(c, seed, T, s, ("set", s), s)
        parts = [(T, modes[s], sets, s)]
        if c["kind"] == "generate":
            for i in range(c["spans"]):
                tag, n = ("tail", i, s), c["cap"]
                E, kept = _span_loss(c, seed, n, tag, ("span", i, s))
                parts.append((n, _route(c, n, E, _budget(c, n, seed + i)), kept, tag))
            if c["tail"]:
                parts.append((c["tail"], np.full((len(blocks), kv), EXACT), {}, ("tail", c["spans"], s)))
            new = _new_rows(c, seed)
        for b, (first, size) in enumerate(blocks):
            xs = [_block_inputs(c, seed, n, tag, size, b) for n, _, _, tag in parts]
            for h in range(kv):
                k, v = ([_rebuild(c, x[t][:, h].double(), m[b][h], kept.get((b, h))) for x, (_, m, kept, _) in zip(xs, parts)]
                        for t in (0, 1))
                for p in range(size):
                    ks, vs = [x[p] for x in k], [x[p] for x in v]
                    if c["kind"] == "generate":
                        ks.append(new[0][first + p, s, h:h + 1].double())
                        vs.append(new[1][first + p, s, h:h + 1].double())
                    out[first + p, s, h * G:(h + 1) * G] = _attend(_heads(q[first + p, s], h, G), ks, vs)
    return {"errors": E, "modes": None, "out": out} if c["kind"] == "prefill" else out


def _span_loss(c, seed, n, tag, row_tag):
    """Losses [blocks][kv][2] and token sets of one sequence's inputs ``tag`` under 32 probe rows."""
    rows = _probe_rows(c, seed, 32, row_tag)
    E, kept = np.zeros((len(_sizes(c)), c["kv"], 2)), {}
    for b, (first, size) in enumerate(_blocks(c)):
        x = _block_inputs(c, seed, n, tag, size, b)[0]
        for h in range(c["kv"]):
            q = torch.stack([_heads(rows[first + p], h, c["group"]).flatten(0, 1) for p in range(size)])
            es, er, _, kept[b, h] = _loss(c, x[:, h].double(), q)
            E[b, h] = es, er
    return E, kept


def _set_masks(c, seed, T, s, row_tag, tag):
    return _span_loss(c, seed, T, tag, row_tag)[1] if c["res_ppm"] >= 0 else {}
