"""The work that a rollout does with this framework, as cases that can be timed
and compared: SD steps (eager and as a replayed HIP graph), their drafts and
verifies alone, autoregressive steps, prompt prefill, the drafter refresh of a
training step and the rejection sampler, on the decoder shapes of
paper_2606_18967_amd/synth.py (four layers of the 8B and the 32B shape, so that
a state is small and rounding does not travel through a whole model).

Inputs stand for a trained policy: the residual branches are scaled as decoders
are initialised (output and down projections by 1/sqrt(2 layers)), and the LM
head points each token's embedding at a successor, so that the next-token
distribution is peaked, the drafter agrees with the target most of the time,
and a draw does not hang on the last bit of a logit.  Contexts are N(0, 1) keys
(post-RoPE) and values.  Lengths follow from the case alone.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

from paper_2606_18967_amd import sdrl, synth

MODELS = {"tiny": synth.TINY, "8b": synth.L4_8B, "32b": synth.L64_32B}
FMTS = ("w4", "w4a", "w8")
T = 1.0
STEP = 3                       # the Philox key's second word; the first is the seed


def case(name, op, model, layers, B, ctx, spread=1, gamma=4, fmt="w4", page=0, slots=0, cap=0):
    """op: sd_step, sd_graph, draft, verify, ar, prefill, refresh or accept.  B live sequences (slots, the
    engine's capacity, may be more) whose cached lengths are spread evenly over ctx (1 +- spread / 2);
    cap: the cache's positions per slot where they are more than the step needs; page: page size or 0."""
    return dict(name=name, op=op, model=model, layers=layers, B=B, ctx=ctx, spread=spread, gamma=gamma, fmt=fmt,
                page=page, slots=max(slots, B), cap=cap)


def listed():
    return [
        # the smallest call: one SD step of the two-layer fp32 decoder (launches and latency)
        case("tiny sd step", "sd_step", "tiny", 2, 4, 64, spread=0),
        # one live sequence, the last of a rollout's long tail, decoded without SD
        case("8b ar step b1", "ar", "8b", 4, 1, 2048),
        # SD in the tail of a long-tailed rollout, as a replayed graph: few live rows, a cache with room for 16k
        case("8b sd graph b4", "sd_graph", "8b", 4, 4, 3000, gamma=5, slots=8, cap=16384),
        # drafts of an odd batch with ragged contexts
        case("8b draft b13", "draft", "8b", 4, 13, 3001, gamma=7, slots=16, cap=8192),
        # verify of a middle batch: 128 rows
        case("8b verify b16", "verify", "8b", 4, 16, 4096, gamma=7, cap=8192),
        # the bulk of a rollout, before SD turns on: autoregressive steps of a large batch
        case("8b ar step b200", "ar", "8b", 4, 200, 1024),
        # the headline workload's drafts and verify, on four of its layers
        case("32b draft b64", "draft", "32b", 4, 64, 8192, spread=0),
        case("32b verify b64", "verify", "32b", 4, 64, 8192, spread=0),
        # prompts of different lengths into an empty cache (an engine that drafts up to 11 tokens)
        case("8b prefill b24", "prefill", "8b", 4, 24, 341, gamma=11),
        # the drafter refresh at the start of a training step
        case("8b refresh", "refresh", "8b", 4, 1, 64),
        # rejection sampling alone, at the 32B vocabulary
        case("accept b64", "accept", "32b", 1, 64, 1000),
        # an SD step with the int8 drafter on a paged cache, odd batch
        case("8b sd step paged w8 b37", "sd_step", "8b", 4, 37, 1500, gamma=3, fmt="w8", page=64),
    ]


def draw(rng):
    most = [work(c) for c in listed() if c["op"] in ("draft", "prefill")]
    while True:
        op = rng.choice(["sd_step", "sd_step", "draft", "verify", "ar", "ar", "prefill", "refresh", "accept", "sd_graph"])
        model = rng.choice(["8b", "8b", "8b", "32b", "32b", "tiny"])
        gamma = rng.randint(1, 11)
        B = int(round(math.exp(rng.uniform(0, math.log(256 if op == "ar" else 64)))))
        ctx = int(round(math.exp(rng.uniform(math.log(40), math.log(1000 if op == "prefill" else 8192)))))
        c = case("", op, model, rng.randint(2, 4), B, ctx, spread=rng.choice([0, 1]), gamma=gamma,
                 fmt=rng.choice(["w4", "w4", "w4a", "w8"]), page=rng.choice([0, 0, 32, 64, 128]),
                 slots=B + rng.choice([0, 0, 3]), cap=rng.choice([0, 0, 2 * ctx + 64]))
        del c["name"]
        w = work(c)
        if c["slots"] * capacity(c) > 64 * 8192 + 4096 or B * (gamma + 1) > 640:
            continue
        if op == "prefill" and cache_size(c) > SMALL:           # its outputs
            continue
        if w["bytes"] <= max(m["bytes"] for m in most) and w["flops"] <= max(m["flops"] for m in most):
            return c


# ------------------------------------------------------------------ shapes
def config(c):
    return dict(MODELS[c["model"]], n_layers=c["layers"])


def lengths(c):
    """Cached length (prefill: prompt length) of each live sequence, in an order that mixes long and short."""
    B = c["B"]
    if B == 1 or not c["spread"]:
        return [c["ctx"]] * B
    even = [max(1, int(c["ctx"] * (1 - c["spread"] / 2 + c["spread"] * i / (B - 1)))) for i in range(B)]
    step = next(s for s in range(B // 2 + 1, 2 * B) if math.gcd(s, B) == 1)
    return [even[i * step % B] for i in range(B)]


def capacity(c):
    need = max(lengths(c)) + c["gamma"] + 2
    return max(need, c["cap"])


def pages_of(c):
    """Pages per slot of a paged cache."""
    return -(-capacity(c) // c["page"])


SMALL = 1 << 26                # elements of a K cache that is compared whole


def cache_size(c):
    cfg = config(c)
    per_slot = pages_of(c) * c["page"] if c["page"] else capacity(c)
    return c["slots"] * per_slot * cfg["n_layers"] * cfg["n_kv"] * cfg["head_dim"]


def weight_count(cfg):
    H, d, F = cfg["hidden"], cfg["head_dim"], cfg["ffn"]
    return (cfg["n_q"] + 2 * cfg["n_kv"]) * d * H + H * cfg["n_q"] * d + 3 * F * H


def work(c):
    cfg = config(c)
    el = 2 if cfg["dtype"] == "bf16" else 4
    H, V, L, B, g = cfg["hidden"], cfg["vocab"], cfg["n_layers"], c["B"], c["gamma"]
    kv = 2 * cfg["n_kv"] * cfg["head_dim"] * el                  # cache bytes of a position of one layer
    lens = lengths(c)
    nw = weight_count(cfg)
    q_el = (1 if c["fmt"] == "w8" else 0.5) + 2 / 128 + (1 / 128 if c["fmt"] == "w4a" else 0)

    def fwd(per_weight, n, off):
        read = sum(s + off + n for s in lens)
        rows = B * n
        att = sum(s + off + i + 1 for s in lens for i in range(n))
        return (L * nw * per_weight + V * H * el + rows * (H * el + 4 * V) + L * kv * (read + rows),
                2 * rows * (L * nw + V * H) + 4 * L * cfg["n_q"] * cfg["head_dim"] * att)

    def total(parts):
        return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}

    drafts = [fwd(q_el, 1, j) for j in range(g)]
    verify = [fwd(el, g + 1, 0)]
    accept = [(4 * V * B * (g + 1) + 4 * V * B, 10 * V * B * (g + 2))]
    op = c["op"]
    if op in ("sd_step", "sd_graph"):
        return total(drafts + verify + [(4 * V * B, 10 * V * B)])
    if op == "draft":
        return total(drafts)
    if op == "verify":
        return total(verify)
    if op == "ar":
        return total([fwd(el, 1, 0)])
    if op == "accept":
        return total(accept)
    if op == "refresh":
        return total([(L * nw * (el + q_el), 4 * L * nw)])
    # prefill: the cache rows of every layer; the last layer needs its K and V only
    rows, H_kv = sum(lens), 2 * cfg["n_kv"] * cfg["head_dim"]
    n = (L - 1) * nw + H_kv * H
    return total([(n * el + rows * (H * el + L * kv),
                   2 * rows * n + 4 * (L - 1) * cfg["n_q"] * cfg["head_dim"] * sum(s * (s + 1) / 2 for s in lens))])


def tolerance(c):
    # bytes and whole numbers decided on given logits
    if c["op"] in ("refresh", "accept"):
        return "exact"
    # fp32 sums in another order
    if c["model"] == "tiny":
        return {"rel": 1e-5, "max": 4e-4, "differ": 0.005}
    # 16-bit activations rounded from sums in another order, through the layers: logits are 0.0047 and new cache rows
    # 0.0036 off the same in 64 bits
    return {"rel": 1.5e-2, "max": 0.12, "differ": 0.01}


# ------------------------------------------------------------------ inputs
def gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def make_weights(cfg, seed):
    g = gen(seed)
    H, V, L = cfg["hidden"], cfg["vocab"], cfg["n_layers"]
    dt = torch.bfloat16 if cfg["dtype"] == "bf16" else torch.float32

    def randn(shape, std):
        return torch.randn(shape, generator=g, device="cuda", dtype=dt).mul_(std)

    std = 1.28 / math.sqrt(H)                                   # 0.02 at hidden 4096
    emb = randn((V, H), 1.0)
    beta = 0.9 if H < 1024 else 0.6
    perm = torch.randperm(V, generator=g, device="cuda")
    head = randn((V, H), std * math.sqrt(1 - beta * beta))
    for i in range(0, V, 16384):
        head[i:i + 16384] += emb[perm[i:i + 16384]] * (std * beta)
    out = [emb, 1 + randn((H,), 0.1), head]
    for _ in range(L):
        for i, shp in enumerate(layer_shapes(cfg)):
            if len(shp) == 1:
                out.append(1 + randn(shp, 0.1))
            else:
                out.append(randn(shp, std / (math.sqrt(2 * L) if i in (2, 5) else 1.0)))
    return out


def layer_shapes(cfg):
    """Shapes of one layer's weights in binding order."""
    H, d, F = cfg["hidden"], cfg["head_dim"], cfg["ffn"]
    return [(H,), ((cfg["n_q"] + 2 * cfg["n_kv"]) * d, H), (H, cfg["n_q"] * d), (H,), (2 * F, H), (H, F)]


def int32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def make_inputs(c, seed):
    """Weights, tokens and lengths of a case, and the function that draws a sequence's cached context."""
    cfg, B = config(c), c["B"]
    s = types.SimpleNamespace(cfg=cfg, lens=lengths(c))
    s.W = make_weights(cfg, seed)
    g = gen(seed + 1_000_003)
    s.slots = torch.randperm(c["slots"], generator=g, device="cuda")[:B].to(torch.int32)
    s.last = torch.randint(0, cfg["vocab"], (B,), generator=g, device="cuda").to(torch.int32)
    s.drafts = torch.randint(0, cfg["vocab"], (B, c["gamma"]), generator=g, device="cuda").to(torch.int32)
    s.prompt = torch.randint(0, cfg["vocab"], (B, max(s.lens)), generator=g, device="cuda").to(torch.int32)
    dt = s.W[0].dtype
    shape = (cfg["n_layers"], cfg["n_kv"])

    def context(b):
        h = gen(seed * 1009 + 17 + b)
        return [torch.randn((*shape, s.lens[b], cfg["head_dim"]), generator=h, device="cuda", dtype=dt) for _ in "kv"]

    s.context = context
    return s


def make_accept(c, seed):
    """Target and drafter logits of a policy between certain and undecided, drafts drawn from the drafter."""
    g = gen(seed)
    B, G, V = c["B"], c["gamma"], config(c)["vocab"]
    p = torch.randn((B, G + 1, V), generator=g, device="cuda") * 2.5
    lead = 4 + 14 * torch.rand((B, G + 1, 1), generator=g, device="cuda")      # how far the likeliest token leads
    top = torch.randint(0, V, (B, G + 1, 1), generator=g, device="cuda")
    p.scatter_(2, top, lead + 5)
    q = p[:, :G] + 0.25 * torch.randn((B, G, V), generator=g, device="cuda")
    gum = -torch.log(-torch.log(torch.rand((B, G, V), generator=g, device="cuda").clamp_(1e-7, 1 - 1e-7)))
    draft = (q / T + gum).argmax(2).to(torch.int32)
    stats = torch.stack([(q / T).amax(2), torch.logsumexp(q.double() / T, 2).float()], 2)
    return types.SimpleNamespace(
        slots=torch.randperm(c["slots"], generator=g, device="cuda")[:B].to(torch.int32),
        kv_len=int32([c["ctx"]] * c["slots"]), draft=draft, q=q.contiguous(), stats=stats.contiguous(), p=p,
        out=torch.zeros((B, G + 1), dtype=torch.int32, device="cuda"),
        n_emit=torch.zeros((B,), dtype=torch.int32, device="cuda"),
        next=torch.zeros((B,), dtype=torch.int32, device="cuda"))


# ------------------------------------------------------------------ the cases' states and passes
def page_table(c):
    """Pages of every slot: handed out in a stride order, as a pool that has been in use gives them."""
    pps = pages_of(c)
    n = c["slots"] * pps
    step = next(s for s in range(int(n * 0.62) + 1, 4 * n + 2) if math.gcd(s, n) == 1)
    return torch.tensor([i * step % n for i in range(n)], dtype=torch.int32, device="cuda").view(c["slots"], pps)


def prepare(c, seed):
    if c["op"] == "accept":
        st = make_accept(c, seed)
        st.case, st.seed = c, seed
        return st
    st = make_inputs(c, seed)
    st.case, st.seed = c, seed
    cfg, B, G = st.cfg, c["B"], c["gamma"]
    st.eng = sdrl.Engine(cfg, c["slots"], capacity(c), G)
    st.eng.bind_weights(st.W)
    cached = c["op"] not in ("prefill", "refresh")
    if c["page"]:
        st.table = page_table(c)
        st.k, st.v, st.kv_len = st.eng.alloc_kv_paged(st.table.numel(), c["page"])
        st.eng.bind_kv_paged(st.k, st.v, st.table, st.kv_len)
    else:
        st.k, st.v, st.kv_len = st.eng.alloc_kv()
        st.eng.bind_kv(st.k, st.v, st.kv_len)
    slots = st.slots.tolist()
    if cached:
        for b in range(B):
            put_context(c, st, slots[b], st.context(b))
    start = [0] * c["slots"]
    for b in range(B):
        start[slots[b]] = st.lens[b] if cached else 0
    st.start = int32(start)
    st.kv_len.copy_(st.start)
    st.len = int32(st.lens)
    if c["op"] in ("sd_step", "sd_graph", "draft", "refresh"):
        st.qbuf = torch.zeros(st.eng.drafter_bytes(c["fmt"]), dtype=torch.uint8, device="cuda")
        st.eng.refresh_drafter(st.qbuf, c["fmt"])
    if c["op"] in ("sd_step", "sd_graph", "draft", "verify"):
        st.bufs = sdrl.SDBuffers(st.eng, B, G)
    if c["op"] == "ar":
        st.tok = torch.zeros((B,), dtype=torch.int32, device="cuda")
        st.logits = torch.zeros((B, cfg["vocab"]), dtype=torch.float32, device="cuda")
    if c["op"] == "sd_graph":
        st.tok = st.last.clone()
        sdrl.sd_step(st.eng, st.bufs, st.slots, st.tok, T, seed, STEP)
        st.graph = sdrl.StepGraph(st.eng, st.bufs, st.slots, st.tok, T, seed, STEP)
    return st


def put_context(c, st, slot, kv):
    S = kv[0].shape[2]
    for pool, x in zip((st.k, st.v), kv):
        if not c["page"]:
            pool[:, slot, :, :S] = x
            continue
        P = c["page"]
        for j in range(-(-S // P)):
            pool[int(st.table[slot, j]), :, :, :min(P, S - j * P)] = x[:, :, j * P:(j + 1) * P]


def small_cache(c, st):
    """The cache as an output, where it is small enough to compare whole."""
    return {"k": st.k, "v": st.v} if cache_size(c) <= SMALL else {}


def run(st):
    c = st.case
    op, G = c["op"], c["gamma"]
    if op == "accept":
        sdrl.accept_noalloc(st.slots, st.kv_len, st.draft, st.q, st.stats, st.p, G, T, st.seed, STEP, st.out, st.n_emit,
                            st.next)
        return {"out": st.out, "n_emit": st.n_emit, "next": st.next}
    e = st.eng
    if op == "refresh":
        e.refresh_drafter(st.qbuf, c["fmt"])
        return {"q": st.qbuf}
    if op == "draft":
        b = st.bufs
        e.draft(st.slots, st.last, G, T, st.seed, STEP, b.draft_tok, b.q_logits, b.q_stats)
        return {"tok": b.draft_tok, "logits": b.q_logits, "stats": b.q_stats, **small_cache(c, st)}
    if op == "verify":
        e.verify(st.slots, st.last, st.drafts, G, st.bufs.p_logits)
        return {"logits": st.bufs.p_logits, **small_cache(c, st)}
    st.kv_len.copy_(st.start)                       # the sequences as they were before the step
    if op == "prefill":
        e.prefill_ragged(st.slots, st.prompt, st.len)
        return {"kv_len": st.kv_len, **small_cache(c, st)}
    if op == "ar":
        e.ar_step(st.slots, st.last, T, st.seed, STEP, st.tok, st.logits)
        return {"tok": st.tok, "logits": st.logits, "kv_len": st.kv_len, **small_cache(c, st)}
    b = st.bufs
    if op == "sd_graph":
        st.tok.copy_(st.last)
        st.graph.replay()
    else:
        sdrl.sd_step(e, b, st.slots, st.last, T, st.seed, STEP)
    return {"tok": b.draft_tok, "q": b.q_logits, "stats": b.q_stats, "p": b.p_logits, "out": b.out_tok,
            "n_emit": b.n_emit, "next": b.next_tok, "kv_len": st.kv_len, **small_cache(c, st)}


# ------------------------------------------------------------------ the same in 64 bits
def rtn64(w, fmt):
    """The drafter's weights: RTN in groups of 128 along K, one fp16 scale each (fp32 arithmetic)."""
    N, K = w.shape
    x = w.float().view(N, K // 128, 128)
    lo, hi = x.amin(2, True), x.amax(2, True)
    amax = x.abs().amax(2, True)
    by = x.new_full((1,), {"w4": 7, "w4a": 15, "w8": 127}[fmt])       # a tensor: divided by, not multiplied by 1/7
    s = ((hi - lo if fmt == "w4a" else amax) / by).half().float()
    r = torch.round(x / torch.where(s == 0, torch.ones_like(s), s))
    if fmt == "w4a":
        z = torch.round(-lo / torch.where(s == 0, torch.ones_like(s), s)).clamp(0, 15)
        q = (r + z).clamp(0, 15) - z
    else:
        m = 8 if fmt == "w4" else 128
        q = r.clamp(-m, m - 1)
    return (q.double() * s.double()).view(N, K)


def norm64(x, gain, eps):
    return x / torch.sqrt((x * x).mean(1, True) + eps) * gain.double()


def rope64(x, pos, theta):
    """x [rows][heads][d], rotate-half at pos [rows]."""
    d = x.shape[2]
    ang = pos.double()[:, None] * theta ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., : d // 2], x[..., d // 2:]
    return torch.cat([a * cos - b * sin, a * sin + b * cos], 2)


def forward64(s, tokens, base, ctx, new, fmt=None, logits=True):
    """tokens[b]: the token ids of sequence b, at positions base[b], base[b] + 1, ...; ctx(b): its cached K and V;
    new[l][b]: K and V rows appended since (this call appends its own).  Returns the logits of all rows."""
    cfg, W = s.cfg, s.W
    d, nq, nkv, L = cfg["head_dim"], cfg["n_q"], cfg["n_kv"], cfg["n_layers"]
    n = [len(t) for t in tokens]
    at = np.concatenate([[0], np.cumsum(n)]).tolist()
    pos = torch.cat([torch.arange(base[b], base[b] + n[b], device="cuda") for b in range(len(n))])
    h = W[0][torch.cat(list(tokens)).long()].double()
    weight = (lambda w: rtn64(w, fmt)) if fmt else (lambda w: w.double())
    for l in range(L):
        g1, wqkv, wo, g2, wgu, wdown = W[3 + 6 * l: 9 + 6 * l]
        x = norm64(h, g1, cfg["rms_eps"]) @ weight(wqkv).T
        q = rope64(x[:, : nq * d].view(-1, nq, d), pos, cfg["rope_theta"])
        k = rope64(x[:, nq * d: (nq + nkv) * d].view(-1, nkv, d), pos, cfg["rope_theta"])
        v = x[:, (nq + nkv) * d:].view(-1, nkv, d)
        att = torch.empty_like(q)
        for b in range(len(n)):
            sl = slice(at[b], at[b + 1])
            old = new[l][b]
            kn, vn = k[sl].transpose(0, 1), v[sl].transpose(0, 1)
            new[l][b] = (kn, vn) if old is None else (torch.cat([old[0], kn], 1), torch.cat([old[1], vn], 1))
            if l == L - 1 and not logits:
                continue
            ck, cv = ctx(b) if ctx else (None, None)
            K = new[l][b][0] if ck is None else torch.cat([ck[l].double(), new[l][b][0]], 1)
            V = new[l][b][1] if cv is None else torch.cat([cv[l].double(), new[l][b][1]], 1)
            qb = q[sl].view(n[b], nkv, nq // nkv, d).permute(1, 2, 0, 3).reshape(nkv, -1, d)
            sc = (qb @ K.transpose(1, 2).contiguous()) / math.sqrt(d)
            last = torch.arange(K.shape[1] - n[b], K.shape[1], device="cuda").repeat(nq // nkv)
            sc.masked_fill_(torch.arange(K.shape[1], device="cuda")[None, None] > last[None, :, None], -math.inf)
            o = (sc.softmax(2) @ V).view(nkv, nq // nkv, n[b], d)
            att[sl] = o.permute(2, 0, 1, 3).reshape(n[b], nq, d)
        if l == L - 1 and not logits:
            return None
        h = h + att.reshape(-1, nq * d) @ weight(wo).T
        x = norm64(h, g2, cfg["rms_eps"]) @ weight(wgu).T
        F = cfg["ffn"]
        h = h + (torch.nn.functional.silu(x[:, :F]) * x[:, F:]) @ weight(wdown).T
    return norm64(h, W[1], cfg["rms_eps"]) @ W[2].double().T


def race64(logits, seed, pos, slot):
    """argmax of logits / T - ln(-ln u): u from Philox-4x64-10, key (seed, step), counter (block, pos, slot, 0)."""
    V = logits.numel()
    before = (pos << 64) + (slot << 128)                        # numpy steps the counter before each block
    bits = np.random.Philox(key=seed + (STEP << 64), counter=(before - 1) % (1 << 256)).random_raw(-(-V // 8) * 4)
    half = np.stack([bits & 0xFFFFFFFF, bits >> np.uint64(32)], 1).reshape(-1)[:V]
    u = torch.from_numpy(((half >> np.uint64(9)).astype(np.float64) + 0.5) / (1 << 23)).to(logits.device)
    return int((logits / T - torch.log(-torch.log(u))).argmax())


def caches64(c, s, new, kv):
    """The caches after the call, where they are outputs: the context, then the new rows."""
    cfg, cap = s.cfg, capacity(c)
    shape = (cfg["n_layers"], c["slots"], cfg["n_kv"], cap, cfg["head_dim"])
    if cache_size(c) > SMALL:
        return {}
    out = {}
    for i, name in enumerate("kv"):
        x = torch.zeros(shape, dtype=torch.float64, device="cuda")
        for b, slot in enumerate(s.slots.tolist()):
            S = 0
            if kv:
                S = s.lens[b]
                x[:, slot, :, :S] = s.context(b)[i].double()
            for l in range(shape[0]):
                rows = new[l][b][i]
                x[l, slot, :, S:S + rows.shape[1]] = rows
        if c["page"]:
            P, pps = c["page"], pages_of(c)
            pad = torch.zeros((shape[0], shape[1], shape[2], pps * P, shape[4]), dtype=torch.float64, device="cuda")
            pad[:, :, :, :cap] = x
            y = torch.empty((shape[1] * pps, shape[0], shape[2], P, shape[4]), dtype=torch.float64, device="cuda")
            y[page_table(c).long()] = pad.view(shape[0], shape[1], shape[2], pps, P, shape[4]).permute(1, 3, 0, 2, 4, 5)
            x = y
        out[name] = x
    return out


def exact(c, seed):
    op = c["op"]
    if op in ("refresh", "accept"):
        return None
    s = make_inputs(c, seed)
    B, G, L, V = c["B"], c["gamma"], s.cfg["n_layers"], s.cfg["vocab"]
    slots = s.slots.tolist()

    def rows():
        return [[None] * B for _ in range(L)]

    if op == "prefill":
        new = rows()
        forward64(s, [s.prompt[b, : s.lens[b]] for b in range(B)], [0] * B, None, new, logits=False)
        return {"kv_len": None, **caches64(c, s, new, False)}
    new = rows()
    if op == "ar":
        p = forward64(s, [s.last[b:b + 1] for b in range(B)], s.lens, s.context, new)
        return {"tok": None, "logits": p, "kv_len": None, **caches64(c, s, new, True)}
    drafts = s.drafts
    if op != "verify":
        tok, q, d = s.last.clone(), [], []
        for j in range(G):
            q.append(forward64(s, [tok[b:b + 1] for b in range(B)], [x + j for x in s.lens], s.context, new, c["fmt"]))
            tok = int32([race64(q[-1][b], seed, s.lens[b] + j + 1, slots[b]) for b in range(B)])
            d.append(tok)
        q, drafts = torch.stack(q, 1), torch.stack(d, 1)
        stats = torch.stack([(q / T).amax(2), torch.logsumexp(q / T, 2)], 2)
        if op == "draft":
            return {"tok": None, "logits": q, "stats": stats, **caches64(c, s, new, True)}
        new = rows()
    p = forward64(s, [torch.cat([s.last[b:b + 1], drafts[b]]) for b in range(B)], s.lens, s.context, new).view(B, G + 1, V)
    cache = caches64(c, s, new, True)
    if op == "verify":
        return {"logits": p, **cache}
    return {"tok": None, "q": q, "stats": stats, "p": p, "out": None, "n_emit": None, "next": None, "kv_len": None, **cache}
