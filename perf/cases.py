"""The calls whose speed is measured: what a serving or rollout loop asks of the library, through the Python binding.

A case is one kind of pass over one cache:

  decode    rlkv_decode_attention of one layer over caches that already hold their context
  step      a whole decode step: rlkv_append_decode of every layer (the cache grows by one token a pass)
  generate  a request from its start: the cache is emptied, the prompt goes in, then `steps` tokens are decoded
            (bf16: prompt through rlkv_prefill_attention; fp32, which has no prefill: through rlkv_append)
  prefill   prompts from their start to their end, in chunks of `chunk` tokens, through rlkv_prefill_attention
  import    prompts whose K/V come from elsewhere (another engine's prefill): rlkv_append_ragged in chunks, then
            one decode step

Shapes are those of the library's own workloads (32 query / 8 KV heads and 28 / 4, head_dim 128, windows of
16 + 112, 64 + 256 and 64 + 512, contexts of 1 k to 64 k tokens, a share `pct` of the KV heads compressed) and of its
tests.  Context lengths are spread evenly over [lo, hi] and do not depend on the seed; values do: K, V and Q are
N(0, 1), keys at positions 0 to 3 four times that (attention sinks).
"""
import math

import torch

import paper_2510_08525_amd as rl

D = 128
SCALE = 1.0 / math.sqrt(D)
ROOM = 4096               # tokens a "step" case can grow by before its cache is filled anew
FILL_CHUNK = 2048         # tokens per append while a context is laid down in prepare()


def _case(name, kind, q_heads, kv_heads, pct, batch, lo, hi, sink, recent, dtype="bf16", layers=1, chunk=0, steps=0,
          page=0, gated=False):
    return dict(name=name, kind=kind, dtype=dtype, q_heads=q_heads, kv_heads=kv_heads, pct=pct, batch=batch, lo=lo, hi=hi,
                sink=sink, recent=recent, layers=layers, chunk=chunk, steps=steps, page=page, gated=gated)


def listed():
    return [
        # One user, one layer in single precision (how the cache is checked against a reference model): a 1024-token
        # prompt and 16 tokens.  The smallest calls: launches and host time.
        _case("generate_f32_b1_1k", "generate", 32, 8, 50, 1, 1024, 1024, 16, 112, dtype="f32", chunk=1024, steps=16),
        # One chat turn: an odd prompt of a few hundred tokens and 32 tokens of answer.
        _case("generate_b1_333", "generate", 32, 8, 60, 1, 333, 333, 64, 256, chunk=512, steps=32),
        # A small server's decode attention: batch 8 at 8 k, few heads compressed.
        _case("decode_b8_8k", "decode", 32, 8, 20, 8, 8192, 8192, 64, 256),
        # The headline: a whole decode step of a 28-layer model, batch 16 at 16 k, 60 % of the heads compressed.
        _case("step_28l_b16_16k", "step", 28, 4, 60, 16, 16384, 16384, 64, 256, layers=28),
        # A busy server with requests of all lengths.
        _case("decode_b32_4k_32k", "decode", 32, 8, 60, 32, 4096, 32768, 64, 512),
        # Long reasoning traces: the largest decode launch.
        _case("decode_b64_16k_64k", "decode", 32, 8, 60, 64, 16384, 65536, 64, 256),
        # The same kind of server with a paged pool whose pages have been shuffled by long service.
        _case("decode_paged_b24_2k_20k", "decode", 28, 4, 60, 24, 2000, 20000, 64, 256, page=64),
        # Rollouts while the gates are still continuous: every head blends full and local attention.
        _case("decode_gated_b16_4k", "decode", 28, 4, 0, 16, 3000, 5000, 64, 256, gated=True),
        # A batch of long prompts, chunked as a scheduler does it.
        _case("prefill_b16_16k", "prefill", 28, 4, 60, 16, 16384, 16384, 64, 256, chunk=2048),
        # One long prompt alone on the card.
        _case("prefill_b1_32k", "prefill", 32, 8, 60, 1, 32500, 32500, 64, 256, chunk=4096),
        # The prompts of a rollout batch, ragged, with continuous gates.
        _case("prefill_gated_b8_1k_4k", "prefill", 28, 4, 0, 8, 1000, 4000, 64, 256, chunk=1024, gated=True),
        # Requests whose prompts were computed elsewhere are admitted: their K/V go into the stores.
        _case("import_b32_1k_6k", "import", 32, 8, 60, 32, 1000, 6000, 64, 512, chunk=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "step", "prefill", "prefill", "generate", "generate", "import"])
    q_heads, kv_heads = rng.choice([(32, 8), (28, 4), (32, 8), (28, 4), (8, 8), (12, 4), (16, 1)])
    pct = rng.choice([0, 20, 40, 60, 60, 80])
    sink, recent = rng.choice([(16, 112), (64, 256), (64, 512), (33, 70), (4, 1000)])
    c = dict(kind=kind, dtype="bf16", q_heads=q_heads, kv_heads=kv_heads, pct=pct, sink=sink, recent=recent, layers=1, chunk=0,
             steps=0, page=0, gated=False)
    if kind == "decode":
        c["batch"] = _log_int(rng, 1, 64)
        hi = _log_int(rng, 100, min(65536, 2 ** 24 // (c["batch"] * kv_heads)))
        c["lo"], c["hi"] = rng.randint(max(1, hi // 8), hi), hi
        c["page"] = rng.choice([0, 0, 0, 32, 64, 256])
        c["gated"] = rng.random() < 0.2
        if not c["page"] and rng.random() < 0.15 and c["batch"] * hi <= 2 ** 17:
            c["dtype"] = "f32"
    elif kind == "step":
        c["layers"] = rng.randint(16, 32)
        c["batch"] = _log_int(rng, 4, 16)
        c["hi"] = _log_int(rng, 4000, 16384)
        c["lo"] = rng.randint(c["hi"] // 2, c["hi"])
    elif kind == "generate":
        c["dtype"] = rng.choice(["bf16", "bf16", "f32"])
        c["batch"] = _log_int(rng, 1, 8)
        c["hi"] = _log_int(rng, 30, 3000)
        c["lo"] = rng.randint(max(1, c["hi"] // 4), c["hi"])
        c["chunk"] = rng.choice([512, 1024, 2048])
        c["steps"] = rng.randint(8, 40)
    elif kind == "prefill":
        c["batch"] = _log_int(rng, 1, 16)
        c["hi"] = _log_int(rng, 200, min(32768, int(2 ** 14 * math.sqrt(16 * 28 / (c["batch"] * q_heads)))))
        c["lo"] = rng.randint(max(1, c["hi"] // 4), c["hi"])
        c["chunk"] = rng.choice([512, 1000, 2048, 4096])
        c["gated"] = rng.random() < 0.25
    else:
        c["batch"] = _log_int(rng, 1, 64)
        c["hi"] = _log_int(rng, 100, min(32768, 2 ** 21 // (c["batch"] * kv_heads)))
        c["lo"] = rng.randint(max(1, c["hi"] // 8), c["hi"])
        c["chunk"] = rng.choice([512, 1024, 2048])
    return c


# ---- sizes of a case -------------------------------------------------------------------------------------------

def _lengths(c):
    """Context (prompt) length of every sequence: spread over [lo, hi] in a scattered order."""
    n, lo, hi = c["batch"], c["lo"], c["hi"]
    return [lo + int((hi - lo) * ((b * 0.6180339887498949 + 0.5) % 1.0) + 0.5) for b in range(n)]


def _mask(c):
    """[layers][kv_heads], 1 = full: a share pct of the heads compressed, fractions carried from layer to layer."""
    H, out = c["kv_heads"], []
    for l in range(c["layers"]):
        n = (l + 1) * c["pct"] * H // 100 - l * c["pct"] * H // 100
        out.append([0 if (h * 3 + l) % H in range(n) and math.gcd(3, H) == 1 else 1 for h in range(H)])
    return out


def _gates(c, seed):
    g = torch.Generator().manual_seed(seed * 1000 + 77)
    return torch.rand(c["layers"], c["kv_heads"], generator=g)


def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _chunks(c, chunk):
    """Per chunk the tokens each sequence brings."""
    ns = _lengths(c)
    return [[max(0, min(n - p, chunk)) for n in ns] for p in range(0, max(ns), chunk)]


def _rows(c, seed, what, layer, index, heads, n, sink_rows=0):
    """[batch][heads][n][D] values of one chunk (index < 0: a decode step's)."""
    g = torch.Generator(device="cuda").manual_seed((((seed * 4 + what) * 64 + layer) * 4096) + index + 2048)
    x = torch.randn(c["batch"], heads, n, D, generator=g, device="cuda", dtype=_dtype(c))
    if sink_rows:
        x[:, :, :min(4, n)] *= 4.0
    return x


def _kv(c, seed, layer, index, n):
    first = index == 0
    return _rows(c, seed, 0, layer, index, c["kv_heads"], n, first), _rows(c, seed, 1, layer, index, c["kv_heads"], n)


def _fill_size(c):
    return c["chunk"] or FILL_CHUNK


# ---- the state a program holds -----------------------------------------------------------------------------------

class State:
    pass


def _fill(s):
    """Lays every sequence's context down (decode and step cases)."""
    c, size = s.case, _fill_size(s.case)
    s.cache.reset()
    for layer in range(c["layers"]):
        for i, counts in enumerate(_chunks(c, size)):
            k, v = _kv(c, s.seed, layer, i, max(counts))
            if min(counts) == max(counts):
                s.cache.append(layer, k, v)
            else:
                s.cache.append_ragged(layer, k, v, counts)
    s.grown = 0


def prepare(case, seed):
    c = case
    s = State()
    s.case, s.seed = c, seed
    ns = _lengths(c)
    grow = {"decode": 0, "step": ROOM, "generate": c["steps"], "prefill": 0, "import": 1}[c["kind"]]
    max_len = [n + grow for n in ns]
    bf16 = c["dtype"] == "bf16"
    prefill = c["chunk"] if bf16 and c["kind"] in ("generate", "prefill") else 0
    pool = sum(-(-n // c["page"]) for n in max_len) if c["page"] else 0
    s.cache = rl.Cache(c["layers"], c["q_heads"], c["kv_heads"], D, c["batch"], c["sink"], c["recent"],
                       rl.RLKV_BF16 if bf16 else rl.RLKV_F32, _mask(c), max_len, page_tokens=c["page"], pool_pages=pool,
                       prefill_tokens=prefill)
    if c["page"]:
        s.cache.pool_shuffle(1234 + seed)
    if c["gated"]:
        s.cache.set_gates(_gates(c, seed).numpy())
    B, Hq, L = c["batch"], c["q_heads"], c["layers"]
    if c["kind"] in ("decode", "step"):
        _fill(s)
        s.q = [_rows(c, seed, 2, l, -1, Hq, 1)[:, :, 0].contiguous() for l in range(L)]
        s.out = [torch.zeros(B, Hq, D, device="cuda", dtype=_dtype(c)) for _ in range(L)]
        if c["kind"] == "step":
            s.new = [_kv(c, seed, l, -1, 1) for l in range(L)]
    else:
        s.chunks = _chunks(c, c["chunk"])
        sizes = [max(counts) for counts in s.chunks]
        s.kv = [_kv(c, seed, 0, i, n) for i, n in enumerate(sizes)]
        if prefill:
            s.pq = [_rows(c, seed, 2, 0, i, Hq, n) for i, n in enumerate(sizes)]
            s.pout = [torch.zeros_like(q) for q in s.pq]
        n_steps = {"generate": c["steps"], "prefill": 0, "import": 1}[c["kind"]]
        s.new = [_kv(c, seed, 0, -1 - t, 1) for t in range(n_steps)]
        s.q = [_rows(c, seed, 2, 0, -1 - t, Hq, 1)[:, :, 0].contiguous() for t in range(n_steps)]
        s.out = [torch.zeros(B, Hq, D, device="cuda", dtype=_dtype(c)) for _ in range(n_steps)]
    torch.cuda.synchronize()
    return s


def run(s):
    c, cache = s.case, s.cache
    if c["kind"] == "decode":
        cache.decode_attention(0, s.q[0], s.out[0], SCALE)
        return s.out[0]
    if c["kind"] == "step":
        if s.grown == ROOM:
            _fill(s)
        for l in range(c["layers"]):
            cache.append_decode(l, s.new[l][0], s.new[l][1], s.q[l], s.out[l], SCALE)
        s.grown += 1
        return s.out
    cache.reset()
    prefill = c["kind"] == "prefill" or (c["kind"] == "generate" and c["dtype"] == "bf16")
    for i, counts in enumerate(s.chunks):
        k, v = s.kv[i]
        if prefill:
            cache.prefill_attention(0, s.pq[i], k, v, counts, s.pout[i], SCALE)
        elif min(counts) == max(counts):
            cache.append(0, k, v)
        else:
            cache.append_ragged(0, k, v, counts)
    for t in range(len(s.q)):
        cache.append_decode(0, s.new[t][0], s.new[t][1], s.q[t], s.out[t], SCALE)
    return (s.pout if prefill else []) + ([torch.stack(s.out)] if s.out else [])


# ---- what a pass cannot do without -----------------------------------------------------------------------------

def _pairs_prefill(n0, t, window):
    """Admitted (query, key) pairs of t queries at positions n0 .. under the causal mask / a window (0 = causal)."""
    full = t * n0 + t * (t + 1) // 2
    if not window:
        return full
    return sum(min(p + 1, window) for p in range(n0, n0 + t)) if n0 < window else t * window


def work(case):
    c = case
    e = 4 if c["dtype"] == "f32" else 2
    row = 2 * D * e                                          # one K and one V row
    W, G = c["sink"] + c["recent"], c["q_heads"] // c["kv_heads"]
    ns, nbytes, flops = _lengths(c), 0, 0
    q_bytes = c["batch"] * c["q_heads"] * D * e
    masks = _mask(c)

    def attend(lengths, mask):                               # one decode attention launch
        keys = sum(sum(n if f else min(n, W) for f in mask) for n in lengths)
        extra = sum(sum(min(n, W) for f in mask if f) for n in lengths) if c["gated"] else 0
        return keys * row + 2 * q_bytes, 4 * D * G * (keys + extra)

    if c["kind"] == "decode":
        nbytes, flops = attend(ns, masks[0])
    elif c["kind"] == "step":
        for m in masks:
            b, f = attend([n + 1 for n in ns], m)
            nbytes, flops = nbytes + b + 2 * c["batch"] * c["kv_heads"] * row, flops + f
    else:
        mask = masks[0]
        prefill = c["kind"] == "prefill" or (c["kind"] == "generate" and c["dtype"] == "bf16")
        at = [0] * c["batch"]
        for counts in _chunks(c, c["chunk"]):
            for b, t in enumerate(counts):
                if prefill and t:
                    nbytes += 2 * t * c["q_heads"] * D * e
                    for f in mask:
                        nbytes += row * (t + (at[b] if f else min(at[b], W)))
                        flops += 4 * D * G * _pairs_prefill(at[b], t, 0 if f else W)
                        if f and c["gated"]:
                            flops += 4 * D * G * _pairs_prefill(at[b], t, W)
                at[b] += t
        for n in ns:                                         # rows that stay: read once, written once
            nbytes += sum((1 if prefill else 2) * row * (n if f else min(n, W)) for f in mask)
        for t in range({"generate": c["steps"], "prefill": 0, "import": 1}[c["kind"]]):
            b, f = attend([n + t + 1 for n in ns], mask)
            nbytes, flops = nbytes + b + 2 * c["batch"] * c["kv_heads"] * row, flops + f
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # fp32: the order of fp32 sums.  bf16: the output's own rounding (2^-9 of each value) plus fp32 sums and weights of
    # at least 11 significant bits.
    return {"rel": 2e-6, "max": 4e-5} if case["dtype"] == "f32" else {"rel": 7e-3, "max": 3e-2}


# ---- the same in 64 bits -----------------------------------------------------------------------------------------

def _attend64(c, gates, q, qpos, history):
    """q [B][Hq][T][D], qpos: per sequence the T query positions (list of tensors), history: list of (first position per
    sequence, tokens per sequence, k, v).  Causal attention of full heads, local of compressed ones, blended by gates."""
    B, Hq, T = q.shape[:3]
    H = c["kv_heads"]
    G, S, R = Hq // H, c["sink"], c["recent"]
    out = torch.zeros(B, Hq, T, D, device="cuda", dtype=torch.float64)
    for b in range(B):
        nq = len(qpos[b])
        if nq == 0:
            continue
        i = qpos[b].cuda()[None, :, None]
        for h in range(H):
            qq = q[b, h * G:(h + 1) * G, :nq].double().reshape(G * nq, D) * SCALE
            res = torch.zeros(G, nq, D, device="cuda", dtype=torch.float64)
            for local, weight in ((False, gates[h]), (True, 1.0 - gates[h])):
                if weight == 0.0:
                    continue
                m = torch.full((G, nq, 1), -math.inf, device="cuda", dtype=torch.float64)
                l, o = torch.zeros_like(m), torch.zeros_like(res)
                for first, counts, k, v in history:
                    if counts[b] == 0:
                        continue
                    if local and first[b] >= S and first[b] + counts[b] <= int(qpos[b].min()) - R + 1:
                        continue
                    j = torch.arange(first[b], first[b] + counts[b], device="cuda")[None, None, :]
                    sc = (qq @ k[b, h, :counts[b]].double().t().contiguous()).reshape(G, nq, counts[b])
                    on = j <= i
                    if local:
                        on = on & ((j < S) | (i - j < R))
                    sc = sc.masked_fill(~on, -math.inf)
                    m2 = torch.maximum(m, sc.amax(-1, keepdim=True))
                    ref = torch.where(m2 == -math.inf, torch.zeros_like(m2), m2)
                    p = torch.exp(sc - ref)
                    a = torch.exp(m - ref)
                    l = l * a + p.sum(-1, keepdim=True)
                    o = o * a + (p.reshape(G * nq, -1) @ v[b, h, :counts[b]].double()).reshape(G, nq, D)
                    m = m2
                res += weight * (o / l)
            out[b, h * G:(h + 1) * G, :nq] = res
    return out


def exact(case, seed):
    c, ns = case, _lengths(case)
    outs = []
    for layer in range(c["layers"]):
        gates = [float(f) for f in _mask(c)[layer]]
        if c["gated"]:
            gates = [float(g) * f for g, f in zip(_gates(c, seed)[layer], gates)]
        size, at, history = _fill_size(c), [0] * c["batch"], []
        prefill = c["kind"] == "prefill" or (c["kind"] == "generate" and c["dtype"] == "bf16")
        for i, counts in enumerate(_chunks(c, size)):
            n = max(counts)
            k, v = _kv(c, seed, layer, i, n)
            history.append((list(at), counts, k, v))
            if prefill:
                q = _rows(c, seed, 2, layer, i, c["q_heads"], n)
                pos = [torch.arange(at[b], at[b] + counts[b]) for b in range(c["batch"])]
                outs.append(_attend64(c, gates, q, pos, history))
            at = [a + t for a, t in zip(at, counts)]
        steps = {"decode": 0, "step": 1, "generate": c["steps"], "prefill": 0, "import": 1}[c["kind"]]
        if c["kind"] == "decode":
            q = _rows(c, seed, 2, layer, -1, c["q_heads"], 1)
            outs.append(_attend64(c, gates, q, [torch.tensor([n - 1]) for n in ns], history)[:, :, 0])
        done = []
        new = [_kv(c, seed, layer, -1 - t, 1) for t in range(steps)]
        prompt = list(history)
        for t in range(steps):
            k, v = (torch.cat([kv[w] for kv in new[:t + 1]], 2) for w in (0, 1))
            history = prompt + [(ns, [t + 1] * c["batch"], k, v)]
            q = _rows(c, seed, 2, layer, -1 - t, c["q_heads"], 1)
            done.append(_attend64(c, gates, q, [torch.tensor([n + t]) for n in ns], history)[:, :, 0])
        if c["kind"] == "step":
            outs += done
        elif done:
            outs.append(torch.stack(done))
    return outs[0] if c["kind"] == "decode" else outs
