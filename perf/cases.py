"""What the decode step is timed on: calls of ff_decode_step as a serving program makes them.

A pass is a few consecutive teacher-forced decode steps of one model on one cache (one launch per
step, nothing between them), so that a later step reads the cache rows an earlier one appended, and at
its end the appended rows of the last layer are read back, as a program does that hands them on.  Its
output is every step's logits and these rows.  The model's weights, its cache with the prompts' rows,
the token ids and the positions are what such a program holds before it calls.

Sizes are this repository's: the tiny shape and the 8B and 70B shapes of its benchmark (all of their
layers, or a block of them under a vocabulary that keeps the head's share of the step), batches of 1
to 16 sequences, contexts of a few to some thousand rows, bf16 / int8 / int4 weights.
"""
import math

import torch

from paper_2505_22758_amd import binding, synth

DEV = "cuda:0"
BF16, INT8, INT4 = 0, 1, 2
GROUP = 128
EPS = 1e-5


def _case(shape, layers, vocab, weights, contexts, steps, skip=-1, **name):
    """contexts: rows already cached per sequence, as a text "1024" or "1024,77"; skip: index of a
    sequence that has stopped early and sits the steps out (-1: none)."""
    d, hq, hkv, hd, f, theta = SHAPES[shape]
    return dict(name, shape=shape, layers=layers, d=d, hq=hq, hkv=hkv, hd=hd, ffn=f, vocab=vocab, theta=theta,
                weights=weights, contexts=contexts, steps=steps, skip=skip)


SHAPES = {   # d_model, query heads, KV heads, head dimension, d_ffn, RoPE theta
    "tiny": (512, 8, 2, 64, 1376, 10000.0),
    "tiny-1408": (512, 8, 2, 64, 1408, 10000.0),   # whole int4 groups
    "1b": (2048, 16, 4, 128, 8192, 500000.0),
    "3b": (3072, 24, 6, 128, 8192, 500000.0),
    "8b": (4096, 32, 8, 128, 14336, 500000.0),
    "70b": (8192, 64, 8, 128, 28672, 500000.0),
}


def _same(ctx, batch):
    return ",".join([str(ctx)] * batch)


def listed():
    return [
        # the smallest call: a 4-layer model of a few megabytes, launch and hand-over latency only
        _case("tiny", 4, 4096, BF16, "128", 4, name="tiny-bf16-b1"),
        # one user at a time, the whole model: the benchmark's headline and its two quantised forms
        _case("8b", 32, 128256, BF16, "1024", 2, name="8b-bf16-b1"),
        _case("8b", 32, 128256, INT4, "2048", 2, name="8b-int4-b1"),
        _case("8b", 8, 32064, INT8, "4096", 2, name="8b-int8-b1-block"),
        # the large model's layers for one user
        _case("70b", 16, 25600, BF16, "2048", 2, name="70b-bf16-b1-block"),
        # a few users: prompts of their own lengths
        _case("8b", 8, 32064, BF16, "1024,371", 2, name="8b-bf16-b2-block"),
        _case("8b", 8, 32064, INT4, _same(2048, 4), 2, name="8b-int4-b4-block"),
        _case("8b", 8, 32064, INT8, "3000,129,1024,40", 2, name="8b-int8-b4-ragged-block"),
        # a serving batch: half full, ragged with one sequence that has stopped, and full
        _case("8b", 8, 32064, BF16, _same(1024, 8), 2, name="8b-bf16-b8-block"),
        _case("8b", 8, 32064, INT8, "4096,97,1500,2048,333,64,700,1,2900,1024,512", 2, skip=5, name="8b-int8-b11-ragged-block"),
        _case("8b", 8, 32064, INT4, _same(2048, 16), 2, name="8b-int4-b16-block"),
        _case("70b", 8, 12800, BF16, _same(2048, 16), 2, name="70b-bf16-b16-block"),
    ]


def draw(rng):
    """Another model block, weight format, batch and set of context lengths of the same ranges."""
    shape = rng.choice(["tiny", "1b", "3b", "8b", "8b", "8b", "70b"])
    weights = rng.choice([BF16, INT8, INT4])
    if shape == "tiny" and weights == INT4:
        shape = "tiny-1408"
    batch = rng.choice([1, 1, 1, 2, 3, 4, rng.randint(5, 8), rng.randint(9, 16)])
    top = {"tiny": 1000, "tiny-1408": 1000}.get(shape, 6000 if batch <= 4 else 4200)

    def length():
        return int(round(math.exp(rng.uniform(math.log(1), math.log(top)))))

    contexts = [length()] * batch if rng.random() < 0.4 else [length() for _ in range(batch)]
    skip = rng.randrange(batch) if batch > 1 and rng.random() < 0.2 else -1
    layers = {"tiny": 4, "tiny-1408": 4, "1b": rng.randint(4, 16), "3b": rng.randint(4, 12), "8b": rng.randint(1, 10),
              "70b": rng.randint(1, 6)}[shape]
    vocab = rng.choice([4096, rng.randint(3000, 16000), 32064])
    return _case(shape, layers, vocab, weights, ",".join(map(str, contexts)), 2, skip=skip)


# ---- inputs, all made from the seed on the GPU ----
def _gen(seed, tag):
    return torch.Generator(device=DEV).manual_seed((seed * 1000003 + tag * 7919 + 12345) % (1 << 62))


def _contexts(case):
    return [int(v) for v in case["contexts"].split(",")]


def _max_ctx(case):
    return max(_contexts(case)) + case["steps"] + 2


def _matrix(g, n, k, weights):
    """A projection matrix, N(0, 0.02): bf16, int8 with one fp16 scale a row (largest value on 127), or
    int4 with an fp16 scale and zero for each group of 128 columns (smallest to largest value on 0..15)."""
    w = torch.empty(n, k, dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
    if weights == BF16:
        return {"w": w}
    if weights == INT8:
        s = (w.abs().amax(dim=1).float() / 127.0).half()
        q = torch.round(w / s.float()[:, None]).clamp_(-127, 127).to(torch.int8)
        return {"w": q, "s": s}
    t = w.view(n, k // GROUP, GROUP)
    lo, hi = t.aminmax(dim=2)
    s = ((hi.float() - lo.float()) / 15.0).half()
    z = torch.round(-lo.float() / s.float()).clamp_(0, 15).half()
    q = torch.round(t / s.float()[..., None]).add_(z.float()[..., None]).clamp_(0, 15).to(torch.uint8).view(n, k)
    return {"w": q[:, 0::2] | (q[:, 1::2] << 4), "s": s, "z": z}


def _gain(g, d):
    return torch.empty(d, dtype=torch.float32, device=DEV).normal_(1.0, 0.02, generator=g).bfloat16()


def _mat_dims(case):
    d, f, q, kv = case["d"], case["ffn"], case["hq"] * case["hd"], case["hkv"] * case["hd"]
    return {"wq": (q, d), "wk": (kv, d), "wv": (kv, d), "wo": (d, q), "w_gate": (f, d), "w_up": (f, d), "w_down": (d, f)}


def _layer(case, seed, l):
    g = _gen(seed, 10 + l)
    out = {"attn_norm": _gain(g, case["d"]), "ffn_norm": _gain(g, case["d"])}
    for name, (n, k) in _mat_dims(case).items():
        out[name] = _matrix(g, n, k, case["weights"])
    return out


def _head(case, seed):
    g = _gen(seed, 1)
    embed = torch.empty(case["vocab"], case["d"], dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
    return {"embed": embed, "final_norm": _gain(g, case["d"]), "lm_head": _matrix(g, case["vocab"], case["d"], case["weights"])}


def _prompt(case, seed, l):
    """Cache rows of one layer: per sequence, K (already rotated) and V, bf16 [rows][kv heads][head dim]."""
    g = _gen(seed, 100000 + l)
    ctx = _contexts(case)
    both = torch.empty(2, sum(ctx), case["hkv"], case["hd"], dtype=torch.bfloat16, device=DEV).normal_(0.0, 1.0, generator=g)
    at, out = 0, []
    for n in ctx:
        out.append((both[0, at:at + n], both[1, at:at + n]))
        at += n
    return out


def _tokens(case, seed):
    batch = len(_contexts(case))
    t = torch.randint(0, case["vocab"], (case["steps"], batch), generator=_gen(seed, 2), device=DEV, dtype=torch.int32)
    if case["skip"] >= 0:
        t[:, case["skip"]] = -1
    return t


def _positions(case):
    c = torch.tensor(_contexts(case), dtype=torch.int32, device=DEV)
    return c[None, :] + torch.arange(case["steps"], dtype=torch.int32, device=DEV)[:, None]


def prepare(case, seed):
    ctx = _contexts(case)
    shape = synth.ModelShape("case", case["layers"], case["d"], case["hq"], case["hkv"], case["hd"], case["ffn"], case["vocab"],
                             EPS, case["theta"])
    dec = binding.Decoder(shape, case["weights"], max_batch=len(ctx), device=DEV)
    for l in range(case["layers"]):
        dec.load_layer(l, _layer(case, seed, l))
    dec.load_head(_head(case, seed))
    dec.alloc_kv(len(ctx), _max_ctx(case))
    for l in range(case["layers"]):
        for b, (k, v) in enumerate(_prompt(case, seed, l)):
            binding.ff_kv_fill(dec.kv, l, b, 0, k, v)
    logits = torch.zeros(case["steps"], len(ctx), case["vocab"], dtype=torch.float32, device=DEV)
    rows = torch.zeros(2, len(ctx), case["steps"], case["hkv"], case["hd"], dtype=torch.bfloat16, device=DEV)
    active = [(b, c) for b, c in enumerate(ctx) if b != case["skip"]]
    return {"dec": dec, "tokens": _tokens(case, seed), "positions": _positions(case), "logits": logits, "rows": rows, "active": active}


def run(state):
    dec, logits, (k, v) = state["dec"], state["logits"], state["rows"]
    for s in range(logits.shape[0]):
        dec.step(state["tokens"][s], state["positions"][s], logits[s])
    for b, c in state["active"]:
        binding.ff_kv_read(dec.kv, dec.shape.n_layers - 1, b, c, k[b], v[b])
    return {"logits": logits, "k": k, "v": v}


def _matrix_bytes(n, k, weights):
    return {BF16: 2 * n * k, INT8: n * k + 2 * n, INT4: n * k // 2 + 4 * n * (k // GROUP)}[weights]


def work(case):
    """Every parameter once a step, every valid cache row once, appended rows and logits written."""
    ctx = [c for b, c in enumerate(_contexts(case)) if b != case["skip"]]
    mats = list(_mat_dims(case).values())
    head = (case["vocab"], case["d"])
    weights = case["layers"] * (sum(_matrix_bytes(n, k, case["weights"]) for n, k in mats) + 4 * case["d"])
    weights += _matrix_bytes(*head, case["weights"]) + 2 * case["d"]
    row = 4 * case["layers"] * case["hkv"] * case["hd"]
    total = flops = 0
    for s in range(case["steps"]):
        total += weights + sum(row * (c + s + 1) for c in ctx) + len(ctx) * (2 * case["d"] + 4 * case["vocab"])
        total += 2 * len(ctx) * 4 * case["hkv"] * case["hd"]   # the last layer's appended rows, read back
        flops += 2 * len(ctx) * (case["layers"] * sum(n * k for n, k in mats) + head[0] * head[1])
        flops += sum(4 * case["layers"] * case["hq"] * case["hd"] * (c + s + 1) for c in ctx)
    return {"bytes": total, "flops": flops}


def tolerance(case):
    # Activations travel between layers as 22-bit numbers and enter the matrix cores as pairs of 8-bit
    # mantissas (17 bits), but what is seen against 64 bits is set by the appended K and V elements that
    # round to the other neighbouring bf16 value, and by what the later layers make of them.  Seen over
    # the listed cases and 50 drawn ones: logits 6e-7 to 8e-4, K and V 0 to 1.6e-3; the largest single
    # difference is one bf16 step of a K or V element, 7.8e-3.  Four times these:
    return {"rel": 6e-3, "max": 3e-2}


# ---- the same in 64 bits ----
def _dense(m, weights):
    if weights == BF16:
        return m["w"].double()
    if weights == INT8:
        return m["w"].double() * m["s"].double()[:, None]
    codes = torch.stack((m["w"] & 15, m["w"] >> 4), dim=2).flatten(1)
    n, k = codes.shape
    t = codes.view(n, k // GROUP, GROUP).double()
    return ((t - m["z"].double()[..., None]) * m["s"].double()[..., None]).view(n, k)


def _norm(x, gain):
    return x * torch.rsqrt((x * x).mean(dim=-1, keepdim=True) + EPS) * gain.double()


def _rotate(x, pos, theta):
    """x [B, heads, hd]: pairs (i, i + hd/2) turned by pos * theta^(-2i/hd)."""
    hd = x.shape[-1]
    inv = theta ** (-torch.arange(0, hd, 2, dtype=torch.float64, device=DEV) / hd)
    ang = pos.double()[:, None] * inv
    c, s = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat((a * c - b * s, b * c + a * s), dim=-1)


def exact(case, seed):
    ctx, weights, batch = _contexts(case), case["weights"], len(_contexts(case))
    hq, hkv, hd, per = case["hq"], case["hkv"], case["hd"], case["hq"] // case["hkv"]
    tokens, positions = _tokens(case, seed), _positions(case)
    head = _head(case, seed)
    xs = [head["embed"][tokens[s].clamp(min=0).long()].double() for s in range(case["steps"])]
    gain, lm = head["final_norm"], head["lm_head"]
    del head
    rows = torch.zeros(2, batch, case["steps"], hkv, hd, dtype=torch.float64, device=DEV)
    for l in range(case["layers"]):
        w = _layer(case, seed, l)
        mats = {name: _dense(w[name], weights) for name in _mat_dims(case)}
        cache = _prompt(case, seed, l)
        new = [([], []) for _ in ctx]
        for s, x in enumerate(xs):
            h = _norm(x, w["attn_norm"])
            q = _rotate((h @ mats["wq"].T).view(batch, hq, hd), positions[s], case["theta"])
            k = _rotate((h @ mats["wk"].T).view(batch, hkv, hd), positions[s], case["theta"]).bfloat16()
            v = (h @ mats["wv"].T).view(batch, hkv, hd).bfloat16()
            rows[0, :, s], rows[1, :, s] = k.double(), v.double()
            heads = []
            for b in range(batch):
                new[b][0].append(k[b:b + 1])
                new[b][1].append(v[b:b + 1])
                K = torch.cat([cache[b][0]] + new[b][0]).double().transpose(0, 1)          # [kv heads, rows, hd]
                V = torch.cat([cache[b][1]] + new[b][1]).double().transpose(0, 1)
                score = (K @ q[b].view(hkv, per, hd).transpose(1, 2).contiguous()) / math.sqrt(hd)   # [kv heads, rows, per]
                p = torch.softmax(score, dim=1).transpose(1, 2).contiguous()
                heads.append((p @ V.contiguous()).reshape(1, hq * hd))
            x = x + torch.cat(heads) @ mats["wo"].T
            h = _norm(x, w["ffn_norm"])
            xs[s] = x + (torch.nn.functional.silu(h @ mats["w_gate"].T) * (h @ mats["w_up"].T)) @ mats["w_down"].T
        del mats, w
    lm = _dense(lm, weights)
    out = torch.stack([_norm(x, gain) @ lm.T for x in xs])
    if case["skip"] >= 0:
        out[:, case["skip"]], rows[:, case["skip"]] = 0.0, 0.0   # its row of the logits is not written, nothing is appended
    return {"logits": out, "k": rows[0], "v": rows[1]}
