"""Shared set-up for GPU parity tests: the same seeded inputs on both sides.

The oracle side gets CPU tensors from the seeded generators, the HIP side gets the same
generators run on the GPU (bit-identical by construction; test_gpu_parity checks that too)."""
import numpy as np
import torch

from paper_2505_22758_amd import synth

# tolerances of the decode step's logits against the fp64 oracle (bf16 weights, fp32 activations
# and accumulation on the GPU): the benchmark statement's bounds
MAX_ABS_TOL = 3e-2
REL_L2_TOL = 1e-2
ARGMAX_MIN_AGREE = 0.99
# Appended cache rows against the oracle's bf16 bits (see test_gpu_parity._check_appended_cache for
# the reading): per sequence, with e / r its largest absolute / relative-L2 logit error,
#   |element - oracle's| <= one bf16 step + KV_ABS_SLACK + KV_SLACK_PER_LOGIT_ERR * e
#   differing words / words <= KV_RATE_FLOOR + KV_RATE_PER_REL_ERR * r
# The GPU runs print the measured ratios; the constants are a few times those (design notes).
KV_ABS_SLACK = 1e-4
KV_SLACK_PER_LOGIT_ERR = 2.0
KV_RATE_FLOOR = 2e-3
KV_RATE_PER_REL_ERR = 1024.0

def prefill_lengths(T0, batch):
    """T0 as one length for every sequence or one length per sequence."""
    return [int(T0)] * batch if np.isscalar(T0) else [int(t) for t in T0]


def oracle_side(shape, seed, wdtype, batch, T0, max_ctx, quant_lm_head=True):
    from oracle import oracle
    layers = [synth.make_layer(shape, seed, l, wdtype, "cpu") for l in range(shape.n_layers)]
    head = synth.make_head(shape, seed, wdtype, "cpu", quant_lm_head)
    M = oracle.OracleModel(shape, layers, head)
    kv = M.new_kv(batch, max_ctx)
    T0s = prefill_lengths(T0, batch)
    for l in range(shape.n_layers):
        for b in range(batch):
            if T0s[b] > 0:
                k, v = synth.make_kv_prefill(shape, seed, l, b, T0s[b], "cpu")
                kv[l, b, 0, :T0s[b]], kv[l, b, 1, :T0s[b]] = oracle._np(k), oracle._np(v)
    return M, kv


def hip_side(shape, seed, wdtype, batch, T0, max_ctx, n_caches=1, quant_lm_head=True, device="cuda:0", max_batch=None):
    """batch: sequences of the caches; max_batch: sequences the model is created for (default: the same)."""
    from paper_2505_22758_amd import binding
    dec = binding.Decoder(shape, wdtype, max_batch=max_batch or batch, quant_lm_head=quant_lm_head, device=device)
    for l in range(shape.n_layers):
        lw = synth.make_layer(shape, seed, l, wdtype, device)
        dec.load_layer(l, lw)
        torch.cuda.synchronize()
        del lw
    hw = synth.make_head(shape, seed, wdtype, device, quant_lm_head)
    dec.load_head(hw)
    torch.cuda.synchronize()
    del hw
    caches = []
    T0s = prefill_lengths(T0, batch)
    for _ in range(n_caches):
        buf = torch.zeros(binding.ff_kv_bytes(dec.model, batch, max_ctx), dtype=torch.uint8, device=device)
        kv = binding.ff_kv_alloc(dec.model, batch, max_ctx, buf)
        for l in range(shape.n_layers):
            for b in range(batch):
                if T0s[b] > 0:
                    k, v = synth.make_kv_prefill(shape, seed, l, b, T0s[b], device)
                    binding.ff_kv_fill(kv, l, b, 0, k, v)
        torch.cuda.synchronize()
        caches.append((kv, buf))
    return dec, caches


def compare_logits(got: np.ndarray, ref: np.ndarray):
    """got fp32 [B,V], ref fp64 [B,V] -> (max_abs, rel_l2, argmax_equal per row)."""
    got = got.astype(np.float64)
    max_abs = float(np.max(np.abs(got - ref)))
    rel_l2 = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    same = (got.argmax(axis=1) == ref.argmax(axis=1))
    return max_abs, rel_l2, same


def both_sides_gpu_generated(shape, seed, wdtype, batch, T0, max_ctx, n_caches=1, quant_lm_head=True, device="cuda:0", max_batch=None):
    """Full-size set-up: every tensor is produced once by the seeded generators on the GPU (fast),
    handed to the HIP loader, and copied to the host for the oracle.  The generators are
    bit-identical on both devices, so this equals generating twice."""
    from oracle import oracle
    from paper_2505_22758_amd import binding

    def to_cpu(obj):
        return {k: to_cpu(v) for k, v in obj.items()} if isinstance(obj, dict) else obj.cpu()

    dec = binding.Decoder(shape, wdtype, max_batch=max_batch or batch, quant_lm_head=quant_lm_head, device=device)
    cpu_layers = []
    for l in range(shape.n_layers):
        lw = synth.make_layer(shape, seed, l, wdtype, device)
        dec.load_layer(l, lw)
        cpu_layers.append(to_cpu(lw))
        torch.cuda.synchronize()
        del lw
    hw = synth.make_head(shape, seed, wdtype, device, quant_lm_head)
    dec.load_head(hw)
    cpu_head = to_cpu(hw)
    torch.cuda.synchronize()
    del hw
    M = oracle.OracleModel(shape, cpu_layers, cpu_head)
    okv = M.new_kv(batch, max_ctx)
    caches = []
    for _ in range(n_caches):
        buf = torch.zeros(binding.ff_kv_bytes(dec.model, batch, max_ctx), dtype=torch.uint8, device=device)
        caches.append((binding.ff_kv_alloc(dec.model, batch, max_ctx, buf), buf))
    T0s = prefill_lengths(T0, batch)
    for l in range(shape.n_layers):
        for b in range(batch):
            if T0s[b] > 0:
                k, v = synth.make_kv_prefill(shape, seed, l, b, T0s[b], device)
                for kv, _ in caches:
                    binding.ff_kv_fill(kv, l, b, 0, k, v)
                okv[l, b, 0, :T0s[b]], okv[l, b, 1, :T0s[b]] = oracle._np(k.cpu()), oracle._np(v.cpu())
    torch.cuda.synchronize()
    return M, okv, dec, caches


def layer_major_both_sides(shape, seed, wdtype, runs, progress, device="cuda:0"):
    """Full-depth set-up for models whose canonical copy does not fit host memory (the 80-layer 70B
    shape).  Inputs are teacher-forced, so layer l at step s needs only layer l-1 at step s and layer
    l's own cache rows of earlier steps: the oracle runs LAYER-MAJOR (for l: for run: for sequence:
    for step), each layer being generated once on the GPU, handed to the HIP loader, copied to the
    host for the oracle's layer step and dropped.  Same function as step-major evaluation.

    runs: list of dicts with batch, T0, steps (independent teacher-forced runs on caches of their
    own; run i draws its tokens from seed + 1000 * (i + 1)).  Fills in per run: toks, kv (HIP cache
    handle), ref (fp64 logits [steps, batch, vocab]), okv_new (the oracle's appended rows, bf16 bits
    [L, batch, 2, steps, n_kv_heads, head_dim]).  Returns the Decoder."""
    from oracle import oracle
    from paper_2505_22758_amd import binding

    def to_cpu(obj):
        return {k: to_cpu(v) for k, v in obj.items()} if isinstance(obj, dict) else obj.cpu()

    dec = binding.Decoder(shape, wdtype, max_batch=max(r["batch"] for r in runs), device=device)
    hw = synth.make_head(shape, seed, wdtype, device)
    dec.load_head(hw)
    cpu_head = to_cpu(hw)
    torch.cuda.synchronize()
    del hw
    H = oracle.OracleModel(shape, [], cpu_head)
    for i, r in enumerate(runs):
        B, S = r["batch"], r["steps"]
        r["toks"] = synth.make_tokens(shape, seed + 1000 * (i + 1), S, B)
        r["x"] = np.stack([np.stack([H.embed(int(r["toks"][s, b])) for b in range(B)]) for s in range(S)])   # [S, B, d] fp64
        r["max_ctx"] = r["T0"] + S + 3
        r["kv_buf"] = torch.zeros(binding.ff_kv_bytes(dec.model, B, r["max_ctx"]), dtype=torch.uint8, device=device)
        r["kv"] = binding.ff_kv_alloc(dec.model, B, r["max_ctx"], r["kv_buf"])
        r["okv_new"] = np.zeros((shape.n_layers, B, 2, S, shape.n_kv_heads, shape.head_dim), dtype=np.uint16)
    for l in range(shape.n_layers):
        lw = synth.make_layer(shape, seed, l, wdtype, device)
        dec.load_layer(l, lw)
        cpu_lw = to_cpu(lw)
        torch.cuda.synchronize()
        del lw
        Ml = oracle.OracleModel(shape, [cpu_lw], cpu_head)
        for r in runs:
            T0, S = r["T0"], r["steps"]
            for b in range(r["batch"]):
                Kc = np.zeros((r["max_ctx"], shape.n_kv_heads, shape.head_dim), dtype=np.uint16)
                Vc = np.zeros_like(Kc)
                if T0 > 0:
                    k, v = synth.make_kv_prefill(shape, seed, l, b, T0, device)
                    binding.ff_kv_fill(r["kv"], l, b, 0, k, v)
                    Kc[:T0], Vc[:T0] = oracle._np(k.cpu()), oracle._np(v.cpu())
                for s in range(S):
                    Ml.layer_step(0, r["x"][s, b], Kc, Vc, T0 + s)   # updates the row of x in place
                r["okv_new"][l, b, 0], r["okv_new"][l, b, 1] = Kc[T0:T0 + S], Vc[T0:T0 + S]
        del Ml, cpu_lw
        if (l + 1) % 4 == 0 or l + 1 == shape.n_layers:
            progress(f"  layer-major oracle: layer {l + 1}/{shape.n_layers} done")
    for r in runs:
        r["ref"] = np.stack([np.stack([H.logits(r["x"][s, b]) for b in range(r["batch"])]) for s in range(r["steps"])])
        progress(f"  layer-major oracle: logits of the batch-{r['batch']} run done")
    torch.cuda.synchronize()
    return dec
