"""The allocation-free entry point (ff_decode_step_static: exchange scratch in a static device
array inside the library) against ff_decode_step, through the C ABI, on two calls in a row, the
second with a smaller input."""
import numpy as np
import pytest
import torch

from paper_2505_22758_amd import synth
from tests import helpers

pytestmark = pytest.mark.gpu


def test_static_scratch_step_equals_the_workspace_step_twice_in_a_row():
    from paper_2505_22758_amd import binding
    S, seed = synth.TINY, 0x5ca7
    # first call: batch 4 on a 40-row context; second call: a smaller input (batch 2, other model
    # instance of another weight type, shorter context) on the same static array
    calls = [(synth.WDTYPE_BF16, 4, 40), (synth.WDTYPE_INT8, 2, 9)]
    shapes = {synth.WDTYPE_BF16: S, synth.WDTYPE_INT8: S.replace(d_ffn=1408)}
    models = {}
    for wd, B, T0 in calls:
        models[wd] = helpers.hip_side(shapes[wd], seed, wd, B, T0, max_ctx=T0 + 4, n_caches=2)
    for rep in range(2):   # the pair of calls twice: the second pair starts from the first pair's leftovers
        for wd, B, T0 in calls:
            dec, caches = models[wd]
            shape = shapes[wd]
            tok = synth.make_tokens(shape, seed + rep, 1, B)[0].to("cuda:0")
            pos = torch.full((B,), T0 + rep, dtype=torch.int32, device="cuda:0")
            want = torch.zeros(B, shape.vocab, device="cuda:0")
            got = torch.full_like(want, -3.0)
            binding.ff_decode_step(dec.model, tok, pos, caches[0][0], want, B)
            binding.ff_decode_step_static(dec.model, tok, pos, caches[1][0], got, B)
            binding.ff_status(dec.model)
            # same kernels, same arithmetic, same order: identical bits
            assert torch.equal(got, want), (rep, wd, B, float((got - want).abs().max()))
            assert torch.equal(caches[0][1], caches[1][1]), "appended cache rows differ"
    # a configuration whose exchange scratch exceeds the static array is rejected, not truncated
    big = synth.LLAMA_8B.replace(n_layers=1, vocab=1024)
    dec = binding.Decoder(big, synth.WDTYPE_BF16, max_batch=4)
    dec.load_layer(0, synth.make_layer(big, 1, 0, synth.WDTYPE_BF16, "cuda:0"))
    dec.load_head(synth.make_head(big, 1, synth.WDTYPE_BF16, "cuda:0"))
    dec.alloc_kv(4, 8)
    tok = torch.zeros(4, dtype=torch.int32, device="cuda:0")
    lg = torch.zeros(4, big.vocab, device="cuda:0")
    with pytest.raises(binding.FFError) as e:
        binding.ff_decode_step_static(dec.model, tok, tok, dec.kv, lg, 4)
    assert e.value.code == binding.FF_ERR_NOMEM
    dec.close()
    for dec, _ in models.values():
        dec.close()


# (layers, batch): images of one set per layer alone exceed the array, one set fits
@pytest.mark.parametrize("wdtype,layers,batch", ((synth.WDTYPE_BF16, 60, 16), (synth.WDTYPE_INT8, 400, 2), (synth.WDTYPE_INT4, 400, 1)),
                         ids=("bf16-x16", "int8-x2", "int4-x1"))
def test_static_scratch_with_one_set_of_images_for_all_layers(wdtype, layers, batch):
    """Where the exchange images of every layer do not fit the static array, the wide pass reuses one set: readers drop
    their cached copies with an acquire fence, and the epochs order a set's next writes behind its last reads.  Several steps
    in a row, each bit for bit the step with images of its own per layer.  Models for 16, 2 and 2 sequences: every operand form."""
    from paper_2505_22758_amd import binding
    S, T0, steps, max_batch = synth.TINY.replace(name="deep", n_layers=layers, d_ffn=1408, vocab=1000), 21, 3, max(batch, 2)
    image_set = 4 * max_batch * (2 * S.d_model + S.n_q_heads * S.head_dim + S.d_ffn)   # bytes: 2 x bf16 per element
    static = 8 << 20   # FF_STATIC_SCRATCH_BYTES
    assert layers * image_set > static > 8 * image_set
    dec = binding.Decoder.synthetic(S, 0x5ca8, wdtype, max_batch)
    bufs = [torch.zeros(binding.ff_kv_bytes(dec.model, batch, T0 + steps), dtype=torch.uint8, device="cuda:0") for _ in range(2)]
    kvs = [binding.ff_kv_alloc(dec.model, batch, T0 + steps, b) for b in bufs]
    for kv in kvs:
        binding.ff_kv_fill_synthetic(kv, 0x5ca8, T0)
    toks = synth.make_tokens(S, 0x5ca8, steps, batch).to("cuda:0")
    want, got = torch.zeros(batch, S.vocab, device="cuda:0"), torch.full((batch, S.vocab), -3.0, device="cuda:0")
    for s in range(steps):
        pos = torch.full((batch,), T0 + s, dtype=torch.int32, device="cuda:0")
        binding.ff_decode_step(dec.model, toks[s], pos, kvs[0], want, batch)
        binding.ff_decode_step_static(dec.model, toks[s], pos, kvs[1], got, batch)
        binding.ff_status(dec.model)
        assert bool(torch.isfinite(want).all()) and torch.equal(got, want), (s, float((got - want).abs().max()))
    assert torch.equal(bufs[0], bufs[1]), "appended cache rows differ"
    for kv in kvs:
        binding.ff_kv_free(kv)
    dec.close()
