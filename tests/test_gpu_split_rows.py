"""GPU parity of the long-pass path on split rows (bfloat16 models, passes of 65 rows or
more) at the sizes where its tiles, K splits and row maps can go wrong.  Logits against
the oracle within 1e-3 at logit gain 1 and |logit| of a few units: keys and values are
kept in float16 (2^-11 relative), which over the six layers of these models moves a
logit by a few 1e-4; activations enter the products with 16 significant bits."""
import pytest

import oracle
import synth
from gpu_harness import forced_run, new_decoder
from test_gpu_forward import check

pytestmark = pytest.mark.gpu

# d = 256: column tiles of 128 and (gate / up) 256; d = 128 with heads of 32: the prefill
# attention's general kernel writes the split rows
D256 = synth.SMALL_F32.replace(dtype="bf16")
D128 = synth.ModelConfig(d_model=128, n_heads=4, n_enc=1, n_lm=1, n_nb=1, n_mb=1, head="lca", dtype="bf16")
TOL = 1e-3


@pytest.mark.parametrize("model,T", [(D256, 64), (D256, 65), (D256, 127), (D256, 128), (D256, 129), (D256, 257),
                                     (D256, 700), (D128, 65), (D128, 200)])
def test_forward_row_edges(model, T):
    raw = synth.make_weights(model, seed=T, gain_jitter=0.3)
    dec = new_decoder(model, raw, 1, T + 8)
    check(dec, oracle.to_float64(raw), model, synth.make_prompt(T, T), TOL)


@pytest.mark.parametrize("kw", [dict(engine=False), dict(kv_dtype=0), dict(kv_dtype=1), dict(max_chunk=100)])
def test_forward_cache_types(kw):
    """Float32 and bfloat16 caches take the general prefill attention; bfloat16 keeps 8
    bits of a key, 8 times the error of float16.  Passes of 100 rows: key blocks that lie
    below, across and above a tile's first query at odd offsets."""
    raw = synth.make_weights(D256, seed=2, gain_jitter=0.3)
    T = 333 if "max_chunk" in kw else 150
    dec = new_decoder(D256, raw, 1, T + 50, **kw)
    check(dec, oracle.to_float64(raw), D256, synth.make_prompt(2, T), TOL * (8 if kw.get("kv_dtype") == 1 else 1))


@pytest.mark.parametrize("batch,head", [(65, "lca"), (70, "lca"), (66, "mlp")])
def test_decode_many_rows(batch, head):
    """Commits of 65 rows and more: the decode attention (one split, and several merged)
    writes split rows; the MLP heads of a large batch run on them."""
    model = D256.replace(head=head, n_mb=2)
    raw = synth.make_weights(model, seed=batch, gain_jitter=0.3)
    W = oracle.to_float64(raw)
    dec = new_decoder(model, raw, batch, 330)
    prompts = [synth.make_prompt(b, 300 if b == 3 else 6 + b % 9) for b in range(batch)]
    forced_run(dec, W, model, prompts, 2, 3, 0.75, tol=TOL, label=f"{head} {batch}")
