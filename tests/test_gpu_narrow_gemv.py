"""GPU parity of the narrow products (K = 128, and K = 256 of bfloat16 weights) of small
models' decode passes: 1 row, 2, and more than one group of 4, with the fused epilogues.
Float32 within 1e-5 as everywhere; bfloat16 models keep float16 keys and values (2^-11
relative, a few 1e-4 of a logit over their layers): 1e-3."""
import pytest
import torch  # noqa: F401  (before the library is loaded: both use torch's HIP runtime)

import oracle
import paper_2608_15454_amd as mbp
import synth
from gpu_harness import forced_run, new_decoder

pytestmark = pytest.mark.gpu

F32 = synth.WORKLOADS["tiny_f32"].model
D128 = F32.replace(dtype="bf16", n_mb=2)
D256 = synth.SMALL_F32.replace(dtype="bf16", n_lm=1)


@pytest.mark.parametrize("model,tol", [(F32, 1e-5), (D128, 1e-3), (D256, 1e-3), (D256.replace(head="mlp"), 1e-3)])
@pytest.mark.parametrize("batch", [1, 2, 7])
def test_narrow_products(model, tol, batch):
    assert mbp.lib().mbp_check_gemv(model.dtype == "bf16", batch, 3 * model.d_model, model.d_model)
    raw = synth.make_weights(model, seed=batch, gain_jitter=0.3)
    dec = new_decoder(model, raw, batch, 80)
    prompts = [synth.make_prompt(b, 24 + 5 * b) for b in range(batch)]
    forced_run(dec, oracle.to_float64(raw), model, prompts, 3, 3, 0.75, tol=tol, label=f"{model.dtype} {model.d_model} x{batch}")
