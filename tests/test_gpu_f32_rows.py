"""The fp32 decoder's few-row GEMMs (k_gemm_f32_rows, k_gemm_q4_f32) and the
tiled one past 192 rows, against the oracle: one SD step whose drafts have 1 to
39 rows and whose verify has 5 to 195, on a decoder with 3 and 5 groups along K
(waves without a group, lanes without a last piece), in every drafter format."""
import pytest

from paper_2606_18967_amd import synth

from gpu_common import run_rollout, say

pytestmark = pytest.mark.gpu

CFG = dict(name="f32-rows", n_layers=1, hidden=384, n_q=6, n_kv=2, head_dim=64, ffn=640, vocab=320, dtype="f32",
           rope_theta=10000.0, rms_eps=1e-5)


@pytest.mark.parametrize("fmt", ["w4", "w4a", "w8"])
@pytest.mark.parametrize("B", [1, 4, 5, 9, 14, 38, 39])
def test_few_row_gemms_match_oracle(B, fmt):
    say("f32 rows", B, fmt)
    W = synth.make_weights(CFG, 3, "cpu", std=0.05)
    prompt = synth.make_tokens(B, 6, CFG["vocab"], 5)
    # fp32 sums of at most 640 products against fp64: 640 * 2^-24 of the row scale, through one layer
    eng, kv, okv, o_len, st = run_rollout(CFG, W, prompt, B, 12, 4, 1.0, 7, 1, 1e-4, n_steps=1, fmt=fmt)
    assert st["checked"] == B and st["exempt"] == 0
    eng.close()
