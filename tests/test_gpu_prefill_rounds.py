"""Ragged prefill over several rounds with packed rows: six prompts of which
some end inside the first, second and third round (the rounds' length follows
from the 2560 rows of a prefill forward), one exactly at a round's end and one
empty, against the oracle's prefill of each alone, dense and paged."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_18967_amd import sdrl, synth

from gpu_common import DeviceKV, host_bits, i32, oracle_models, say
from test_gpu_e2e import SMALL_GQA

pytestmark = pytest.mark.gpu

LENS = [1100, 1, 426, 0, 700, 853]          # rounds of 2560 // 6 = 426 positions


@pytest.mark.parametrize("cfg,tol,page", [(synth.TINY, 5e-3, 0), (SMALL_GQA, 2e-2, 0), (SMALL_GQA, 2e-2, 32)],
                         ids=["f32", "bf16", "bf16-paged"])
def test_packed_rounds_match_oracle(cfg, tol, page):
    say("packed prefill rounds", cfg["name"], page)
    B, ld, seed = len(LENS), max(LENS), 33
    slots = [4, 2, 0, 5, 1, 3]
    cap = ld + 4
    W = synth.make_weights(cfg, seed, "cpu")
    eng = sdrl.Engine(cfg, B, cap, 3)
    eng.bind_weights([w.cuda() for w in W])
    kv = DeviceKV(eng, cap, page, seed)
    tokens = synth.make_tokens(B, ld, cfg["vocab"], seed + 1)
    for b, n in enumerate(LENS):
        tokens[b, n:] = -1                    # never read
    eng.prefill_ragged(i32(slots), tokens.cuda(), i32(LENS))
    eng.sync()
    kd, vd = kv.dense()
    kv_len = kv.kv_len.cpu().numpy()
    target, _ = oracle_models(cfg, host_bits(W))
    for b, (s, n) in enumerate(zip(slots, LENS)):
        assert kv_len[s] == n
        okv = oracle.KV(cfg, cap)
        if n:
            oracle.forward_seq(target, okv, tokens[b, :n].numpy(), 0, want_logits=False)
        for dev, ref in ((kd, okv.k), (vd, okv.v)):
            x, r = dev[:, s, :, :n].float().cpu().numpy(), ref[:, :, :n]
            assert n == 0 or np.abs(x - r).max() <= tol * np.abs(r).max(), b
            assert not dev[:, s, :, n:].any(), b         # nothing past a prompt's end
    eng.close()
