"""GPU parity of the attention where a KV head's query rows take several
work-groups (more than 64 rows: a prefill's rounds, a verify with a long draft).

Each slice of 64 rows walks its item's positions up to the last one that it
attends.  Prompts that end one row before, at and after a slice's edge, an empty
one and ones longer than a round, on top of random context that the work items
cut, so that items start before, inside and past the positions that a slice
attends.  The second layer's cache rows come from the first layer's attention,
so the cache is compared with the oracle's, and a verify's logits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_18967_amd import sdrl, synth

from gpu_common import DeviceKV, host_bits, i32, oracle_kv_from_device, oracle_models, say
from test_gpu_attention_plan import verify_against_oracle

pytestmark = pytest.mark.gpu

# two query heads per KV head, a hidden size that keeps the oracle quick
GQA_F32 = dict(synth.TINY, name="gqa-f32", n_kv=2)
GQA_D64 = dict(GQA_F32, name="gqa-d64", dtype="bf16")
GQA4 = dict(name="gqa4", n_layers=2, hidden=256, n_q=8, n_kv=2, head_dim=128, ffn=512, vocab=512, dtype="bf16",
            rope_theta=500000.0, rms_eps=1e-5)
LONG = dict(GQA4, name="gqa5-long", n_layers=2, hidden=512, n_q=40, n_kv=8)


def prefill_against_oracle(cfg, lens, ctx0, page, tol, seed=57):
    B, ld = len(lens), max(lens)
    cap = ctx0 + ld + 4
    W = synth.make_weights(cfg, seed, "cpu")
    eng = sdrl.Engine(cfg, B, cap, 3)
    eng.bind_weights([w.cuda() for w in W])
    kv = DeviceKV(eng, cap, page, seed)
    kv.fill_context(ctx0, seed + 100)
    torch.cuda.synchronize()
    kd0, vd0 = (x.clone() for x in kv.dense())
    tokens = synth.make_tokens(B, ld, cfg["vocab"], seed + 1)
    for b, n in enumerate(lens):
        tokens[b, n:] = -1                               # never read
    eng.prefill_ragged(i32(range(B)), tokens.cuda(), i32(lens))
    eng.sync()
    kd, vd = kv.dense()
    kv_len = kv.kv_len.cpu().numpy()
    target, _ = oracle_models(cfg, host_bits(W))
    for b, n in enumerate(lens):
        assert kv_len[b] == ctx0 + n
        okv = oracle_kv_from_device(cfg, kd0, vd0, b, ctx0, cap)
        if n:
            oracle.forward_seq(target, okv, tokens[b, :n].numpy(), ctx0, want_logits=False)
        end = ctx0 + n
        for dev, ref, was in ((kd, okv.k, kd0), (vd, okv.v, vd0)):
            x, r = dev[:, b, :, ctx0:end].float().cpu().numpy(), ref[:, :, ctx0:end]
            assert n == 0 or np.abs(x - r).max() <= tol * np.abs(r).max(), b
            assert torch.equal(dev[:, b, :, :ctx0], was[:, b, :, :ctx0]), b
            assert torch.equal(dev[:, b, :, end:], was[:, b, :, end:]), b
    eng.close()


@pytest.mark.parametrize("lens,ctx0", [([63, 64, 65, 0, 1], 300), ([700, 129, 1, 0, 513], 530), ([900], 0)],
                         ids=["edges", "rounds", "single"])
@pytest.mark.parametrize("cfg,page,tol", [(synth.TINY, 0, 5e-3), (GQA_F32, 0, 5e-3), (GQA_F32, 32, 5e-3),
                                          (GQA_D64, 0, 2e-2), (GQA_D64, 64, 2e-2), (GQA4, 0, 2e-2), (GQA4, 32, 2e-2)],
                         ids=["f32", "f32-gqa", "f32-gqa-paged", "d64", "d64-paged", "d128", "d128-paged"])
def test_sliced_prefill_matches_oracle(cfg, page, tol, lens, ctx0):
    say("sliced prefill", cfg["name"], page, lens, ctx0)
    prefill_against_oracle(cfg, lens, ctx0, page, tol)


@pytest.mark.parametrize("cfg,gamma,tol", [(GQA_F32, 31, 5e-3), (GQA_F32, 32, 5e-3), (GQA4, 15, 2e-2), (GQA4, 16, 2e-2),
                                           (GQA4, 31, 2e-2), (GQA4, 32, 2e-2)],
                         ids=["f32-64", "f32-66", "d128-64", "d128-68", "d128-128", "d128-132"])
def test_long_draft_verify_matches_oracle(cfg, gamma, tol):
    say("long draft verify", cfg["name"], gamma)
    verify_against_oracle([0, 300, 611], 700, gamma, 0, tol=tol, cfg=cfg)


def piece_ratio(cfg, n, pieces):
    """Time of one prefill of a prompt of n tokens over the time of the same prompt in pieces."""
    eng = sdrl.Engine(cfg, 1, n + 4, 3)
    eng.bind_weights([w.cuda() for w in synth.make_weights(cfg, 3, "cpu")])
    kv = DeviceKV(eng, n + 4)
    tokens = synth.make_tokens(1, n, cfg["vocab"], 5).cuda()
    parts = [t.contiguous() for t in tokens.chunk(pieces, 1)]

    def best(calls):
        t = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in "ab")
            kv.kv_len.zero_()
            a.record()
            for c in calls:
                eng.prefill(i32([0]), c)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    r = best([tokens]) / best(parts)
    eng.sync()
    eng.close()
    return r


@pytest.mark.parametrize("cfg,n,pieces", [(synth.TINY, 1000, 4), (LONG, 2500, 8)], ids=["f32", "bf16"])
def test_a_prompt_in_one_round_takes_no_longer_than_in_pieces(cfg, n, pieces):
    r = piece_ratio(cfg, n, pieces)
    say("one round against", pieces, "pieces:", round(r, 3))
    assert r < 1.1
