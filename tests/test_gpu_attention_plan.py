"""GPU parity of the attention's work items (make_att_plan): contexts cut into
chunks by the sequences' own lengths, longest items first.

A mirror of the rule picks the cases: a batch below the item target, in a
cache much larger than its contexts, whose chunk starts fall 1 to 4 positions
into the rows that a verify appends (so two work-groups write them), a batch
above the target (every sequence one item, longest first) with an empty sequence
and an unusable slot among the others, and batches of one to four waves of
sequences on two KV heads, cut or whole and in order.  Logits against the
oracle's forward over the same tokens, dense and paged."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_18967_amd import sdrl, synth

from gpu_common import DeviceKV, host_bits, i32, oracle_kv_from_device, oracle_models, say

pytestmark = pytest.mark.gpu

CFG = dict(name="plan-bf16", n_layers=2, hidden=512, n_q=8, n_kv=8, head_dim=64, ffn=512, vocab=512, dtype="bf16",
           rope_theta=500000.0, rms_eps=1e-5)
TARGET_WGS, FULL, SHORTEST, UNIT = 512, 512, 128, 32


def chunks(ctx, n_kv):
    """Chunk length of every sequence (contexts in positions, new rows included), query rows in one slice."""
    up = lambda x: -(-x // UNIT) * UNIT  # noqa: E731
    target, top = TARGET_WGS // n_kv, max(up(max(ctx)), SHORTEST)
    ch = top
    if len(ctx) < target:
        even, fewer = -(-sum(ctx) // target), -(-sum(ctx) // max(target // 4, 1))
        base = min(up(max(even, min(fewer, FULL), SHORTEST)), top)
        more = (top - base) // UNIT
        cand = [base + -(-more * k * k // 3969) * UNIT for k in range(64)]
        ch = next(c for c in cand if sum(-(-x // c) for x in ctx) <= target)
    return [up(-(-x // -(-x // ch))) for x in ctx]


def verify_against_oracle(lens, max_ctx, gamma, page, slots=None, check=None, seed=41, tol=2e-2, cfg=CFG):
    B = len(lens)
    W = synth.make_weights(cfg, seed, "cpu")
    eng = sdrl.Engine(cfg, B, max_ctx, gamma)
    eng.bind_weights([w.cuda() for w in W])
    kv = DeviceKV(eng, max_ctx, page, seed)
    kv.fill_context(max(lens), seed + 100)
    kv.kv_len.copy_(i32(lens))
    torch.cuda.synchronize()
    kd0, vd0 = kv.dense()
    V = cfg["vocab"]
    toks = synth.make_tokens(B, gamma + 1, V, seed + 1)
    p = torch.zeros((B, gamma + 1, V), dtype=torch.float32, device="cuda")
    eng.verify(i32(slots or range(B)), toks[:, 0].cuda().contiguous(), toks[:, 1:].cuda().contiguous(), gamma, p)
    if slots:
        with pytest.raises(sdrl.SDError, match="slot"):
            eng.sync()
    else:
        eng.sync()
    kd, vd = kv.dense()
    target, _ = oracle_models(cfg, host_bits(W))
    pd = p.cpu().numpy()
    assert np.isfinite(pd).all()
    for b in check if check is not None else range(B):
        kl = lens[b]
        okv = oracle_kv_from_device(cfg, kd0, vd0, b, kl, max_ctx)
        ol = oracle.forward_seq(target, okv, toks[b].numpy(), kl)
        for j in range(gamma + 1):
            assert np.abs(pd[b, j] - ol[j]).max() <= tol * np.abs(ol[j]).max(), (b, j)
        end = kl + gamma + 1
        for dev, ref in ((kd, okv.k), (vd, okv.v)):
            r = ref[:, :, kl:end]
            assert np.abs(dev[:, b, :, kl:end].float().cpu().numpy() - r).max() <= tol * np.abs(r).max(), b
    eng.close()


@pytest.mark.parametrize("page", [0, 32], ids=["dense", "paged"])
def test_chunk_starts_inside_the_new_rows(page):
    gamma, n = 4, 5
    lens, offsets = [300, 1200, 801, 0], {}
    for i in (1, 2):                                     # a chunk start 3 and 1 positions into the new rows
        want = (3, 1)[i - 1]
        for kl in range(lens[i], lens[i] + 400):
            trial = lens[:i] + [kl] + lens[i + 1:]
            clen = chunks([x + n for x in trial], CFG["n_kv"])[i]
            if (kl + want) % clen == 0 and kl + n > clen:
                lens = trial
                break
        offsets[i] = want
    lens_ctx = [x + n for x in lens]
    cl = chunks(lens_ctx, CFG["n_kv"])
    assert all((lens[i] + offsets[i]) % cl[i] == 0 for i in offsets), (lens, cl)
    say("chunk starts inside the new rows", page, lens, cl)
    verify_against_oracle(lens, 6000, gamma, page)


@pytest.mark.parametrize("page", [0, 32], ids=["dense", "paged"])
def test_more_sequences_than_items_with_an_empty_and_an_unusable_one(page):
    B = 70
    lens = [(37 * b) % 211 for b in range(B)]
    lens[5], lens[69] = 0, 500
    slots = list(range(B))
    slots[11] = -1
    say("more sequences than items", page, max(lens))
    verify_against_oracle(lens, 640, 2, page, slots, check=[0, 5, 10, 12, 40, 68, 69])


@pytest.mark.parametrize("max_ctx", [512, 513], ids=["whole", "cut"])
def test_caches_on_either_side_of_the_short_rule(max_ctx):
    lens = [509, 0, 31, 257, 127, 128, 380]              # the longest fills the short cache
    say("short cache", max_ctx)
    verify_against_oracle(lens, max_ctx, 2, 0)


@pytest.mark.parametrize("B", [63, 64, 65, 200, 255, 256])
def test_batches_of_several_waves_of_sequences(B):
    cfg = dict(CFG, name="plan-two-heads", n_q=2, n_kv=2)       # 256 items: 255 sequences are cut, 256 are not
    lens = [(53 * b) % 97 + (900 if b % 50 == 7 else 0) for b in range(B)]
    say("waves of sequences", B)
    verify_against_oracle(lens, 1100, 2, 0, check=[0, 7, 57, 61, B - 2, B - 1], cfg=cfg)
