"""The bf16 GEMMs with K splits against torch in fp32, through AR steps of a
one-layer decoder on empty caches (attention over a sequence's own token alone is
its value row, so the whole step is a few matrix products): the DMA-fed tiles of
both widths at every height, whose down projection a mirror of the plan splits,
and the weight-streaming kernel (an LM head of an odd multiple of 64)."""
import pytest
import torch

from paper_2606_18967_amd import sdrl, synth

from gpu_common import say

pytestmark = pytest.mark.gpu


def dma_plan(M, N, K):
    """(tile height / 32, width / 64, splits) by the rule of the GEMM's launcher."""
    KB, best, least = K // 64, None, 0.0
    for wcn in (4, 2):
        if N % (64 * wcn):
            continue
        mt = 2 if M <= 64 else 10 if M > 256 else 8 if M > 192 else 6 if M > 160 else -(-M // 32)
        mt += mt % 2 if wcn == 2 else 0
        tiles = N // (64 * wcn) * -(-M // (32 * mt))
        stage = (.42 + .125 * mt) * (1. if wcn == 2 else 1.45 if mt == 10 else 1.65)
        for S in range(1, min(32, KB // 2) + 1):
            if KB % S:
                continue
            wgs = tiles * S
            t = (1. if wgs <= 256 else wgs / 256 + .35) * (KB // S + (2 if mt == 10 else 3)) * stage
            t += 8 + 8e-6 / 5 * S * M * N if S > 1 else 0.
            if best is None or t < least:
                best, least = (mt, wcn, S), t
    return best


def ar_against_torch(cfg, B, seed=61):
    W = synth.make_weights(cfg, seed, "cuda")
    eng = sdrl.Engine(cfg, B, 4, 1)
    eng.bind_weights(W)
    k, v, kv_len = eng.alloc_kv()
    eng.bind_kv(k, v, kv_len)
    kv_len.zero_()
    last = synth.make_tokens(B, 1, cfg["vocab"], seed + 1)[:, 0].contiguous().cuda()
    tok = torch.zeros((B,), dtype=torch.int32, device="cuda")
    logits = torch.full((B, cfg["vocab"]), float("nan"), dtype=torch.float32, device="cuda")
    eng.ar_step(torch.arange(B, dtype=torch.int32, device="cuda"), last, 1.0, 1, 1, tok, logits)
    eng.sync()
    emb, fin, head, n1, wqkv, wo, n2, wgu, wdown = W
    d, nq, nkv, F = cfg["head_dim"], cfg["n_q"], cfg["n_kv"], cfg["ffn"]

    def r16(x):
        return x.to(torch.bfloat16).float()

    def mm(x, w):
        return x @ w.float().t()

    def norm(x, g):
        return r16(x * torch.rsqrt(x.pow(2).mean(1, keepdim=True) + cfg["rms_eps"]) * g.float())

    h = emb[last.long()].float()
    val = r16(mm(norm(h, n1), wqkv)[:, (nq + nkv) * d:]).view(B, nkv, 1, d)
    h = h + mm(val.expand(B, nkv, nq // nkv, d).reshape(B, nq * d), wo)
    gu = mm(norm(h, n2), wgu)
    h = h + mm(r16(torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]), wdown)
    ref = mm(norm(h, fin), head)
    # both sides round to bf16 at the same points; sums in another order flip the rounding of single activations,
    # by 2^-8 of one of K terms each, while a wrong K range or a lost split is of the order of the logits
    assert (logits - ref).abs().max().item() <= 2 ** -8 * ref.abs().max().item()
    eng.close()


WIDE = dict(name="wide-splits", n_layers=1, hidden=5120, n_q=8, n_kv=2, head_dim=128, ffn=27648, vocab=1024, dtype="bf16",
            rope_theta=10000.0, rms_eps=1e-5)
NARROW = dict(WIDE, name="narrow-splits", hidden=1024, ffn=8192)


@pytest.mark.parametrize("B", [40, 65, 80, 120, 128, 150, 160, 190, 250, 330, 650])
@pytest.mark.parametrize("cfg,wcn", [(WIDE, 4), (NARROW, 2)], ids=["wide", "narrow"])
def test_split_tiles_match_torch(cfg, wcn, B):
    plan = dma_plan(B, cfg["hidden"], cfg["ffn"])
    say("split tiles", cfg["name"], B, plan)
    assert plan[2] > 1 and plan[1] == wcn
    ar_against_torch(cfg, B)


@pytest.mark.parametrize("hidden", [384, 1024], ids=["whole", "split"])
@pytest.mark.parametrize("B", [1, 16, 17, 48, 64, 65, 130])
def test_streamed_head_matches_torch(B, hidden):
    say("streamed LM head", B, hidden)
    ar_against_torch(dict(WIDE, name="odd-vocab", hidden=hidden, ffn=512, vocab=64 * 5), B)
