"""GPU parity of the attention's RoPE and new-row cache write where the new
rows straddle a context chunk.

With a bf16 cache the attention kernel itself rotates its query rows and
writes its KV head's new K (rotated) and V rows of its own context chunk
before reading them (k_attn_mfma).  The new rows are the last of a
sequence's context, so they cross a chunk start only where the last chunk is
that short; here each sequence's cached length (7k to 9k) puts a chunk start 1,
2, 3 or 4 positions into the gamma + 1 = 5 positions a verify writes: two
work-groups of every KV head each write their part, and the query rows read
rows both of them wrote.  The verify logits of every row and the new cache rows are
checked against the oracle's forward over the same tokens (positions
0 .. kv_len - 1 are the same random context on both sides), on a dense and
on a paged cache.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_18967_amd import sdrl, synth

from gpu_common import DeviceKV, host_bits, i32, oracle_kv_from_device, oracle_models, say
from test_gpu_attention_plan import chunks
from test_gpu_e2e import SMALL_GQA

pytestmark = pytest.mark.gpu

def _straddling_lengths(cfg, B, gamma, lo, hi):
    """B cached lengths whose gamma + 1 new positions cross a chunk start of their sequence, b + 1 positions in.
    Every sequence's chunks follow from all the lengths."""
    n = gamma + 1

    def inside(lens, b):
        return (lens[b] + b + 1) % chunks([x + n for x in lens], cfg["n_kv"])[b] == 0

    lens = [lo + 137 * b for b in range(B)]
    for b in range(B):
        for kl in range(lens[b], hi):
            trial = lens[:b] + [kl] + lens[b + 1:]
            if all(inside(trial, i) for i in range(b + 1)):
                lens = trial
                break
    assert all(inside(lens, b) for b in range(B)), lens
    return lens


@pytest.mark.parametrize("page", [0, 64], ids=["dense", "paged"])
def test_verify_rows_across_a_chunk_boundary_match_oracle(page):
    cfg, gamma, seed, tol = SMALL_GQA, 4, 21, 2e-2
    B, max_ctx = 4, 9000
    lens = _straddling_lengths(cfg, B, gamma, 7000, max_ctx - gamma - 1)
    say("verify across chunk boundaries", page, lens)
    W = synth.make_weights(cfg, seed, "cpu")
    eng = sdrl.Engine(cfg, B, max_ctx, gamma)
    eng.bind_weights([w.cuda() for w in W])
    kv = DeviceKV(eng, max_ctx, page, seed)
    kv.fill_context(max(lens), seed + 100)
    kv.kv_len.copy_(i32(lens))
    eng.refresh_drafter()
    torch.cuda.synchronize()
    kd0, vd0 = kv.dense()
    okv = [oracle_kv_from_device(cfg, kd0, vd0, b, lens[b], max_ctx) for b in range(B)]
    V = cfg["vocab"]
    toks = synth.make_tokens(B, gamma + 1, V, seed + 1)
    p = torch.zeros((B, gamma + 1, V), dtype=torch.float32, device="cuda")
    eng.verify(i32(range(B)), toks[:, 0].cuda().contiguous(), toks[:, 1:].cuda().contiguous(), gamma, p)
    eng.sync()
    kd, vd = kv.dense()
    target, _ = oracle_models(cfg, host_bits(W))
    pd = p.cpu().numpy()
    for b, kl in enumerate(lens):
        ol = oracle.forward_seq(target, okv[b], toks[b].numpy(), kl)
        for j in range(gamma + 1):
            assert np.abs(pd[b, j] - ol[j]).max() <= tol * np.abs(ol[j]).max(), (b, j)
        end = kl + gamma + 1
        kn = kd[:, b, :, kl:end].float().cpu().numpy()
        vn = vd[:, b, :, kl:end].float().cpu().numpy()
        ok, ov = okv[b].k[:, :, kl:end], okv[b].v[:, :, kl:end]
        assert np.abs(kn - ok).max() <= tol * np.abs(ok).max(), b
        assert np.abs(vn - ov).max() <= tol * np.abs(ov).max(), b
        # the cached context before the new rows is untouched
        assert torch.equal(kd[:, b, :, :kl], kd0[:, b, :, :kl]), b
    eng.close()
