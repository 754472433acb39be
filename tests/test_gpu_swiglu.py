"""SwiGLU of the fp32 decoder, bit for bit: SiLU(g) u with the quotient
g / (1 + e^-g) correctly rounded.

The decoder's one layer is made to hand (g, u) pairs from the embedding to the
logits without rounding: attention weights are zero, the gate, up and down
projections and the LM head pick single coordinates, and coordinate 0 holds
2^24, so that both norms divide by 2^20 exactly (the gains give it back).  For g
in [10, 16] the rounded 1 + e^-g is known whatever the exponential's last bits
are, except close to a tie (left out)."""
import numpy as np
import pytest
import torch

from paper_2606_18967_amd import sdrl

from gpu_common import i32, say

pytestmark = pytest.mark.gpu

P = 64                                             # pairs per token
CFG = dict(name="swiglu-f32", n_layers=1, hidden=256, n_q=2, n_kv=2, head_dim=64, ffn=128, vocab=128, dtype="f32",
           rope_theta=10000.0, rms_eps=1e-5)
EDGES = {-88.0: 1000.0, -88.5: 1000.0, -200.0: 5.0, 200.0: 3.0, 0.0: 7.0}   # 1 + e^-g past 2^126, infinite, 1; g = 0


def test_fp32_swiglu_is_the_rounded_quotient_times_u():
    say("fp32 swiglu")
    H, F, V = CFG["hidden"], CFG["ffn"], CFG["vocab"]
    rng = np.random.default_rng(3)
    g = rng.uniform(10, 16, (V, P)).astype(np.float32)
    u = rng.uniform(-4, 4, (V, P)).astype(np.float32)
    for i, (a, b) in enumerate(EDGES.items()):
        g[i, 0], u[i, 0] = a, b
    emb = np.zeros((V, H), np.float32)
    emb[:, 0], emb[:, 1:1 + P], emb[:, 1 + P:1 + 2 * P] = 2.0 ** 24, g, u
    at = np.arange(P)
    wgu, wdown, head = np.zeros((2 * F, H), np.float32), np.zeros((H, F), np.float32), np.zeros((V, H), np.float32)
    wgu[at, 1 + at] = 1
    wgu[F + at, 1 + P + at] = 1
    wdown[1 + 2 * P + at, at] = 1
    head[at, 1 + 2 * P + at] = 1
    head[P, 0] = 1
    gain, qkv = np.full(H, 2.0 ** 20, np.float32), 3 * 2 * 64
    W = [emb, gain, head, gain, np.zeros((qkv, H), np.float32), np.zeros((H, 128), np.float32), gain, wgu, wdown]
    eng = sdrl.Engine(CFG, V, 8, 1)
    eng.bind_weights([torch.from_numpy(w).cuda() for w in W])
    eng.bind_kv(*eng.alloc_kv())
    tok, out = i32(range(V)), torch.zeros(V, dtype=torch.int32, device="cuda")
    logits = torch.zeros((V, V), device="cuda")
    eng.ar_step(i32(range(V)), tok, 1.0, 1, 1, out, logits)
    eng.sync()
    got = logits.cpu().numpy()
    eng.close()
    assert (got[:, P] == 2.0 ** 24).all()          # both norms were exact
    got = got[:, :P]
    with np.errstate(over="ignore"):
        d64 = 1 + np.exp(-g.astype(np.float64))
        d = d64.astype(np.float32)
        want = g / d * u
    for i, a in enumerate(EDGES):                  # e^-g to a few times |g| 2^-24; the norms' 2^-20 leaves 2^-18 of -88's
        x = float(a / d64[i, 0] * EDGES[a])
        assert abs(got[i, 0] - x) <= 1e-4 * abs(x) + 1e-42, (a, got[i, 0], x)
    units = (d64 - 1) * 2.0 ** 23
    sure = (g >= 10) & (g <= 16) & (np.abs(units - np.floor(units) - 0.5) > 0.01)
    assert sure.mean() > 0.9
    assert np.array_equal(got[sure], want[sure]), (got[sure] != want[sure]).mean()
