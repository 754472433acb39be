"""The drafter refresh's short code path for bf16 weights against the division
path that fp32 weights take: the same weights in either type give the same
codes, scales and zero points, bit for bit."""
import pytest
import torch

from paper_2606_18967_amd import sdrl, synth

from gpu_common import say

pytestmark = pytest.mark.gpu

# K of 128 (one group, a work-group's last three waves idle), 384 and 640
CFG = dict(name="codes", n_layers=1, hidden=384, n_q=2, n_kv=1, head_dim=64, ffn=640, vocab=64, dtype="bf16",
           rope_theta=10000.0, rms_eps=1e-5)


def hard_groups(N, K, seed):
    """Rows of: N(0, 1) from 2^-30 to 2^30; exact ties of every code; offsets; zeros, constants, subnormal scales,
    infinities and NaN."""
    g = torch.Generator().manual_seed(seed)
    w = torch.randn((N, K), generator=g)
    w *= torch.exp2(torch.randint(-30, 31, (N, 1), generator=g).float())
    for r in range(0, N, 4):                       # multiples of half a scale, the largest 7, 15 or 127 scales
        most = (7, 15, 127)[(r // 4) % 3]
        c = 2.0 ** (r % 19 - 9) * (1 if most > 7 else 1 + 2 * (r % 8))
        half = torch.randint(-2 * most + 1, 2 * most, (K,), generator=g)
        half[::128] = 2 * most
        half[1::128] = 0 if most == 15 else -2 * most
        w[r] = half.abs() * c / 2 if most == 15 else half * c / 2
    for r in range(1, N, 16):
        w[r] = w[r] * 1e-3 + 4 * w[r].abs().max()  # zero points clamped at either end
        w[r + 1] = w[r].neg()
    w[2, :128] = 0
    w[6, :128] = 0.01
    w[10, :128] *= 0
    w[10, 5] = float("inf")
    w[14, 7] = float("nan")
    w[18, 9] = -float("inf")
    w[22] = 1e5 * 7                                # fp16 scale overflows
    w[26, :128] = torch.randn(128, generator=g) * 2e-7
    return w.to(torch.bfloat16)


@pytest.mark.parametrize("fmt", ["w4", "w4a", "w8"])
@pytest.mark.parametrize("seed", [1, 2])
def test_bf16_codes_equal_the_division_path(fmt, seed):
    say("refresh codes", fmt, seed)
    W = synth.make_weights(CFG, seed, "cpu")
    for i in (4, 5, 7, 8):
        W[i] = hard_groups(*W[i].shape, seed * 10 + i)
    got = []
    for dtype in ("bf16", "f32"):
        eng = sdrl.Engine(dict(CFG, dtype=dtype), 1, 8, 1)
        Wd = [(w.float() if dtype == "f32" else w).cuda() for w in W]
        eng.bind_weights(Wd)
        qbuf = torch.zeros(eng.drafter_bytes(fmt), dtype=torch.uint8, device="cuda")
        eng.refresh_drafter(qbuf, fmt)
        torch.cuda.synchronize()
        got.append(qbuf.cpu())
        eng.close()
    assert torch.equal(*got), int((got[0] != got[1]).sum())
