"""The DMA-fed bf16 GEMM tiles at their edges: every height's last and next
row, widths of 128 and 256 columns, two, four, six and 18 K stages and rings that go
round, against torch in fp32; and the SwiGLU epilogue of every height against
the separate kernel, bit for bit (a verify whose gate/up runs unsplit)."""
import pytest
import torch

from paper_2606_18967_amd import sdrl, synth

from gpu_common import make_engine, say

pytestmark = pytest.mark.gpu


# N = 128 * odd takes 128-column tiles, 98304 (384 tiles of 256) the wide ones; K = 128: two stages; tiles start
# their K range at different stages with K = 4096 up to 160 rows, with 384 wide tiles from 65 to 160
@pytest.mark.parametrize("N,K", [(384, 128), (640, 384), (98304, 256), (1152, 1152), (512, 4096)])
@pytest.mark.parametrize("M", [64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 256, 257, 320, 321])
def test_dense_gemm_tile_edges(M, N, K):
    say("gemm tile edges", M, N, K)
    g = torch.Generator(device="cuda").manual_seed(M * 11 + N + K)
    A = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((N, K), generator=g, device="cuda").to(torch.bfloat16)
    out = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    sdrl.dense_gemm_bf16(A, W, out)
    ref = A.float() @ W.float().t()
    torch.cuda.synchronize()
    # exact products of bf16 values; K sums of them in fp32 on both sides: 2 K ulp of the largest |partial sum|,
    # far below 1e-5 of the row scale sqrt(K)
    assert (out - ref).abs().max().item() <= 1e-5 * K ** 0.5 * 8


# hidden 128 (K = 128) leaves no split, so the gate/up runs fused; F = 1024 in 128-column tiles, 50176 (odd count of
# 256-wide ones); with hidden 4096 F = 14336 runs unsplit up to 64 and from 97 rows, tiles starting at different stages
@pytest.mark.parametrize("rows,hidden,F", [(r, 128, f) for r in (64, 72, 100, 150, 190, 250, 330) for f in (1024, 50176)] +
                         [(r, 4096, 14336) for r in (2, 64, 100, 150)])
def test_fused_swiglu_equals_separate_kernel_at_every_height(rows, hidden, F):
    cfg = dict(name="heights", n_layers=1, hidden=hidden, n_q=2, n_kv=2, head_dim=64, ffn=F, vocab=256, dtype="bf16",
               rope_theta=500000.0, rms_eps=1e-5)
    gamma, S, B = 1, 16, rows // 2
    say("fused swiglu heights", rows, hidden, F)
    W = [w.cuda() for w in synth.make_weights(cfg, 23, "cpu" if hidden == 128 else "cuda")]
    eng, k, v, kv_len = make_engine(cfg, W, B, S + gamma + 4, gamma)
    synth.fill_kv_context(k, v, S, 29)
    kv_len.fill_(S)
    slots = torch.arange(B, dtype=torch.int32, device="cuda")
    toks = synth.make_tokens(B, gamma + 1, cfg["vocab"], 31).cuda()
    outs = []
    for unfused in (False, True):
        eng.set_debug(False, unfused_swiglu=unfused)
        p = torch.zeros((B, gamma + 1, cfg["vocab"]), dtype=torch.float32, device="cuda")
        eng.verify(slots, toks[:, 0].contiguous(), toks[:, 1:].contiguous(), gamma, p)
        eng.sync()
        outs.append(p.cpu())
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
    eng.close()
