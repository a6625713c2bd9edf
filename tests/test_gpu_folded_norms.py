"""GPU tests of the norms that the action head's GEMMs carry: the RMSNorm folded
across two launches, the gated residual update, the LayerNorm applied as the
operand is loaded, and the launch of its own that stands in for it."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import synth  # noqa: E402
from oracle import vla_oracle as O  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    assert torch.cuda.is_available()
    import paper_2609_22335_amd as mod
    return mod


# Row sums in blocks of 16 columns (N <= 1024) and of 32 (beyond), a last block
# of 8 and of 32 columns, the most blocks there are (64); one row, row tiles of
# one row and of two, all four
@pytest.mark.parametrize("dtype,M,N,K", [
    (1, 1, 8, 40), (1, 17, 1024, 1032), (1, 50, 1024, 4096), (1, 64, 1032, 520), (1, 1, 1056, 72), (1, 50, 1056, 2056),
    (1, 17, 2048, 136), (1, 64, 2048, 4104), (0, 50, 1024, 264), (0, 17, 1032, 1544), (0, 64, 2048, 72), (0, 1, 2040, 8),
])
@pytest.mark.parametrize("gated", [False, True])
def test_folded_rmsnorm(V, dtype, M, N, K, gated):
    import gpu_util as g
    g.say(f"folded norm {dtype} {M}x{N}x{K} gated {gated}")
    gen = torch.Generator(device="cuda").manual_seed(M * 7919 + N * 31 + K)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    opt = torch.bfloat16 if dtype else torch.float32
    N2 = 72
    A, W, W2 = r(M, K).to(opt), (0.05 * r(N, K)).to(opt), (0.05 * r(N2, N)).to(opt)
    cs, gain, x0 = r(N) if gated else None, 1 + 0.1 * r(N), r(M, N)
    x, norm = x0.clone(), torch.full((M, N), float("nan"), dtype=opt, device="cuda")
    out = torch.full((M, N2), float("nan"), device="cuda")
    V.vla_debug_gemm_fold(dtype, M, N, K, A, W, cs, gain, x, norm, N2, W2, out)
    d = lambda t: t.double()
    one = d(cs).abs() if gated else 1.0
    ref = d(x0) + (d(cs) if gated else 1.0) * (d(A) @ d(W).T)
    # fp32 sums of K products, then the update's roundings
    bound = 2 * K * 2.0 ** -24 * one * (d(A).abs() @ d(W).abs().T) + 2.0 ** -22 * (ref.abs() + d(x0).abs())
    err = (d(x) - ref).abs()
    assert bool((err <= bound).all()), float((err / bound).max())
    # the operand is the new x, as it was stored, times the gain, rounded once
    ref = d(x) * d(gain)
    err = (d(norm) - ref).abs()
    assert bool((err <= (2.0 ** -8 if dtype else 2.0 ** -23) * ref.abs()).all())
    # and the consumer's product is scaled by the rms of that x: N squares in
    # blocks and the blocks in a tree, the root and the division, 16 roundings
    rms = torch.sqrt((d(x) ** 2).mean(1, keepdim=True) + 1e-6)
    ref = d(norm) @ d(W2).T / rms
    bound = 2 * N * 2.0 ** -24 * (d(norm).abs() @ d(W2).abs().T) / rms + 2.0 ** -20 * ref.abs()
    err = (d(out) - ref).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


# K of one 16-byte piece and ragged, at and past the 512, 1024 and 1536 columns
# where the kernel's registers change; row tiles as above
@pytest.mark.parametrize("dtype,M,N,K", [
    (1, 1, 8, 8), (1, 17, 72, 504), (1, 50, 1024, 512), (1, 64, 1032, 520), (1, 16, 40, 1016), (1, 50, 2048, 1024),
    (1, 33, 72, 1032), (1, 64, 1536, 1536), (0, 1, 8, 40), (0, 50, 128, 512), (0, 17, 1032, 520), (0, 64, 72, 1024),
])
@pytest.mark.parametrize("form", ["plain", "adaptive", "gelu"])
def test_gemm_over_layernorm(V, dtype, M, N, K, form):
    import gpu_util as g
    g.say(f"gemm over a layernorm {dtype} {M}x{N}x{K} {form}")
    gen = torch.Generator(device="cuda").manual_seed(M * 7919 + N * 31 + K)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    opt = torch.bfloat16 if dtype else torch.float32
    x, W, b = 2 * r(M, K) + 0.5, (0.05 * r(N, K)).to(opt), r(N)
    plus = form == "adaptive"  # gain 1 + scale, as the timestep's modulation gives it
    gain, shift = (0.1 * r(K) if plus else 1 + 0.1 * r(K)), None if form == "plain" else 0.1 * r(K)
    out = torch.full((M, N), float("nan"), dtype=opt, device="cuda")
    V.vla_debug_gemm_ln(dtype, M, N, K, x, gain, int(plus), shift, W, b, form == "gelu", out)
    d = lambda t: t.double()
    c = d(x) - d(x).mean(1, keepdim=True)
    h = c / torch.sqrt((c * c).mean(1, keepdim=True) + 1e-6) * (d(gain) + plus)
    if shift is not None:
        h = h + d(shift)
    ref = h @ d(W).T + d(b)
    # the operand's rounding to its type, the fp32 statistics and the product's
    # fp32 sums
    half = 2.0 ** -9 if dtype else 0.0
    bound = ((half + 2.0 ** -16) * (1 + h.abs()) + 2 * K * 2.0 ** -24 * h.abs()) @ d(W).abs().T
    bound = bound + 2.0 ** -22 * (ref.abs() + d(b).abs())
    if form == "gelu":
        ref = torch.from_numpy(O.gelu_tanh(ref.cpu().numpy())).cuda()
        bound = 1.13 * bound + 2.0 ** -20 * ref.abs()
    err = (d(out) - ref).abs()
    bound = bound + (2.0 ** -8 if dtype else 2.0 ** -22) * (ref.abs() + bound) + 1e-6
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("dtype,M,N,K", [(1, 50, 64, 1544), (0, 50, 64, 1032), (1, 33, 6144, 1536)])
def test_layernorm_shapes_that_need_a_launch(V, dtype, M, N, K):
    """Too wide a row, or too many tiles, is refused here; the model runs the
    norm as a launch of its own (below)."""
    t = torch.zeros(1, device="cuda")
    with pytest.raises(V.VlaError) as e:
        V.vla_debug_gemm_ln(dtype, M, N, K, t, t, 0, None, t, None, False, t)
    assert e.value.code == -4


# pi0 widths past 1024 (row sums in blocks of 32 columns), one frame and groups
@pytest.mark.parametrize("dtype,ex_dim", [(synth.BF16, 1056), (synth.F32, 1056), (synth.BF16, 2048)])
def test_wide_expert(V, dtype, ex_dim):
    import test_gpu_parity as P
    P.test_phases_vs_oracle(V, f"micro-wide-{dtype}-{ex_dim}", dict(synth.micro(dtype), ex_dim=ex_dim, chunk_len=50))


# the norm as a launch before the GEMM: more tiles than it takes (chunk rows
# from 33 at 8192 columns), and fp32 rows past 1024 columns
@pytest.mark.parametrize("cfg", [dict(synth.micro_dit(synth.BF16), chunk_len=40, ex_mlp=8192),
                                 dict(synth.micro_dit(synth.F32), ex_dim=1056, ex_heads=12),
                                 dict(synth.micro_cog(synth.F32), ex_dim=1056, ex_heads=12)],
                         ids=["dit-tiles", "dit-fp32-wide", "cog-fp32-wide"])
def test_layernorm_as_a_launch(V, cfg):
    import test_gpu_parity as P
    if cfg["head"] == synth.HEAD_COG:
        P.test_cog_phases_vs_oracle(V, "norm-launch", cfg)
    else:
        P.test_dit_phases_vs_oracle(V, "norm-launch", cfg)
