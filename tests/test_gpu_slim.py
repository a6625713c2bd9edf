"""GPU tests of the action head's GEMM and of the short-key cache attention at
the sizes where their tiles, rounds and splits change."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from oracle import vla_oracle as O  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    assert torch.cuda.is_available()
    import paper_2609_22335_amd as mod
    return mod


# (dtype, M, N, K): row tiles 1, 1 + 1 row, 3 + 2 rows, 4; a last column block
# of 8; K of one piece, of a slab and a piece, at and past a wave's 4, 8, 16 and
# 24 slabs, and in rounds. resid_norm is the residual update and a norm launch
# after it; the norm folded into the update has a test file of its own
@pytest.mark.parametrize("dtype,M,N,K", [
    (1, 1, 8, 8), (1, 16, 40, 40), (1, 17, 1024, 1032), (1, 50, 1024, 2056), (1, 64, 1032, 4104), (1, 18, 2048, 6152),
    (0, 1, 8, 8), (0, 17, 72, 264), (0, 50, 1032, 1544), (0, 64, 128, 3080),
])
@pytest.mark.parametrize("kind", ["bias", "t", "gelu", "resid_norm"])
def test_action_gemm_edges(V, kind, dtype, M, N, K):
    import gpu_util as g
    g.say(f"slim gemm {kind} {dtype} {M}x{N}x{K}")
    rng = np.random.default_rng(M * 7919 + N * 31 + K)
    a = rng.standard_normal((M, K)).astype(np.float32)
    w = (0.05 * rng.standard_normal((N, K))).astype(np.float32)
    b = rng.standard_normal(N).astype(np.float32)
    opt = torch.bfloat16 if dtype else torch.float32
    A, W = torch.from_numpy(a).cuda().to(opt), torch.from_numpy(w).cuda().to(opt)
    a, w = A.double().cpu().numpy(), W.double().cpu().numpy()
    v = a @ w.T
    delta = 2 * K * 2.0 ** -24 * (np.abs(a) @ np.abs(w).T) + 2.0 ** -22 * (np.abs(v) + np.abs(b))
    ulp = 2.0 ** -8 if dtype else 2.0 ** -22
    bd = torch.from_numpy(b).cuda()
    if kind == "resid_norm":
        x0 = rng.standard_normal((M, N)).astype(np.float32)
        gain = (1 + 0.02 * rng.standard_normal(N)).astype(np.float32)
        x, out = torch.from_numpy(x0).cuda(), torch.full((M, N), float("nan"), dtype=opt, device="cuda")
        V.vla_debug_gemm_epi(dtype, M, N, K, A, W, kind, skinny=True, out=out, resid=x,
                             gain=torch.from_numpy(gain).cuda())
        ref = x0 + v
        assert (np.abs(x.double().cpu().numpy() - ref) <= delta + 2.0 ** -23 * np.abs(ref)).all()
        rms = np.sqrt((ref * ref).mean(1, keepdims=True) + 1e-6)
        ref = ref / rms * gain
        # the norm carries each row's largest error through 1 / rms
        bound = 4 * (np.abs(gain) + np.abs(ref)) * delta.max(1, keepdims=True) / rms + (ulp + 2.0 ** -20) * np.abs(ref)
    else:
        out = torch.full((M, N), float("nan"), dtype=torch.float32 if kind == "bias" else opt, device="cuda")
        V.vla_debug_gemm_epi(dtype, M, N, K, A, W, kind, skinny=True, bias=bd, out=out)
        ref = v + b
        if kind == "gelu":  # slope at most 1.13; the kernel's exp2 and reciprocal are good to about 1 ulp
            ref, delta = O.gelu_tanh(ref), 1.13 * delta + 2.0 ** -20 * np.abs(ref)
        bound = delta + (0 if kind == "bias" else ulp) * np.abs(ref) + 1e-30
    err = np.abs(out.double().cpu().numpy() - ref)
    assert (err <= bound).all(), (err.max(), (err / bound).max())


# (Sq, nq, nkv, hd, S0, S1): tiles split four ways, in two and unsplit along
# the head dim; key blocks at 8, 12 and 16 and one past, two and three chunks;
# ragged segments; a last query tile of one row
@pytest.mark.parametrize("Sq,nq,nkv,hd,S0,S1", [
    (50, 8, 1, 256, 305, 50), (50, 8, 1, 256, 256, 0), (50, 8, 1, 256, 257, 0), (33, 8, 1, 256, 384, 0),
    (51, 8, 1, 256, 352, 33), (50, 8, 1, 256, 833, 50), (130, 8, 1, 256, 512, 1), (305, 8, 1, 256, 305, 0),
    (833, 8, 1, 256, 833, 0), (1, 1, 1, 256, 1, 0), (16, 4, 4, 128, 96, 0), (96, 16, 16, 128, 96, 0),
    (17, 3, 1, 128, 300, 17), (40, 16, 2, 128, 1100, 31), (200, 8, 8, 128, 513, 0),
])
def test_cache_attention_chunks(V, Sq, nq, nkv, hd, S0, S1):
    import gpu_util as g
    g.say(f"cache attention {Sq} {nq}/{nkv} hd {hd} keys {S0}+{S1}")
    rng = np.random.default_rng(Sq * 1009 + S0)
    rnd = lambda s, n: torch.from_numpy(rng.standard_normal((s, n, hd)).astype(np.float32)).to(torch.bfloat16)
    q, k, v = 2 * rnd(Sq, nq), rnd(S0 + S1, nkv), rnd(S0 + S1, nkv)
    dk, dv = [], []
    for x, y in ((k[:S0], v[:S0]), (k[S0:], v[S0:])):
        if not x.shape[0]:
            dk.append(None)
            dv.append(None)
            continue
        kc, vc = cache_layout(x, y)
        dk.append(kc.cuda())
        dv.append(vc.cuda())
    out = torch.full((Sq, nq, hd), float("nan"), dtype=torch.bfloat16, device="cuda")
    V.vla_debug_attention_cache(1, Sq, nq, nkv, hd, q.cuda(), dk[0], dv[0], S0, dk[1], dv[1], S1, out)
    torch.cuda.synchronize()
    ref = O.attention(*(t.double().numpy() for t in (q, k, v)))
    err = np.abs(out.double().cpu().numpy() - ref)
    # one bf16 rounding; scores and P (two bf16 parts) to well under 1e-4 of values of order 1
    assert (err <= 2.0 ** -8 * np.abs(ref) + 2e-4).all(), err.max()


# The same on both sides of each line between the two cache-attention kernels:
# one chunk of 16 key blocks and one block more, two full chunks, the second
# nearly full or not, three chunks with 8 query tiles and with fewer, and the
# long keys that k_attn2 splits over workgroups
@pytest.mark.parametrize("Sq,nq,nkv,hd,S0,S1", [
    (50, 8, 1, 128, 512, 0), (50, 8, 1, 128, 513, 0), (17, 8, 2, 128, 896, 0), (17, 8, 2, 128, 870, 27),
    (3, 16, 16, 128, 1024, 0), (50, 8, 1, 128, 1000, 25), (1, 8, 1, 128, 3000, 0), (50, 8, 1, 256, 1024, 0),
    (50, 8, 1, 256, 1025, 0), (16, 8, 1, 256, 1480, 50), (15, 8, 1, 256, 1480, 50), (50, 4, 4, 256, 1537, 0),
    (1, 1, 1, 256, 3000, 17),
])
def test_cache_attention_kernel_choice(V, Sq, nq, nkv, hd, S0, S1):
    test_cache_attention_chunks(V, Sq, nq, nkv, hd, S0, S1)


def test_long_prefix_bf16_heads(V):
    """A model whose key blocks lie past the first chunk: one frame against
    the oracle; action groups of four, three and two bit for bit alike
    (launches that may be batched take one kernel, unsplit, whatever the group)."""
    import gpu_util as g
    import synth
    import test_gpu_parity as P
    cfg = dict(synth.micro(synth.BF16), head_dim=128, n_text=560)
    P.test_phases_vs_oracle(V, "micro-bf16-hd128-long", cfg)
    frames = [g.DevFrame(synth.make_frame(cfg, 0, r)) for r in range(5)]
    noise = torch.stack([f.noise for f in frames])
    got = []
    with g.model(cfg, 0) as m:
        for batch in (4, 3, 2):  # (five frames: 4 + 1, 3 + 2, 2 + 2 + 1)
            out = torch.full_like(noise, float("nan"))
            V.vla_pipeline_run(m, [f.c for f in frames], noise, 5, mode="serial", actions=out, act_batch=batch,
                               vlm_batch=2)
            torch.cuda.synchronize()
            got.append(out)
    # (a group of one frame takes the one-frame action phase)
    assert bool(torch.isfinite(got[0]).all())
    assert torch.equal(got[0][:4], got[1][:4]) and torch.equal(got[0][:4], got[2][:4])


def cache_layout(k, v):
    """bf16 K / V rows [S, nkv, hd] in the KV-cache layout (include/vla.h);
    unused K positions hold NaN, unused V positions zero."""
    S, nkv, hd = k.shape
    nb, ns, ndt = (S + 31) // 32, (hd + 31) // 32, (hd + 15) // 16
    p = torch.arange(S).view(S, 1, 1)
    j = torch.arange(nkv).view(1, nkv, 1)
    d = torch.arange(hd).view(1, 1, hd)
    b, kin = p // 32, p % 32
    ki = ((((j * nb + b) * 2 + (kin // 4) % 2) * ns + d // 32) * 64 + 16 * ((d % 32) // 8) + 4 * (kin // 8) + kin % 4) * 8 + d % 8
    vi = (((j * nb + b) * ndt + d // 16) * 64 + 16 * (kin // 8) + d % 16) * 8 + kin % 8
    K = torch.full((nkv * nb * 32 * ns * 32,), float("nan"), dtype=torch.bfloat16)
    W = torch.zeros(nkv * nb * 32 * ndt * 16, dtype=torch.bfloat16)
    K[ki.reshape(-1)] = k.reshape(-1)
    W[vi.reshape(-1)] = v.reshape(-1)
    return K, W


# (kind, M, N, K, row padding): each launch of the tiled GEMM, at its edges.
# 64 x 64 in the ring of four (one K-tile and a piece, three, four, five; one
# row and one column past a tile; split K) and, past 512 tiles, in two stages;
# 128 x 128 with whole and ragged last tiles; the 320-row tile from 257 to 320
# rows; 256 x 256 plans that run in 128 x 128 tiles or stay; GELU, whose 256 x 256
# tiles have four waves
@pytest.mark.parametrize("kind,M,N,K,pad", [
    ("f32", 33, 8, 8, 0), ("f32", 64, 64, 72, 8), ("f32", 65, 72, 192, 0), ("f32", 129, 200, 256, 8),
    ("f32", 100, 1032, 328, 0), ("f32", 40, 64, 4104, 0), ("f32", 400, 1024, 1024, 64), ("f32", 520, 4168, 136, 0),
    ("f32", 256, 16384, 64, 0), ("f32", 385, 10248, 200, 8), ("f32", 257, 24576, 136, 0), ("f32", 320, 24584, 264, 8),
    ("f32", 321, 24576, 72, 0), ("f32", 1025, 12936, 72, 0), ("f32", 2440, 8192, 328, 0), ("f32", 4096, 4096, 136, 8),
    ("geglu", 400, 8192, 200, 0), ("geglu", 305, 32768, 136, 0), ("geglu", 2440, 32768, 136, 0),
    ("geglu", 100, 1056, 328, 0), ("gelu", 2048, 4304, 136, 0), ("gelu", 4100, 4304, 200, 0), ("t", 256, 3456, 1152, 0),
])
def test_gemm_tiles(V, kind, M, N, K, pad):
    import gpu_util as g
    g.say(f"gemm {kind} {M}x{N}x{K} +{pad}")
    gen = torch.Generator(device="cuda").manual_seed(M * 7919 + N * 31 + K)
    bias = torch.randn(N, generator=gen, device="cuda") if kind != "geglu" else None
    # rows of K + pad elements, the padding infinite: nothing of it may be read into a sum
    ops = []
    for rows, scale in ((M, 1.0), (N, 0.05)):
        buf = torch.full((rows * (K + pad) + 8,), float("inf"), dtype=torch.bfloat16, device="cuda")
        val = (scale * torch.randn(rows, K, generator=gen, device="cuda")).bfloat16()
        ops.append((buf, val))

    def run(off):
        """The operands start `off` elements past 16 bytes."""
        for buf, val in ops:
            buf[off:off + val.shape[0] * (K + pad)].view(val.shape[0], K + pad)[:, :K] = val
        A, W = (buf[off:] for buf, _ in ops)
        out = torch.full((M, N // 2 if kind == "geglu" else N), float("nan"), device="cuda",
                         dtype=torch.float32 if kind == "f32" else torch.bfloat16)
        if kind == "f32":
            V.vla_debug_gemm(1, M, N, K, A, K + pad, W, K + pad, bias, out)
        else:
            V.vla_debug_gemm_epi(1, M, N, K, A, W, kind, bias=bias, out=out)
        torch.cuda.synchronize()
        return out

    out = run(0)
    a, w = (val.double() for _, val in ops)
    v, mag = a @ w.T, a.abs() @ w.abs().T
    delta = 2 * K * 2.0 ** -24 * mag
    if kind == "geglu":
        (gt, up), (dg, du) = v.chunk(2, 1), delta.chunk(2, 1)  # W holds the gate rows, then the up rows
        act = 0.5 * gt * (1 + torch.tanh((2 / np.pi) ** 0.5 * (gt + 0.044715 * gt ** 3)))
        ref = act * up
        delta = up.abs() * 1.13 * dg + act.abs() * du + 1.13 * dg * du + 2.0 ** -20 * ref.abs()
    else:
        ref = v + bias.double()
        delta = delta + 2.0 ** -22 * (v.abs() + bias.abs())
        if kind == "gelu":
            ref = 0.5 * ref * (1 + torch.tanh((2 / np.pi) ** 0.5 * (ref + 0.044715 * ref ** 3)))
            delta = 1.13 * delta + 2.0 ** -20 * ref.abs()
    # (1e-6: gelu's tail, where 1 + tanh loses what tanh rounds away)
    bound = delta + (0 if kind == "f32" else 2.0 ** -8) * (ref.abs() + delta) + 1e-6
    err = (out.double() - ref).abs()
    assert bool((err <= bound).all()), (float(err.max()), float((err / bound).max()))
    # operands 8 bytes past a 16-byte boundary go through the register-staged
    # tile: the same sums, bit for bit
    assert torch.equal(run(4), out)


# K on both sides of the lines between the 64 x 64 tile's ring, its two stages
# and its register-staged form (two K-tiles and three, five and six), and
# between the 320-row tile and the 128 one (K 256)
@pytest.mark.parametrize("kind,M,N,K", [
    ("geglu", 150, 1024, 8), ("geglu", 150, 1056, 128), ("geglu", 150, 1024, 136), ("t", 150, 1032, 64),
    ("t", 129, 1024, 320), ("t", 129, 1024, 328), ("gelu", 65, 72, 320), ("f32", 400, 4096, 128),
    ("geglu", 300, 32768, 192), ("geglu", 300, 32768, 256), ("f32", 257, 24584, 248),
])
def test_gemm_short_k(V, kind, M, N, K):
    test_gemm_tiles(V, kind, M, N, K, 0)


# Operands off 16 bytes by one, two and four elements, and with rows of more
# than 2 MB, on every tile they take: the sums of aligned, packed operands
@pytest.mark.parametrize("M,N,K,ld", [(2440, 8192, 328, 0), (1025, 16384, 72, 0), (305, 16384, 200, 0), (400, 1024, 136, 0),
                                      (129, 4104, 72, (1 << 20) + 8), (257, 16392, 72, (1 << 20) + 8)])
def test_gemm_unaligned(V, M, N, K, ld):
    import gpu_util as g
    g.say(f"gemm unaligned {M}x{N}x{K} ld {ld}")
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    w = (0.05 * torch.randn(N, K, generator=gen, device="cuda")).bfloat16()

    def run(off, lda):
        A = torch.full((M * lda + 8,), float("inf"), dtype=torch.bfloat16, device="cuda")
        W = torch.full((N * K + 8,), float("inf"), dtype=torch.bfloat16, device="cuda")
        A[off:off + M * lda].view(M, lda)[:, :K] = a
        W[off:off + N * K] = w.flatten()
        out = torch.full((M, N), float("nan"), device="cuda")
        V.vla_debug_gemm(1, M, N, K, A[off:], lda, W[off:], K, None, out)
        torch.cuda.synchronize()
        return out

    ref = run(0, K)
    bound = 2 * K * 2.0 ** -24 * (a.double().abs() @ w.double().abs().T)
    assert bool(((ref.double() - a.double() @ w.double().T).abs() <= bound).all())
    for off, lda in ((0, ld),) if ld else ((1, K), (2, K), (4, K)):
        assert torch.equal(run(off, lda), ref), (off, lda)


# Streams of fewer CUs take other launch shapes (one, two or four row tiles of
# the action GEMMs, ring or two stages of the 64 x 64 tile), each with a graph of
# its own: the same chunks, bit for bit, one mask after another on one model
@pytest.mark.parametrize("batch", [1, 2])
def test_masked_launch_shapes(V, batch):
    import gpu_util as g
    import synth
    cfg = dict(synth.micro(synth.BF16), chunk_len=50, ex_dim=256, ex_mlp=1024)
    frames = [g.DevFrame(synth.make_frame(cfg, 0, r)) for r in range(4)]
    noise = torch.stack([f.noise for f in frames])

    with g.model(cfg, 0) as m:
        def run(**kw):
            out = torch.full_like(noise, float("nan"))
            V.vla_pipeline_run(m, [f.c for f in frames], noise, 4, actions=out, act_batch=batch, vlm_batch=batch, **kw)
            torch.cuda.synchronize()
            return out

        ref = run(mode="serial")
        assert bool(torch.isfinite(ref).all())
        for vlm, act in ((64, 8), (8, 16), (128, 24), (152, 40), (16, 64)):
            for graphs in (True, False, True):
                g.say(f"masks {vlm}/{act} graphs {graphs} batch {batch}")
                assert torch.equal(run(mode="cu_masked", vlm_cus=vlm, act_cus=act, graphs=graphs), ref), (vlm, act)


def test_large_tiles_under_a_workgroup_cap(V):
    """The 320-row tile (one frame's prefix of 287 rows) and a plan of 256 x 256
    tiles that runs in 128 x 128 ones (four frames), each with more tiles than
    the 256 workgroups of the cap: the bits of the uncapped launches."""
    import gpu_util as g
    import synth
    import test_gpu_parity as P
    cfg = dict(synth.micro(synth.BF16), lm_dim=256, lm_mlp=20480, n_text=270, lm_layers=2, ex_layers=2)
    P.test_phases_vs_oracle(V, "micro-bf16-wide-lm", cfg)
    frames = [g.DevFrame(synth.make_frame(cfg, 0, r)) for r in range(4)]
    noise = torch.stack([f.noise for f in frames])
    with g.model(cfg, 0) as m:
        ref = None
        for kw in (dict(mode="serial"), dict(mode="serial", vlm_batch=4), dict(mode="wg_capped", vlm_wg_cap=1),
                   dict(mode="wg_capped", vlm_wg_cap=1, vlm_batch=4), dict(mode="wg_capped", vlm_wg_cap=1, graphs=True)):
            g.say(f"large tiles {kw}")
            out = torch.full_like(noise, float("nan"))
            V.vla_pipeline_run(m, [f.c for f in frames], noise, 4, actions=out, **kw)
            torch.cuda.synchronize()
            ref = out if ref is None else ref
            assert bool(torch.isfinite(out).all()) and torch.equal(out, ref), kw


def test_attention_parts_in_groups(V):
    """Action attention at head dim 256: groups of two and four frames split a
    query tile along the head dim in two, a group of eight does not (200 tiles);
    the chunks are the same bits."""
    import gpu_util as g
    import synth
    cfg = dict(synth.micro(synth.BF16), head_dim=256, lm_heads=8, chunk_len=50)
    frames = [g.DevFrame(synth.make_frame(cfg, 0, r)) for r in range(8)]
    noise = torch.stack([f.noise for f in frames])
    got = []
    with g.model(cfg, 0) as m:
        for batch in (8, 4, 2):
            g.say(f"attention groups of {batch}")
            out = torch.full_like(noise, float("nan"))
            V.vla_pipeline_run(m, [f.c for f in frames], noise, 8, mode="serial", actions=out, act_batch=batch)
            torch.cuda.synchronize()
            got.append(out)
    assert bool(torch.isfinite(got[0]).all())
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


# Vectors that are there but neutral (zero bias and shift, a column scale of
# one) and splits that are there but zero take other variants of the norms:
# the same sums, bit for bit. Rows of one wave (d <= 1024) and of a workgroup.
@pytest.mark.parametrize("dtype,rows,d,rms", [(1, 1, 8, 1), (1, 400, 1024, 1), (1, 17, 1028, 0), (1, 5000, 2048, 1),
                                              (0, 3, 256, 0), (0, 70, 2048, 0)])
def test_norm_variants(V, dtype, rows, d, rms):
    import gpu_util as g
    g.say(f"norm variants {dtype} {rows}x{d} rms {rms}")
    gen = torch.Generator(device="cuda").manual_seed(rows + d)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    x0, gain, zero, one = r(rows, d), 1 + 0.1 * r(d), torch.zeros(d, device="cuda"), torch.ones(d, device="cuda")
    part = torch.zeros(9, rows, d, device="cuda")
    part[:4] = 0.25 * r(4, rows, d)

    def run(splits, vecs):
        x = x0.clone()
        out = torch.full((rows, d), float("nan"), dtype=torch.bfloat16 if dtype else torch.float32, device="cuda")
        V.vla_debug_norm(dtype, rows, d, x, d, part if splits else None, splits, zero if vecs else None,
                         one if vecs and splits else None, gain, 0, zero if vecs else None, rms, out, d, 0)
        torch.cuda.synchronize()
        return x, out

    for counts in ((0,), (4, 5, 8, 9)):
        got = [run(sp, v) for sp in counts for v in (False, True)]
        x = x0.double() + (part[:4].double().sum(0) if counts[0] else 0)
        c = x if rms else x - x.mean(1, keepdim=True)
        ref = c / torch.sqrt((c * c).mean(1, keepdim=True) + 1e-6) * gain.double()
        # sums of at most 2048 values of a row of standard deviation ~1, and one rounding
        bound = (2.0 ** -8 if dtype else 2.0 ** -23) * ref.abs() + 64 * 2.0 ** -23 * (1 + ref.abs())
        assert bool(((got[0][1].double() - ref).abs() <= bound).all())
        for y in got[1:]:
            assert torch.equal(y[0], got[0][0]) and torch.equal(y[1], got[0][1])
