"""Performance cases: the work that users of this library have it do.

Kinds of case (all through the binding's public entry points):

* ``frame``     one robot's control step: ``vla_vlm_prefill`` then
                ``vla_action_denoise`` on one stream; the action chunk;
* ``denoise``   the action phase alone on a prefilled context;
* ``pipeline``  ``vla_pipeline_run`` over R frames with a schedule; every chunk;
* ``gemm``      ``vla_gemm_noalloc``: one projection, row-major weights;
* ``attention`` ``vla_debug_attention_cache``: one attention layer over the
                KV cache (prefix segment, and the expert's own segment);
* ``norm``      ``vla_debug_norm``: one LayerNorm / RMSNorm over many rows.

A model is named by a preset, with some of its fields changed where the case
says so (``set_<field>``): a model with one or two layers of full width is how
a single block of a stack is measured end to end. Models keep the weights of
seed 0 and are shared by the states that use them, as in a serving program;
images, instructions, states, noise and the operands of single kernels come
from the case's seed.
"""
import math
import threading
from collections import OrderedDict

import numpy as np
import torch

import paper_2609_22335_amd as V

DEV = "cuda"
MODEL_SEED = 0
HEAD_PI0, HEAD_DIT, HEAD_COG = 0, 1, 2
F32, BF16 = 0, 1


# --------------------------------------------------------------------------
# Cases
# --------------------------------------------------------------------------

def listed():
    return [
        # the smallest whole call: a tiny fp32 policy's control step, bound by
        # launches (and the only use of fp32 operands in the models)
        {"name": "tiny_frame", "kind": "frame", "preset": "tiny"},
        # one robot, one frame: the latency of a PaliGemma-3B-shaped policy
        # with a flow-matching expert
        {"name": "pi0_frame", "kind": "frame", "preset": "pi0"},
        # the action loop alone: a further chunk from a context that is there
        # (asynchronous inference), 10 Euler steps
        {"name": "pi0_denoise", "kind": "denoise", "preset": "pi0"},
        # the two-phase overlap of independent one-frame phases: eight robots,
        # no batching, two action lanes, graphs
        {"name": "pi0_overlap", "kind": "pipeline", "preset": "pi0", "R": 8, "mode": "concurrent",
         "act_streams": 2, "graphs": True, "vlm_batch": 1, "act_batch": 1, "act_chunks": 1},
        # eight robots streaming frames, four steps: prefills of eight beside
        # action loops of eight (the largest throughput workload)
        {"name": "pi0_serving", "kind": "pipeline", "preset": "pi0", "R": 32, "mode": "concurrent",
         "act_streams": 2, "graphs": True, "vlm_batch": 8, "act_batch": 8, "act_chunks": 1},
        # three cameras per robot (833-row prefixes), eight robots, two steps
        {"name": "pi0_3view_serving", "kind": "pipeline", "preset": "pi0_3view", "R": 16, "mode": "concurrent",
         "act_streams": 2, "graphs": True, "vlm_batch": 8, "act_batch": 8, "act_chunks": 1},
        # the DiT head (one-frame loops only) under batched prefills
        {"name": "gr00t_serving", "kind": "pipeline", "preset": "gr00t", "R": 16, "mode": "concurrent",
         "act_streams": 4, "graphs": True, "vlm_batch": 8, "act_batch": 1, "act_chunks": 1},
        # the cognition-token diffusion head, one robot's control step (DDIM)
        {"name": "cogact_frame", "kind": "frame", "preset": "cogact"},
        # single blocks of the pi0-shaped stacks: one ViT, two LM and two
        # expert layers, two cameras, ragged text and chunk, two Euler steps
        {"name": "pi0_block", "kind": "frame", "preset": "pi0", "set_n_views": 2, "set_n_text": 23,
         "set_vit_layers": 1, "set_lm_layers": 2, "set_ex_layers": 2, "set_chunk_len": 37, "set_n_steps": 2},
        # one projection of the LM MLP over one frame's prefix
        {"name": "gemm_prefix", "kind": "gemm", "dtype": BF16, "M": 305, "N": 16384, "K": 2048, "bias": False},
        # the expert's joint attention: 50 action queries over [prefix; own]
        {"name": "attention_expert", "kind": "attention", "dtype": BF16, "Sq": 50, "nq": 8, "nkv": 1, "hd": 256,
         "S0": 305, "S1": 50},
        # one pre-norm over the stacked prefixes of eight robots
        {"name": "norm_prefix", "kind": "norm", "dtype": BF16, "rows": 2440, "d": 2048, "rms": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["gemm", "attention", "norm", "block", "denoise", "pipeline"], [5, 4, 2, 5, 2, 4])[0]
    if kind == "gemm":
        dtype = F32 if rng.random() < 0.15 else BF16
        while True:
            M, N, K = _log_int(rng, 1, 4096), _log_int(rng, 16, 32768), 8 * _log_int(rng, 4, 2048)
            if M * N * K <= (1 << 33 if dtype == F32 else 1 << 37):
                return {"kind": "gemm", "dtype": dtype, "M": M, "N": N, "K": K, "bias": rng.random() < 0.5}
    if kind == "attention":
        dtype = F32 if rng.random() < 0.15 else BF16
        hd = rng.choice([32, 48, 64, 72, 96, 128] + ([256, 256, 256] if dtype == BF16 else []))
        nkv = rng.choice([1, 1, 2, 4, 16])
        nq = nkv * rng.choice([1, 2, 8]) if nkv < 16 else nkv
        if rng.random() < 0.5:  # an action head over [prefix; own keys]
            Sq = rng.randint(4, 64)
            S0, S1 = _log_int(rng, 16, 1536), Sq
        else:  # a prefix over itself
            Sq = S0 = _log_int(rng, 16, 1536)
            S1 = 0
        return {"kind": "attention", "dtype": dtype, "Sq": Sq, "nq": nq, "nkv": nkv, "hd": hd, "S0": S0, "S1": S1}
    if kind == "norm":
        return {"kind": "norm", "dtype": F32 if rng.random() < 0.2 else BF16, "rows": _log_int(rng, 1, 6664),
                "d": 4 * _log_int(rng, 8, 512), "rms": rng.random() < 0.5}
    if kind == "block":
        # one or two layers of each stack at ragged sizes
        dtype = F32 if rng.random() < 0.2 else BF16
        big = dtype == BF16 and rng.random() < 0.6
        preset = rng.choice(["pi0", "pi0", "gr00t", "cogact"] if big else ["tiny", "tiny_dit", "tiny_cog", "tiny_ddim"])
        layers = rng.randint(1, 2)
        c = {"kind": "frame", "preset": preset, "set_dtype": dtype, "set_n_views": rng.randint(1, 3),
             "set_n_text": rng.randint(0, 80), "set_vit_layers": rng.randint(1, 2), "set_lm_layers": layers,
             "set_ex_layers": layers if preset in ("pi0", "tiny", "tiny_ddim") else 2 * rng.randint(1, 2),
             "set_chunk_len": rng.randint(3, 62), "set_action_dim": rng.randint(3, 32),
             "set_state_dim": 0 if preset in ("cogact", "tiny_cog") else rng.choice([0, 7, 32]),
             "set_n_steps": rng.randint(1, 4),
             "set_lm_mlp": (16 * _log_int(rng, 64, 1024)) if big else 16 * rng.randint(8, 128),
             "set_ex_mlp": (16 * _log_int(rng, 32, 256)) if big else 16 * rng.randint(4, 64)}
        if preset in ("tiny_ddim", "tiny_cog", "cogact"):
            c["set_n_steps"] = rng.randint(4, 10)
        return c
    if kind == "denoise":
        return {"kind": "denoise", "preset": rng.choice(["pi0", "pi0", "gr00t", "cogact"])}
    # schedules of the pi0-shaped pipeline
    vb, ab = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 3, 4, 8])
    serial = rng.random() < 0.2
    chunks = rng.choice([1, 1, 1, 2])
    most = 32 if max(vb, ab) >= 4 else 6
    return {"kind": "pipeline", "preset": "pi0", "R": max(1, rng.randint(2, most) // chunks),
            "mode": "serial" if serial else "concurrent", "act_streams": 1 if serial else rng.randint(1, 3),
            "graphs": rng.random() < 0.8, "vlm_batch": vb, "act_batch": ab, "act_chunks": chunks}


# --------------------------------------------------------------------------
# Models
# --------------------------------------------------------------------------

def config(case):
    cfg = dict(V.vla_preset(case["preset"]))
    for k, v in case.items():
        if k.startswith("set_"):
            cfg[k[4:]] = int(v)
    return cfg


class Model:
    """A model handle, destroyed with its last user (at the process's own end
    the module may be gone first)."""

    def __init__(self, cfg):
        self.cfg = cfg
        self.h = V.vla_create(cfg, MODEL_SEED)

    def __del__(self):
        if getattr(self, "h", None) and V is not None and V.vla_destroy is not None:
            V.vla_destroy(self.h)
            self.h = None


class Context:
    def __init__(self, model):
        self.model = model  # outlives the context
        self.h = V.vla_ctx_create(model.h)

    def __del__(self):
        if getattr(self, "h", None) and V is not None and V.vla_ctx_destroy is not None:
            V.vla_ctx_destroy(self.h)
            self.h = None


_models = OrderedDict()  # the last few models in use
_models_lock = threading.Lock()


def model(cfg):
    key = tuple(sorted(cfg.items()))
    with _models_lock:
        if key in _models:
            _models.move_to_end(key)
        else:
            _models[key] = Model(cfg)
            while len(_models) > 4:
                _models.popitem(last=False)
        return _models[key]


def sizes(cfg):
    tview = (cfg["img_h"] // cfg["patch"]) * (cfg["img_w"] // cfg["patch"])
    nimg = cfg["n_views"] * tview // cfg["shuffle"] ** 2
    prefix = nimg + cfg["n_text"] + (cfg["state_dim"] > 0) + (cfg["head"] == HEAD_COG)
    return tview, nimg, prefix


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 13)


def frame_inputs(cfg, g, chunks=1):
    """One robot frame: pixels in [-1, 1), instruction ids, state, noise."""
    pix = torch.rand(cfg["n_views"], cfg["img_h"], cfg["img_w"], 3, device=DEV, generator=g) * 2 - 1
    ids = torch.randint(0, cfg["vocab"], (max(cfg["n_text"], 1),), device=DEV, generator=g, dtype=torch.int32)
    state = torch.randn(max(cfg["state_dim"], 1), device=DEV, generator=g)
    noise = torch.randn(chunks, cfg["chunk_len"], cfg["action_dim"], device=DEV, generator=g)
    return pix, ids, state if cfg["state_dim"] > 0 else None, noise


def _op(x, dtype):
    return x.to(torch.bfloat16) if dtype == BF16 else x.float()


def gemm_inputs(case, seed):
    g = _gen(seed)
    A = _op(torch.randn(case["M"], case["K"], device=DEV, generator=g), case["dtype"])
    W = _op(torch.randn(case["N"], case["K"], device=DEV, generator=g) * 0.02, case["dtype"])
    b = torch.randn(case["N"], device=DEV, generator=g) * 0.02 if case["bias"] else None
    return A, W, b


def attention_inputs(case, seed):
    g = _gen(seed)
    nq, nkv, hd = case["nq"], case["nkv"], case["hd"]

    def rows(s, n):
        return _op(torch.randn(s, n, hd, device=DEV, generator=g), case["dtype"])

    q, k0, v0 = rows(case["Sq"], nq), rows(case["S0"], nkv), rows(case["S0"], nkv)
    k1, v1 = (rows(case["S1"], nkv), rows(case["S1"], nkv)) if case["S1"] else (None, None)
    return q, k0, v0, k1, v1


def norm_inputs(case, seed):
    g = _gen(seed)
    x = torch.randn(case["rows"], case["d"], device=DEV, generator=g) * 2 + 0.1
    gain = 1 + 0.02 * torch.randn(case["d"], device=DEV, generator=g)
    shift = None if case["rms"] else 0.02 * torch.randn(case["d"], device=DEV, generator=g)
    return x, gain, shift


def cache_layout(k, v, dtype):
    """K and V rows [S, nkv, hd] in the KV-cache layout (include/vla.h)."""
    S, nkv, hd = k.shape
    vec = 8 if dtype == BF16 else 4
    sw = 4 * vec
    nb, ns, ndt, pvs = (S + 31) // 32, -(-hd // sw), -(-hd // 16), 32 // sw
    p = torch.arange(S, device=DEV).view(S, 1, 1)
    j = torch.arange(nkv, device=DEV).view(1, nkv, 1)
    d = torch.arange(hd, device=DEV).view(1, 1, hd)
    b, kin = p // 32, p % 32
    nt, i = ((kin // 4) % 2, 4 * (kin // 8) + kin % 4) if dtype == BF16 else (kin // 16, kin % 16)
    ki = ((((j * nb + b) * 2 + nt) * ns + d // sw) * 64 + 16 * ((d % sw) // vec) + i) * vec + d % vec
    vi = ((((j * nb + b) * ndt + d // 16) * pvs + kin // sw) * 64 + 16 * ((kin % sw) // vec) + d % 16) * vec + kin % vec
    K = torch.zeros(nkv * nb * 32 * ns * sw, device=DEV, dtype=k.dtype)
    W = torch.zeros(nkv * nb * 32 * ndt * 16, device=DEV, dtype=v.dtype)
    K[ki.reshape(-1)] = k.reshape(-1)
    W[vi.reshape(-1)] = v.reshape(-1)
    return K, W


# --------------------------------------------------------------------------
# prepare / run
# --------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "gemm":
        s["A"], s["W"], s["b"] = gemm_inputs(case, seed)
        s["C"] = torch.empty(case["M"], case["N"], device=DEV)
    elif kind == "attention":
        q, k0, v0, k1, v1 = attention_inputs(case, seed)
        s["q"] = q
        s["k0"], s["v0"] = cache_layout(k0, v0, case["dtype"])
        s["k1"], s["v1"] = cache_layout(k1, v1, case["dtype"]) if case["S1"] else (None, None)
        s["out"] = torch.empty_like(q)
    elif kind == "norm":
        s["x"], s["gain"], s["shift"] = norm_inputs(case, seed)
        s["out"] = _op(torch.empty_like(s["x"]), case["dtype"])
    else:
        cfg = config(case)
        s["m"] = model(cfg)
        g = _gen(seed)
        if kind == "pipeline":
            k = max(1, case["act_chunks"])
            ins = [frame_inputs(cfg, g, k) for _ in range(case["R"])]
            s["frames"] = [V.make_frame(p, i, st) for p, i, st, _ in ins]
            s["noise"] = torch.cat([n for *_, n in ins])
            s["actions"] = torch.empty_like(s["noise"])
        else:
            p, i, st, n = frame_inputs(cfg, g)
            s["frame"] = V.make_frame(p, i, st)
            s["noise"] = n[0].contiguous()
            s["actions"] = torch.empty_like(s["noise"])
            s["ctx"] = Context(s["m"])
            if kind == "denoise":
                V.vla_vlm_prefill(s["m"].h, s["frame"], s["ctx"].h, torch.cuda.current_stream().cuda_stream)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    st = torch.cuda.current_stream().cuda_stream
    if kind == "gemm":
        V.vla_gemm_noalloc(c["dtype"], c["M"], c["N"], c["K"], s["A"], c["K"], s["W"], c["K"], s["b"], s["C"], st)
        return s["C"]
    if kind == "attention":
        V.vla_debug_attention_cache(c["dtype"], c["Sq"], c["nq"], c["nkv"], c["hd"], s["q"], s["k0"], s["v0"],
                                    c["S0"], s["k1"], s["v1"], c["S1"], s["out"], st)
        return s["out"]
    if kind == "norm":
        V.vla_debug_norm(c["dtype"], c["rows"], c["d"], s["x"], c["d"], None, 0, None, None, s["gain"], 0,
                         s["shift"], int(c["rms"]), s["out"], c["d"], st)
        return s["out"]
    m = s["m"].h
    if kind == "pipeline":
        V.vla_pipeline_run(m, s["frames"], s["noise"], c["R"], mode=c["mode"], actions=s["actions"],
                           act_streams=c["act_streams"], graphs=c["graphs"], act_batch=c["act_batch"],
                           vlm_batch=c["vlm_batch"], act_chunks=c["act_chunks"])
        return s["actions"]
    if kind == "frame":
        V.vla_vlm_prefill(m, s["frame"], s["ctx"].h, st)
    V.vla_action_denoise(m, s["ctx"].h, s["noise"], s["actions"], st)
    return s["actions"]


# --------------------------------------------------------------------------
# Work and tolerances
# --------------------------------------------------------------------------

def _vlm_work(cfg, frames):
    """(weight bytes, flops) of one prefill of `frames` frames."""
    tv, nimg, P = sizes(cfg)
    es = 2 if cfg["dtype"] == BF16 else 4
    dv, dl, F = cfg["vit_dim"], cfg["lm_dim"], cfg["lm_mlp"]
    hd, nq, nkv = cfg["head_dim"], cfg["lm_heads"], cfg["lm_kv_heads"]
    rows = cfg["n_views"] * tv
    vit = cfg["vit_layers"] * (4 * dv * dv + 2 * dv * cfg["vit_mlp"]) + 3 * cfg["patch"] ** 2 * dv
    proj = dl * dv * cfg["shuffle"] ** 2
    qkv, rest = dl * (nq + 2 * nkv) * hd, nq * hd * dl + 3 * dl * F
    full = cfg["lm_layers"] - (cfg["head"] == HEAD_PI0)  # the last layer's output is not used
    lm = cfg["lm_layers"] * qkv + full * rest
    flops = 2 * (rows * vit + nimg * proj + P * lm)
    flops += 4 * (cfg["vit_layers"] * rows * tv * dv + full * P * P * nq * hd)
    wts = vit + proj + lm
    if cfg["head"] == HEAD_DIT:
        cross = (cfg["ex_layers"] + 1) // 2 * 2 * cfg["ex_dim"] * dl
        wts += cross
        flops += 2 * P * cross
    return wts * es, flops * frames


def _act_work(cfg, frames):
    """(weight bytes of one step, flops of the loop) of `frames` chunks."""
    _, _, P = sizes(cfg)
    es = 2 if cfg["dtype"] == BF16 else 4
    de, F, L = cfg["ex_dim"], cfg["ex_mlp"], cfg["ex_layers"]
    H = cfg["chunk_len"]
    if cfg["head"] == HEAD_PI0:
        qd, kvd = cfg["lm_heads"] * cfg["head_dim"], cfg["lm_kv_heads"] * cfg["head_dim"]
        w = L * (de * (qd + 2 * kvd) + qd * de + 3 * de * F) + 2 * de * de
        att = L * 4 * H * (P + H) * qd
    elif cfg["head"] == HEAD_DIT:
        even = (L + 1) // 2
        w = L * (2 * de * de + 2 * de * F) + (L - even) * 2 * de * de
        att = 4 * H * de * (even * P + (L - even) * H)
    else:
        H += 2
        w = L * (4 * de * de + 2 * de * F)
        att = L * 4 * H * H * de
    w += 2 * de * cfg["action_dim"]
    return w * es, cfg["n_steps"] * frames * (2 * H * w + att)


def work(case):
    kind = case["kind"]
    es = 2 if case.get("dtype", BF16) == BF16 else 4
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": es * (M * K + N * K) + 4 * M * N, "flops": 2 * M * N * K}
    if kind == "attention":
        S, w = case["S0"] + case["S1"], case["nq"] * case["hd"]
        return {"bytes": es * (2 * case["Sq"] * w + 2 * S * case["nkv"] * case["hd"]),
                "flops": 4 * case["Sq"] * S * w}
    if kind == "norm":
        return {"bytes": case["rows"] * case["d"] * (4 + es), "flops": 5 * case["rows"] * case["d"]}
    # Models: a prefill reads its weights once for the frames it stacks; a
    # loop reads the head's weights once per step (they exceed what the chip
    # keeps between steps, except in the tiny models)
    cfg = config(case)
    R = case.get("R", 1)
    vb, ab = max(1, case.get("vlm_batch", 1)), max(1, case.get("act_batch", 1))
    items = R * max(1, case.get("act_chunks", 1))
    bytes_, flops = 0, 0
    if kind != "denoise":
        wb, fl = _vlm_work(cfg, R)
        bytes_ += wb * -(-R // vb) + R * 12 * cfg["n_views"] * cfg["img_h"] * cfg["img_w"]
        flops += fl
    wb, fl = _act_work(cfg, items)
    steps = cfg["n_steps"] if wb > (64 << 20) else 1
    bytes_ += wb * steps * -(-items // ab) + 8 * items * cfg["chunk_len"] * cfg["action_dim"]
    flops += fl
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "gemm":  # exact products, fp32 sums
        return {"rel": 5e-6, "max": 1e-4}
    if kind == "attention":  # bf16: one rounding of the output, P in 16 bits
        return {"rel": 4e-3, "max": 2e-2} if case["dtype"] == BF16 else {"rel": 5e-6, "max": 1e-4}
    if kind == "norm":  # bf16: an output near a rounding boundary goes either way
        return {"rel": 1e-3, "max": 1e-2} if case["dtype"] == BF16 else {"rel": 5e-6, "max": 1e-4}
    cfg = config(case)
    if cfg["dtype"] == F32:
        return {"rel": 5e-6, "max": 5e-5}  # chunks measured 0.6 to 1.3e-7 off 64 bits
    # a flipped bf16 rounding travels through every later layer and step
    # (chunks measured 0.2 to 1.8e-3 off 64 bits, single values 5.7e-3)
    return {"rel": 7e-3, "max": 3e-2}


# --------------------------------------------------------------------------
# 64-bit values
# --------------------------------------------------------------------------

F64 = torch.float64


def _layer_norm(x, g, b):
    mu = x.mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt(((x - mu) ** 2).mean(-1, keepdim=True) + 1e-6) * g + b


def _rms(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6) * g


def _gelu(x):
    return 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3)))


def _swish(x):
    return x / (1 + torch.exp(-x))


def _attend(q, k, v):
    """q [.., Sq, nq, hd] over k, v [.., S, nkv, hd]."""
    rep = q.shape[-2] // k.shape[-2]
    k, v = (t.repeat_interleave(rep, dim=-2).transpose(-2, -3).contiguous() for t in (k, v))
    s = q.transpose(-2, -3).contiguous() @ k.transpose(-1, -2).contiguous() / math.sqrt(q.shape[-1])
    return (torch.softmax(s, -1) @ v).transpose(-2, -3).flatten(-2)


def _rope(x, pos):
    half = x.shape[-1] // 2
    inv = 10000.0 ** (-torch.arange(half, device=DEV, dtype=F64) / half)
    a = (pos[:, None].to(F64) * inv)[:, None]
    c, s = torch.cos(a), torch.sin(a)
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _phi(t, dim):
    half = dim // 2
    frac = torch.arange(half, device=DEV, dtype=F64) / max(half - 1, 1)
    x = 2 * math.pi * t / (4e-3 * 1000.0 ** frac)
    return torch.cat([torch.sin(x), torch.cos(x)])[None]


class _Params:
    """A model's parameters in 64 bits, as they are stored, fetched when used."""

    def __init__(self, m):
        self.m, self.n = m, {}
        for i in range(V.vla_param_count(m.h)):
            name, numel = V.vla_param_info(m.h, i)
            self.n[name] = numel
        self.kept = {}

    def vec(self, name):
        if name not in self.kept:
            self.kept[name] = torch.from_numpy(V.vla_export_param(self.m.h, name, self.n[name])).to(DEV)
        return self.kept[name].to(F64)

    def lin(self, x, name, bias=True):
        w = self.vec(name + ".w").view(-1, x.shape[-1])
        y = x @ w.t()
        return y + self.vec(name + ".b") if bias else y


def _decoder(p, cfg, pre, x, pos, past=None, kv_only=False):
    hd = cfg["head_dim"]
    h = _rms(x, p.vec(pre + "rms1.g"))
    q, k, v = (p.lin(h, pre + n, False).unflatten(-1, (-1, hd)) for n in "qkv")
    q, k = _rope(q, pos), _rope(k, pos)
    if kv_only:
        return x, k, v
    ka, va = (k, v) if past is None else (torch.cat([past[0], k], -3), torch.cat([past[1], v], -3))
    x = x + p.lin(_attend(q, ka, va), pre + "o", False)
    h = _rms(x, p.vec(pre + "rms2.g"))
    f = _gelu(p.lin(h, pre + "gate", False)) * p.lin(h, pre + "up", False)
    return x + p.lin(f, pre + "down", False), k, v


def _exact_prefill(p, cfg, pix, ids, state):
    """Frames stacked on the first axis -> the hand-off."""
    n, nv, H, W, _ = pix.shape
    pt, dv = cfg["patch"], cfg["vit_dim"]
    gh, gw = H // pt, W // pt
    x = pix.to(F64).view(n * nv, gh, pt, gw, pt, 3).permute(0, 1, 3, 2, 4, 5).reshape(n * nv, gh * gw, -1)
    x = p.lin(x, "vit.patch") + p.vec("vit.pos").view(gh * gw, dv)
    for l in range(cfg["vit_layers"]):
        b = "vit.%d." % l
        h = _layer_norm(x, p.vec(b + "ln1.g"), p.vec(b + "ln1.b"))
        q, k, v = (p.lin(h, b + c).unflatten(-1, (cfg["vit_heads"], -1)) for c in "qkv")
        x = x + p.lin(_attend(q, k, v), b + "o")
        h = _layer_norm(x, p.vec(b + "ln2.g"), p.vec(b + "ln2.b"))
        x = x + p.lin(_gelu(p.lin(h, b + "fc1")), b + "fc2")
    x = _layer_norm(x, p.vec("vit.post.g"), p.vec("vit.post.b"))
    s = cfg["shuffle"]
    x = x.view(n * nv, gh // s, s, gw // s, s, dv).permute(0, 1, 3, 2, 4, 5).reshape(n, -1, s * s * dv)
    dl = cfg["lm_dim"]
    rows = [p.lin(x, "proj")]
    if cfg["n_text"]:
        rows.append(p.vec("lm.embed").view(-1, dl)[ids.long()] * math.sqrt(dl))
    if cfg["state_dim"]:
        rows.append(p.lin(state.to(F64), "state")[:, None])
    if cfg["head"] == HEAD_COG:
        rows.append(p.vec("lm.cog").view(1, 1, dl).expand(n, 1, dl))
    x = torch.cat(rows, 1)
    pos = torch.arange(x.shape[1], device=DEV)
    kv = []
    for l in range(cfg["lm_layers"]):
        x, k, v = _decoder(p, cfg, "lm.%d." % l, x, pos, kv_only=cfg["head"] == HEAD_PI0 and l == cfg["lm_layers"] - 1)
        kv.append((k, v))
    if cfg["head"] == HEAD_PI0:
        return kv
    x = _rms(x, p.vec("lm.final.g"))
    if cfg["head"] == HEAD_COG:
        return p.lin(x[:, -1:], "cog")
    return {l: tuple(p.lin(x, "ex.%d.%s" % (l, c), False).unflatten(-1, (cfg["ex_heads"], -1)) for c in "kv")
            for l in range(0, cfg["ex_layers"], 2)}


def _token_positions(n, dim):
    w = 10000.0 ** (-torch.arange(dim // 2, device=DEV, dtype=F64) / (dim // 2))
    a = torch.arange(n, device=DEV, dtype=F64)[:, None] * w
    return torch.cat([torch.sin(a), torch.cos(a)], 1)


def _head(p, cfg, ho, x, t):
    H, de = x.shape[-2], cfg["ex_dim"]
    if cfg["head"] == HEAD_PI0:
        P = ho[0][0].shape[-3]
        a = p.lin(x, "ex.in")
        u = p.lin(_swish(p.lin(torch.cat([a, _phi(t, de).expand(*a.shape[:-1], de)], -1), "ex.time1")), "ex.time2")
        pos = torch.arange(P, P + H, device=DEV)
        for l in range(cfg["ex_layers"]):
            u, _, _ = _decoder(p, cfg, "ex.%d." % l, u, pos, past=ho[l])
        return p.lin(_rms(u, p.vec("ex.final.g")), "ex.out")
    nh = cfg["ex_heads"]
    tok = p.lin(_swish(p.lin(_phi(t, 256), "ex.time1")), "ex.time2")
    x = p.lin(x, "ex.in") + _token_positions(H, de)
    if cfg["head"] == HEAD_COG:
        x = torch.cat([x, ho, tok.expand(x.shape[0], 1, de)], 1)
        for l in range(cfg["ex_layers"]):
            b = "ex.%d." % l
            h = _layer_norm(x, p.vec(b + "ln1.g"), p.vec(b + "ln1.b"))
            q, k, v = (p.lin(h, b + c, False).unflatten(-1, (nh, -1)) for c in "qkv")
            x = x + p.lin(_attend(q, k, v), b + "o", False)
            h = _layer_norm(x, p.vec(b + "ln2.g"), p.vec(b + "ln2.b"))
            x = x + p.lin(_gelu(p.lin(h, b + "fc1", False)), b + "fc2", False)
        return p.lin(_layer_norm(x[:, :H], p.vec("ex.final.g"), p.vec("ex.final.b")), "ex.out")
    c = _swish(tok)
    for l in range(cfg["ex_layers"]):
        b = "ex.%d." % l
        sh1, sc1, g1, sh2, sc2, g2 = p.lin(c, b + "ada")[0].view(6, de)
        h = _layer_norm(x, 1 + sc1, sh1)
        q = p.lin(h, b + "q", False).unflatten(-1, (nh, -1))
        k, v = ho[l] if l % 2 == 0 else (p.lin(h, b + n, False).unflatten(-1, (nh, -1)) for n in "kv")
        x = x + g1 * p.lin(_attend(q, k, v), b + "o", False)
        h = _layer_norm(x, 1 + sc2, sh2)
        x = x + g2 * p.lin(_gelu(p.lin(h, b + "fc1", False)), b + "fc2", False)
    sh, sc = p.lin(c, "ex.final.ada")[0].view(2, de)
    return p.lin(_layer_norm(x, 1 + sc, sh), "ex.out")


def _sample(p, cfg, ho, noise):
    N, x = cfg["n_steps"], noise.to(F64)
    if cfg["sampler"] == 0:
        dt = float(np.float32(-1) / np.float32(N))
        for k in range(N):
            x = x + dt * _head(p, cfg, ho, x, float(np.float32(N - k) / np.float32(N)))
        return x
    ab = np.cumprod(1 - np.linspace(1e-4, 0.02, 1000))
    s = [(N - k) * 1000 // N - 1 for k in range(N)]
    a = [ab[i] for i in s] + [1.0]
    for k in range(N):
        e = _head(p, cfg, ho, x, float(np.float32(s[k]) / np.float32(1000)))
        x = math.sqrt(a[k + 1]) * (x - math.sqrt(1 - a[k]) * e) / math.sqrt(a[k]) + math.sqrt(1 - a[k + 1]) * e
    return x


_params = OrderedDict()


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        A, W, b = gemm_inputs(case, seed)
        C = A.to(F64) @ W.to(F64).t()
        return C if b is None else C + b.to(F64)
    if kind == "attention":
        q, k0, v0, k1, v1 = (None if t is None else t.to(F64) for t in attention_inputs(case, seed))
        k, v = (k0, v0) if k1 is None else (torch.cat([k0, k1]), torch.cat([v0, v1]))
        return _attend(q, k, v).view(q.shape)
    if kind == "norm":
        x, g, b = (None if t is None else t.to(F64) for t in norm_inputs(case, seed))
        return _rms(x, g) if case["rms"] else _layer_norm(x, g, b)
    cfg = config(case)
    m = model(cfg)
    key = id(m)
    if key not in _params or _params[key].m is not m:
        _params.clear()
        _params[key] = _Params(m)
    p = _params[key]
    g = _gen(seed)
    R, k = case.get("R", 1), max(1, case.get("act_chunks", 1))
    ins = [frame_inputs(cfg, g, k) for _ in range(R)]
    outs = []
    for at in range(0, R, 8):  # a few frames at a time
        part = ins[at:at + 8]
        pix = torch.stack([i[0] for i in part])
        ids = torch.stack([i[1] for i in part])
        state = torch.stack([i[2] for i in part]) if cfg["state_dim"] else None
        noise = torch.stack([i[3] for i in part])
        ho = _exact_prefill(p, cfg, pix, ids, state)
        outs.append(torch.stack([_sample(p, cfg, ho, noise[:, j]) for j in range(k)], 1).flatten(0, 1))
    x = torch.cat(outs)
    return x if kind == "pipeline" else x[0]
