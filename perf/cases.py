"""What this engine is used for, as timed cases: one pass each through its public entry points.

Two levels.  `stage` cases are what a pipeline-parallel training program does with a stage: an op list of F, B and W over a
few microbatches through stage_run_schedule, for stages of one or two layers (the layer is what repeats; depth only
repeats it).  The other kinds are a layer's blocks through the kernel-level entry points of include/stage_kernels.h: `mlp`
(FFN products with their fused activations, input and weight gradients), `attention` (forward and backward), `norm`
(forward and backward) and `linear` (one product).  Shapes are the workloads of paper_2507_00217_amd/synth.py, the reduced
shapes of the tests, or generic ones of the same family; `draw` spreads over the whole range between them.

Gradients accumulate over passes, as they do over the microbatches of an iteration; a new state starts from zero.
"""
import ctypes as C
import math

import torch

from paper_2507_00217_amd import stage as S
from paper_2507_00217_amd import synth

DEV = "cuda:0"
EPS = 1e-5
TORCH_DTYPE = {"fp32": torch.float32, "bf16": torch.bfloat16}


def _stage(name, **kw):
    return dict(dict(name=name, kind="stage", n_layers=1, n_kv_heads=kw["n_heads"], head_dim=kw["hidden"] // kw["n_heads"],
                     mb_size=1, n_mb=2, rope=0, bias=0, recompute=0, schedule="1f1b"), **kw)


def listed():
    return [
        # the fp32 stage on which a user first checks a schedule: small layers, so launches and latency count
        _stage("stage_fp32_small", dtype="fp32", n_layers=2, hidden=256, n_heads=4, ffn=1024, seq=128, n_mb=4,
               norm="layernorm", act="gelu"),
        # a Llama-style stage in fp32, as used to tell arithmetic from storage rounding; ragged sequence
        _stage("stage_fp32_llama", dtype="fp32", hidden=512, n_heads=4, ffn=1408, seq=448, n_mb=2, norm="rmsnorm", act="swiglu"),
        # a small GPT-style bf16 layer, two short ragged sequences per microbatch: few tiles, short kernels
        _stage("stage_gpt_ragged", dtype="bf16", hidden=640, n_heads=5, ffn=1728, seq=200, mb_size=2, n_mb=3, bias=1,
               norm="layernorm", act="gelu"),
        # the GPT-style layer with biases at an ordinary size, W right behind its B
        _stage("stage_gpt_layer", dtype="bf16", hidden=2048, n_heads=16, ffn=8192, seq=2048, bias=1, norm="layernorm", act="gelu"),
        # one GPU's share of a Llama-style layer under 4-way tensor parallelism: grouped queries, rotary embedding, narrow FFN
        _stage("stage_tp_share", dtype="bf16", hidden=4096, n_heads=8, n_kv_heads=2, head_dim=128, ffn=3584, seq=4096, rope=1,
               norm="rmsnorm", act="swiglu"),
        # the full Llama-style layer, both W ops at the end of the list (they merge into one reduction): the largest case
        _stage("stage_llama_layer", dtype="bf16", hidden=4096, n_heads=32, ffn=11008, seq=4096, schedule="w_deferred",
               norm="rmsnorm", act="swiglu"),
        # the FFN block of one microbatch, forward, input gradients and weight gradients, SwiGLU of a tensor-parallel share
        dict(name="mlp_swiglu", kind="mlp", dtype="bf16", act="swiglu", rows=4096, hidden=4096, ffn=3584),
        # the same for a mid-size GELU layer on a ragged token count
        dict(name="mlp_gelu_ragged", kind="mlp", dtype="bf16", act="gelu", rows=1000, hidden=1280, ffn=5120),
        # attention forward and backward at the ordinary training length, grouped queries
        dict(name="attention_gqa", kind="attention", dtype="bf16", b=1, s=4096, h=32, hkv=8, hd=128, causal=1),
        # several short ragged sequences, narrow heads
        dict(name="attention_ragged", kind="attention", dtype="bf16", b=3, s=777, h=12, hkv=12, hd=64, causal=1),
        # a layer norm on its own, forward and backward
        dict(name="norm_layer", kind="norm", dtype="bf16", norm="layernorm", rows=4096, hidden=5120),
        # one input-gradient product with a long reduction
        dict(name="linear_dgrad", kind="linear", dtype="bf16", mode=1, M=4096, N=5120, K=13824),
    ]


def _log_int(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        c = _draw_one(rng)
        if _cost(c) <= limit:
            return c


def _cost(case):
    w = work(case)
    rate = 100e12 if case["dtype"] == "fp32" else 1000e12
    return w["flops"] / rate + w["bytes"] / 5e12


def _draw_one(rng):
    kind = rng.choice(["stage32", "stage16", "stage16", "stage16", "stage16", "mlp", "mlp", "attention", "attention", "norm", "linear"])
    if kind in ("stage32", "stage16"):
        fp32 = kind == "stage32"
        hd = rng.choice([64, 128])
        hidden = _log_int(rng, 256, 1024, 128) if fp32 else _log_int(rng, 512, 4096, 128)
        share = 1 if fp32 else rng.choice([1, 1, 2, 4])          # tensor-parallel degree: fewer heads, narrower FFN
        heads = max(1, hidden // hd // share)
        kv = heads // rng.choice([g for g in (1, 1, 2, 4, 8) if heads % g == 0])
        llama = rng.random() < 0.6
        return dict(kind="stage", dtype="fp32" if fp32 else "bf16", n_layers=1, hidden=hidden, n_heads=heads, n_kv_heads=kv, head_dim=hd,
                    ffn=max(64, int(hidden * rng.uniform(2.0, 4.0) / share) // 64 * 64), seq=_log_int(rng, 100, 700 if fp32 else 4096),
                    mb_size=rng.choice([1, 1, 2]), n_mb=rng.choice([1, 2, 3]), rope=int(llama and rng.random() < 0.6),
                    bias=int(not llama and rng.random() < 0.5), recompute=int(rng.random() < 0.15),
                    schedule=rng.choice(["1f1b", "w_deferred"]), norm="rmsnorm" if llama else "layernorm", act="swiglu" if llama else "gelu")
    if kind == "mlp":
        return dict(kind="mlp", dtype="bf16", act=rng.choice(["gelu", "swiglu"]), rows=_log_int(rng, 200, 8192),
                    hidden=_log_int(rng, 512, 8192, 64), ffn=_log_int(rng, 704, 14336, 64))
    if kind == "attention":
        h = rng.choice([4, 8, 12, 16, 20, 32, 40])
        return dict(kind="attention", dtype="bf16", b=rng.choice([1, 1, 2, 3]), s=_log_int(rng, 128, 8192), h=h,
                    hkv=h // rng.choice([g for g in (1, 1, 4, 8) if h % g == 0]), hd=rng.choice([64, 128, 128]), causal=int(rng.random() < 0.85))
    if kind == "norm":
        return dict(kind="norm", dtype="bf16", norm=rng.choice(["layernorm", "rmsnorm"]), rows=_log_int(rng, 128, 16384),
                    hidden=_log_int(rng, 512, 8192, 64))
    return dict(kind="linear", dtype="bf16", mode=rng.choice([0, 1]), M=_log_int(rng, 200, 8192), N=_log_int(rng, 512, 14336, 64),
                K=_log_int(rng, 512, 14336, 64))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype, mean=0.0, std=1.0):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).mul_(std).add_(mean).to(TORCH_DTYPE[dtype])


def _engine_config(case):
    return dict(n_layers=case["n_layers"], hidden=case["hidden"], n_heads=case["n_heads"], n_kv_heads=case["n_kv_heads"],
                head_dim=case["head_dim"], ffn=case["ffn"], seq=case["seq"], mb_size=case["mb_size"], n_microbatches=case["n_mb"],
                norm=case["norm"], act=case["act"], dtype=case["dtype"], rope_theta=10000.0 if case["rope"] else 0.0, bias=case["bias"],
                recompute=case["recompute"], enforce_mb_order=1)


def _stage_inputs(case, seed):
    """Weights per layer (name -> tensor), boundary activations and gradients, in the compute dtype."""
    g, cfg = _gen(seed), _engine_config(case)
    params = []
    for _ in range(case["n_layers"]):
        params.append({n: _normal(g, synth.param_shape(cfg, n), case["dtype"], 1.0 if n in ("g1", "g2") else 0.0, 0.02)
                       for n in synth.param_names(cfg)})
    shape = (case["n_mb"], case["mb_size"], case["seq"], case["hidden"])
    return params, _normal(g, shape, case["dtype"]), _normal(g, shape, case["dtype"])


class _Buffers:
    """A stage over caller-owned device buffers, as a program on the C interface sets one up."""

    def __init__(self, case, params):
        cfg = _engine_config(case)
        ops = synth.schedule_w_deferred(case["n_mb"], 1, case["n_mb"]) if case["schedule"] == "w_deferred" else synth.schedule_1f1b(case["n_mb"], 1)
        cfg["stash_cap"] = synth.peak_live(ops)
        sizes = S.stage_query_sizes(cfg)
        self.weights, self.grads, self.stash, self.workspace = (
            torch.empty(sizes[n], dtype=torch.uint8, device=DEV) for n in ("weights", "grads", "stash", "workspace"))
        flat, flat_g = self.weights.view(TORCH_DTYPE[case["dtype"]]), self.grads.view(torch.float32)
        self.grad = []
        for li, lp in enumerate(params):
            views = {}
            for name, w in lp.items():
                off, r, c = S.stage_param_layout(cfg, li, name)
                flat[off:off + r * c].copy_(w.reshape(-1))
                views[name] = flat_g[off:off + r * c].view(w.shape)
            self.grad.append(views)
        self.lib, self.n_ops, self.ops = S.lib(), len(ops), S.make_ops(ops)
        self.handle = C.c_void_p()
        rc = self.lib.stage_init(C.byref(S.make_config(cfg)), self.weights.data_ptr(), self.grads.data_ptr(), self.stash.data_ptr(),
                                 self.workspace.data_ptr(), torch.cuda.current_stream().cuda_stream, C.byref(self.handle))
        if rc:
            raise S.StageError(rc, "stage_init")

    def __del__(self):
        if self.handle:
            torch.cuda.synchronize()
            self.lib.stage_destroy(self.handle)
            self.handle = None


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    return state["call"](state)


def _prepare_stage(case, seed):
    params, x, dy = _stage_inputs(case, seed)
    return dict(call=_run_stage, engine=_Buffers(case, params), x=x, dy=dy, y=torch.zeros_like(x), dx=torch.zeros_like(x))


def _run_stage(st):
    e = st["engine"]
    rc = e.lib.stage_run_schedule(e.handle, e.ops, e.n_ops, st["x"].data_ptr(), st["dy"].data_ptr(), st["y"].data_ptr(), st["dx"].data_ptr())
    if rc:
        raise S.StageError(rc, "stage_run_schedule")
    return {"y": st["y"], "dx": st["dx"], "grad": e.grad}


_vp, _i, _i64, _f = C.c_void_p, C.c_int, C.c_int64, C.c_float
_SIGNATURES = {
    "stage_kernel_gemm": [_i, _i, _i, _i, _i, _vp, _i64, _vp, _i64, _vp, _i64, _vp, _i64, _i, _i, _vp],
    "stage_kernel_gemm_act": [_i, _i, _i, _i, _i, _vp, _i64, _vp, _i64, _vp, _i64, _vp, _i64, _i, _vp],
    "stage_kernel_gemm_act_bwd": [_i, _i, _i, _i, _i, _vp, _i64, _vp, _i64, _vp, _i64, _vp, _i, _vp],
    "stage_kernel_wgrad_group": [_i, _i] + [_vp] * 9 + [_i, _vp],
    "stage_kernel_attention_fwd": [_i] * 7 + [_vp, _vp, _vp, _i, _vp],
    "stage_kernel_attention_bwd_ws": [_i] * 7 + [_vp] * 7 + [C.c_size_t, _i, _vp],
    "stage_kernel_norm_fwd": [_i, _i, _i, _i, _f, _vp, _vp, _vp, _vp, _vp, _vp],
    "stage_kernel_norm_bwd": [_i, _i, _i, _i] + [_vp] * 10,
    "stage_kernel_norm_partial_bytes": [_i],
    "stage_kernel_attention_bwd_scratch_bytes": [_i] * 5,
}


def _kernel(name):
    fn = getattr(S.lib(), name)
    fn.argtypes = _SIGNATURES[name]
    fn.restype = C.c_size_t if name.endswith("_bytes") else C.c_int
    return fn


def _call(fn, *args):
    rc = fn(*args)
    if rc:
        raise S.StageError(rc, "kernel entry point")


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _mlp_inputs(case, seed):
    g, dt = _gen(seed), case["dtype"]
    T, d, f = case["rows"], case["hidden"], case["ffn"]
    fin = 2 * f if case["act"] == "swiglu" else f
    # W_in keeps the pre-activation at the unit scale that a normalised input and trained weights give it
    return (_normal(g, (T, d), dt), _normal(g, (d, fin), dt, std=1.0 / math.sqrt(d)), _normal(g, (f, d), dt, std=0.02), _normal(g, (T, d), dt),
            _normal(g, (T, d), dt))


def _prepare_mlp(case, seed):
    x, win, wout, dy, resid = _mlp_inputs(case, seed)
    T, d, f = case["rows"], case["hidden"], case["ffn"]
    fin = win.shape[1]
    empty = lambda *s: torch.empty(s, dtype=x.dtype, device=DEV)
    st = dict(call=_run_mlp, case=case, x=x, win=win, wout=wout, dy=dy, resid=resid, z=empty(T, fin), a=empty(T, f), y=empty(T, d), dx=empty(T, d),
              gin=torch.zeros((d, fin), device=DEV), gout=torch.zeros((f, d), device=DEV))
    ints, longs, ptrs = (lambda *v: (C.c_int * len(v))(*v)), (lambda *v: (C.c_int64 * len(v))(*v)), (lambda *t: (C.c_void_p * len(t))(*[u.data_ptr() for u in t]))
    st["group"] = (ints(d, f), ints(fin, d), ints(T, T), ptrs(x, st["a"]), longs(d, f), ptrs(st["z"], dy), longs(fin, d), ptrs(st["gin"], st["gout"]), longs(fin, d))
    st["fn"] = [_kernel("stage_kernel_" + n) for n in ("gemm_act", "gemm", "gemm_act_bwd", "wgrad_group")]
    return st


def _run_mlp(st):
    c = st["case"]
    T, d, f, fin = c["rows"], c["hidden"], c["ffn"], st["win"].shape[1]
    act, dt, s = S.ACT[c["act"]], S.DTYPE[c["dtype"]], _stream()
    gemm_act, gemm, gemm_act_bwd, wgrad_group = st["fn"]
    x, win, wout, dy, z, a = (st[n].data_ptr() for n in ("x", "win", "wout", "dy", "z", "a"))
    _call(gemm_act, dt, act, T, f, d, x, d, win, fin, z, fin, a, f, 0, s)                                       # z = x.Win, a = act(z)
    _call(gemm, dt, 0, T, d, f, a, f, wout, d, st["y"].data_ptr(), d, st["resid"].data_ptr(), d, 0, 0, s)       # y = a.Wout + residual
    _call(gemm_act_bwd, dt, act, T, f, d, dy, d, wout, d, z, fin, None, 0, s)                                   # z := dz
    _call(gemm, dt, 1, T, d, fin, z, fin, win, fin, st["dx"].data_ptr(), d, None, 0, 0, 0, s)                   # dx = dz.Win^T
    _call(wgrad_group, dt, 2, *st["group"], 0, s)                                                               # both weight gradients
    return {"a": st["a"], "y": st["y"], "dz": st["z"], "dx": st["dx"], "gin": st["gin"], "gout": st["gout"]}


def _attention_inputs(case, seed):
    g = _gen(seed)
    rows, hd = case["b"] * case["s"], case["hd"]
    return (_normal(g, (rows, (case["h"] + 2 * case["hkv"]) * hd), case["dtype"]), _normal(g, (rows, case["h"] * hd), case["dtype"]))


def _prepare_attention(case, seed):
    qkv, do = _attention_inputs(case, seed)
    n = _kernel("stage_kernel_attention_bwd_scratch_bytes")(*(case[k] for k in ("b", "s", "h", "hkv", "hd")))
    stat = lambda: torch.empty((case["b"], case["h"], case["s"]), device=DEV)
    return dict(call=_run_attention, shape=tuple(case[k] for k in ("b", "s", "h", "hkv", "hd", "causal")), dtype=S.DTYPE[case["dtype"]], qkv=qkv, do=do,
                o=torch.empty_like(do), lse=stat(), delta=stat(), dqkv=torch.empty_like(qkv), bytes=n,
                scratch=torch.empty(n, dtype=torch.uint8, device=DEV) if n else None,
                fwd=_kernel("stage_kernel_attention_fwd"), bwd=_kernel("stage_kernel_attention_bwd_ws"))


def _run_attention(st):
    s, p = _stream(), {k: st[k].data_ptr() for k in ("qkv", "do", "o", "lse", "delta", "dqkv")}
    _call(st["fwd"], st["dtype"], *st["shape"], p["qkv"], p["o"], p["lse"], 0, s)
    _call(st["bwd"], st["dtype"], *st["shape"], p["qkv"], p["o"], p["lse"], p["do"], p["dqkv"], p["delta"],
          st["scratch"].data_ptr() if st["bytes"] else None, st["bytes"], 0, s)
    return {"o": st["o"], "lse": st["lse"], "dqkv": st["dqkv"]}


def _norm_inputs(case, seed):
    g, dt = _gen(seed), case["dtype"]
    shape, d = (case["rows"], case["hidden"]), (case["hidden"],)
    return (_normal(g, shape, dt, 0.1, 1.5), _normal(g, d, dt, 1.0, 0.02), _normal(g, d, dt, 0.0, 0.02), _normal(g, shape, dt), _normal(g, shape, dt))


def _prepare_norm(case, seed):
    x, gamma, beta, dout, resid = _norm_inputs(case, seed)
    d = case["hidden"]
    grad = lambda: torch.zeros(d, device=DEV)
    return dict(call=_run_norm, head=(S.DTYPE[case["dtype"]], S.NORM[case["norm"]], case["rows"], d), x=x, gamma=gamma, beta=beta, dout=dout, resid=resid,
                out=torch.empty_like(x), dx=torch.empty_like(x), stats=torch.empty((case["rows"], 2), device=DEV), dgamma=grad(), dbeta=grad(),
                partial=torch.empty(_kernel("stage_kernel_norm_partial_bytes")(d), dtype=torch.uint8, device=DEV),
                fwd=_kernel("stage_kernel_norm_fwd"), bwd=_kernel("stage_kernel_norm_bwd"))


def _run_norm(st):
    s, p = _stream(), {k: v.data_ptr() for k, v in st.items() if isinstance(v, torch.Tensor)}
    _call(st["fwd"], *st["head"], EPS, p["x"], p["gamma"], p["beta"], p["out"], p["stats"], s)
    _call(st["bwd"], *st["head"], p["x"], p["stats"], p["gamma"], p["dout"], p["resid"], p["dx"], p["dgamma"], p["dbeta"], p["partial"], s)
    return {"out": st["out"], "stats": st["stats"], "dx": st["dx"], "dgamma": st["dgamma"], "dbeta": st["dbeta"]}


def _linear_inputs(case, seed):
    g, M, N, K = _gen(seed), case["M"], case["N"], case["K"]
    return _normal(g, (M, K), case["dtype"]), _normal(g, (N, K) if case["mode"] == 1 else (K, N), case["dtype"], std=0.02)


def _prepare_linear(case, seed):
    a, b = _linear_inputs(case, seed)
    return dict(call=_run_linear, case=case, a=a, b=b, c=torch.empty((case["M"], case["N"]), dtype=a.dtype, device=DEV), fn=_kernel("stage_kernel_gemm"))


def _run_linear(st):
    c = st["case"]
    _call(st["fn"], S.DTYPE[c["dtype"]], c["mode"], c["M"], c["N"], c["K"], st["a"].data_ptr(), c["K"], st["b"].data_ptr(), st["b"].shape[1],
          st["c"].data_ptr(), c["N"], None, 0, 0, 0, _stream())
    return st["c"]


_PREPARE = {"stage": _prepare_stage, "mlp": _prepare_mlp, "attention": _prepare_attention, "norm": _prepare_norm, "linear": _prepare_linear}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    es = 4 if case["dtype"] == "fp32" else 2
    k = case["kind"]
    if k == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": es * (M * K + K * N + M * N), "flops": 2.0 * M * N * K}
    if k == "norm":      # forward: x in, out; backward: x, dout, residual in, dx out
        n = case["rows"] * case["hidden"]
        return {"bytes": es * 6 * n, "flops": 20.0 * n}
    if k == "attention":
        b, s, h, hkv, hd = (case[x] for x in ("b", "s", "h", "hkv", "hd"))
        rows, fwd = b * s, (2.0 if case["causal"] else 4.0) * b * s * s * h * hd
        return {"bytes": es * rows * hd * (3 * (h + 2 * hkv) + 4 * h), "flops": 3.5 * fwd}
    if k == "mlp":
        T, d, f = case["rows"], case["hidden"], case["ffn"]
        fin = 2 * f if case["act"] == "swiglu" else f
        return {"bytes": es * (T * (5 * d + fin + f) + 2 * (d * fin + f * d)) + 8 * (d * fin + f * d), "flops": 6.0 * T * d * (fin + f)}
    # stage: F and B read the weights, W reads and writes the fp32 gradients; a microbatch's boundary tensors travel once
    # each and its stash (what F leaves for B and W) is written and read once
    d, f, s, b = case["hidden"], case["ffn"], case["seq"], case["mb_size"]
    fin = 2 * f if case["act"] == "swiglu" else f
    da, dkv, T = case["n_heads"] * case["head_dim"], case["n_kv_heads"] * case["head_dim"], s * b
    params = d * (da + 2 * dkv) + da * d + d * fin + f * d
    attn = 2.0 * b * s * s * da
    stash = T * (4 * d + 2 * (da + 2 * dkv) + da + fin + f)
    n = case["n_layers"]
    return {"bytes": n * (case["n_mb"] * es * (4 * T * d / n + 2 * params + 2 * stash) + 8 * params),
            "flops": n * case["n_mb"] * (6.0 * T * params + 3.5 * attn)}


# Measured against `exact` on the listed cases and a few drawn ones; stated at about four times the largest seen.
# bf16: one rounding of an output is 1.7e-3 of it in the 2-norm, the rest are the roundings of tensors between kernels.
def tolerance(case):
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    return {"rel": {"stage": 3.5e-2, "mlp": 1.2e-2, "attention": 1e-2, "norm": 7e-3, "linear": 7e-3}[case["kind"]]}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _act64(act, z):
    if act == "gelu":
        return 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))
    gate, up = z.chunk(2, dim=-1)
    return gate * torch.sigmoid(gate) * up


def _norm64(norm, x, gamma, beta):
    mean = x.mean(-1, keepdim=True) if norm == "layernorm" else torch.zeros_like(x[:, :1])
    rstd = ((x - mean) ** 2).mean(-1, keepdim=True).add(EPS).rsqrt()
    y = (x - mean) * rstd * gamma
    return (y + beta if norm == "layernorm" else y), mean, rstd


def _rope64(x, hd, theta):
    """x: [s, heads * hd] of one sequence; pairs (2p, 2p+1) turn by position * theta^(-2p/hd)."""
    s = x.shape[0]
    p = torch.arange(hd // 2, device=DEV, dtype=torch.float64)
    ang = torch.arange(s, device=DEV, dtype=torch.float64)[:, None] * theta ** (-2.0 * p / hd)[None, :]
    cos, sin = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    v = x.view(s, -1, hd // 2, 2)
    a, b = v[..., 0], v[..., 1]
    return torch.stack((a * cos - b * sin, a * sin + b * cos), dim=-1).reshape(s, -1)


def _attend64(q, k, v, causal):
    """One head of one sequence."""
    sc = (q @ k.t()) / math.sqrt(q.shape[1])
    if causal:
        sc = sc.masked_fill(torch.ones_like(sc, dtype=torch.bool).triu(1), -math.inf)
    lse = torch.logsumexp(sc, -1)
    return torch.exp(sc - lse[:, None]) @ v, lse


def _heads64(qkv, h, hkv, hd, causal):
    """One sequence: [s, (h + 2 hkv) hd] -> [s, h hd] and lse [h, s]."""
    q, k, v = qkv.split([h * hd, hkv * hd, hkv * hd], dim=1)
    col = lambda t, j: t[:, j * hd:(j + 1) * hd]
    out = [_attend64(col(q, j), col(k, j // (h // hkv)), col(v, j // (h // hkv)), causal) for j in range(h)]
    return torch.cat([o for o, _ in out], 1), torch.stack([l for _, l in out])


def exact(case, seed):
    return _EXACT[case["kind"]](case, seed)


def _exact_stage(case, seed):
    params, X, dY = _stage_inputs(case, seed)
    P = [{n: w.double().requires_grad_() for n, w in lp.items()} for lp in params]
    h, hkv, hd, s = case["n_heads"], case["n_kv_heads"], case["head_dim"], case["seq"]
    qk = (h + hkv) * hd
    ys, dxs = [], []
    for m in range(case["n_mb"]):
        x0 = X[m].reshape(-1, case["hidden"]).double().requires_grad_()
        x = x0
        for p in P:
            lin = lambda t, w, b: t @ p[w] + p[b] if case["bias"] else t @ p[w]
            qkv = lin(_norm64(case["norm"], x, p["g1"], p.get("b1"))[0], "wqkv", "bqkv")
            o = []
            for seq in qkv.split(s, 0):
                if case["rope"]:
                    seq = torch.cat((_rope64(seq[:, :qk], hd, 10000.0), seq[:, qk:]), 1)
                o.append(_heads64(seq, h, hkv, hd, True)[0])
            x1 = x + lin(torch.cat(o, 0), "wo", "bo")
            a = _act64(case["act"], lin(_norm64(case["norm"], x1, p["g2"], p.get("b2"))[0], "win", "bin"))
            x = x1 + lin(a, "wout", "bout")
        x.backward(dY[m].reshape(x.shape).double())
        ys.append(x.detach())
        dxs.append(x0.grad)
    return {"y": torch.stack(ys).view(X.shape), "dx": torch.stack(dxs).view(X.shape), "grad": [{n: w.grad for n, w in p.items()} for p in P]}


def _exact_mlp(case, seed):
    x, win, wout, dy, resid = (t.double() for t in _mlp_inputs(case, seed))
    z = (x @ win).requires_grad_()
    a = _act64(case["act"], z)
    a.backward(dy @ wout.t())
    a = a.detach()
    return {"a": a, "y": a @ wout + resid, "dz": z.grad, "dx": z.grad @ win.t(), "gin": x.t() @ z.grad, "gout": a.t() @ dy}


def _exact_attention(case, seed):
    qkv, do = (t.double() for t in _attention_inputs(case, seed))
    qkv.requires_grad_()
    o, lse = zip(*(_heads64(t, case["h"], case["hkv"], case["hd"], case["causal"]) for t in qkv.split(case["s"], 0)))
    o, lse = torch.cat(o, 0), torch.stack(lse)
    o.backward(do)
    return {"o": o.detach(), "lse": lse.detach(), "dqkv": qkv.grad}


def _exact_norm(case, seed):
    x, gamma, beta, dout, resid = (t.double() for t in _norm_inputs(case, seed))
    for t in (x, gamma, beta):
        t.requires_grad_()
    out, mean, rstd = _norm64(case["norm"], x, gamma, beta)
    out.backward(dout)
    return {"out": out.detach(), "stats": torch.cat((mean, rstd), 1).detach(), "dx": x.grad + resid, "dgamma": gamma.grad,
            "dbeta": beta.grad if beta.grad is not None else torch.zeros_like(gamma)}


def _exact_linear(case, seed):
    a, b = (t.double() for t in _linear_inputs(case, seed))
    return a @ (b.t() if case["mode"] == 1 else b)


_EXACT = {"stage": _exact_stage, "mlp": _exact_mlp, "attention": _exact_attention, "norm": _exact_norm, "linear": _exact_linear}
