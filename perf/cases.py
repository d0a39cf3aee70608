"""The work a user has this library do, as cases that can be timed.

A case is one call (or one step) through the public entry points of
paper_2403_01164_amd: a single linear, a linear on tile-ordered weights, a decode step
over a stack of decoder layers, the same step over a KV cache, a step whose weights are
split between host and GPU, and filling the KV cache from a prompt.  The sizes are those
of the OPT shapes the library's tests and benchmark use, and odd ones between them.

Inputs follow the library's recipe: weights and biases N(0, 0.02), activations N(0, 1),
keys and values of a cache N(0, 1).  The layers of one model share the host copy of their
weights (one layer's worth, to keep preparation short); every layer has its own copy in
device memory.
"""
import atexit
import math
import weakref

import torch

import paper_2403_01164_amd as hg

DTYPE = {"f16": (hg.F16, torch.float16), "bf16": (hg.BF16, torch.bfloat16), "f32": (hg.F32, torch.float32)}
LN_EPS = 1e-5

_context = None
_open = weakref.WeakSet()


def _ctx():
    """One context per process, as a serving program keeps it."""
    global _context
    if _context is None:
        _context = hg.hetegen_create(0)
    return _context


@atexit.register
def _close():
    global _context
    for s in list(_open):
        s.close()
    if _context is not None:
        hg.hetegen_destroy(_context)
        _context = None


class State:
    """What a program holds between calls; a model is freed with its state."""

    def __init__(self):
        self.model = None
        _open.add(self)

    def close(self):
        if self.model is not None and _context is not None:
            torch.cuda.synchronize()
            hg.hetegen_model_destroy(_context, self.model)
        self.model = None

    def __del__(self):
        self.close()


def listed():
    return [
        # one small resident linear at batch 1: a call whose latency counts, not its bytes
        dict(name="linear_b1", kind="linear", B=1, N=4096, K=1024, dtype="f16", out="f16"),
        # a resident linear at an odd batch and ragged sizes, binary32 output
        dict(name="linear_b5_ragged", kind="linear", B=5, N=10007, K=5128, dtype="bf16", out="f32"),
        # the FFN up-projection of OPT-6.7B for a batch of eight, weights as the user stored them
        dict(name="linear_b8", kind="linear", B=8, N=16384, K=4096, dtype="f16", out="f16"),
        # OPT-13B's FFN down-projection on tile-ordered weights
        dict(name="tiled_b4", kind="tiled", B=4, N=5120, K=20480, dtype="bf16", out="bf16"),
        # decode of one token at a time, all weights resident: OPT-6.7B shapes (the headline workload)
        dict(name="step_b1", kind="step", B=1, L=4, H=4096, F=16384, dtype="f16"),
        # the same layers decoding eight sequences together
        dict(name="step_b8", kind="step", B=8, L=4, H=4096, F=16384, dtype="f16"),
        # a small model (OPT-350M's hidden size), two sequences: short linears, many launches
        dict(name="step_b2_small", kind="step", B=2, L=24, H=1024, F=4096, dtype="bf16"),
        # one layer of the largest shapes in the benchmark (OPT-66B), eight sequences
        dict(name="step_b8_large", kind="step", B=8, L=1, H=9216, F=36864, dtype="bf16"),
        # OPT-13B shapes, half of the linears in pinned host memory: rows split between the host
        # cores and the link, as the planner places them on a machine with a fast host
        dict(name="step_hetero_b1", kind="hetero", B=1, L=1, H=5120, F=20480, dtype="f16", alpha=0.875),
        # a full decode step with attention over a 512-token context, one sequence
        dict(name="kv_step_b1", kind="kv_step", B=1, L=4, H=4096, F=16384, dtype="f16", D=128, ctx=512),
        # eight sequences of 2048 tokens, OPT-13B shapes
        dict(name="kv_step_b8_long", kind="kv_step", B=8, L=2, H=5120, F=20480, dtype="bf16", D=128, ctx=2048),
        # a prompt's keys and values into one layer's cache and back out (a session swapped in and out)
        dict(name="kv_fill_b8", kind="kv_fill", B=8, L=1, H=4096, F=512, dtype="f16", D=128, ctx=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "tiled", "step", "step", "kv_step", "kv_step", "kv_fill", "hetero"])
    B = rng.randint(1, 8)
    dtype = rng.choice(["f16", "bf16"])
    if kind in ("linear", "tiled"):
        K = 8 * _log(rng, 32, 4608)
        N = min(_log(rng, 256, 40000), 300_000_000 // K)
        return dict(kind=kind, B=B, N=N, K=K, dtype=dtype, out=rng.choice([dtype, "f32"]))
    if kind == "kv_fill":
        D = rng.choice([64, 128])
        H = D * max(1, _log(rng, 512, 9216) // D)
        return dict(kind=kind, B=B, L=1, H=H, F=512, dtype=dtype, D=D, ctx=_log(rng, 16, 1024))
    if kind == "hetero":
        H = 8 * _log(rng, 64, 640)
        return dict(kind=kind, B=B, L=1, H=H, F=4 * H, dtype=dtype, alpha=rng.choice([0.75, 0.875, 0.95]))
    if kind == "step":
        H = 8 * _log(rng, 64, 1152)
        F = rng.choice([4 * H, 4 * H, 8 * _log(rng, H // 4, H // 2)])
        L = max(1, min(12, 500_000_000 // (4 * H * H + 2 * H * F)))
        return dict(kind=kind, B=B, L=L, H=H, F=F, dtype=dtype)
    D = rng.choice([64, 128])
    H = D * max(1, _log(rng, 512, 7168) // D)
    L = max(1, min(6, 400_000_000 // (12 * H * H)))
    return dict(kind=kind, B=B, L=L, H=H, F=4 * H, dtype=dtype, D=D, ctx=_log(rng, 1, 4096))


def _shapes(c):
    H, F = c["H"], c["F"]
    return [(3 * H, H), (H, H), (F, H), (H, F)]  # qkv, out, fc1, fc2


def _normal(g, shape, dt, std=1.0):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dt)


def _inputs(c, seed):
    """The case's tensors on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = DTYPE[c["dtype"]][1]
    if c["kind"] in ("linear", "tiled"):
        return dict(x=_normal(g, (c["B"], c["K"]), dt), W=_normal(g, (c["N"], c["K"]), dt, 0.02),
                    b=_normal(g, (c["N"],), dt, 0.02))
    t = dict(x=_normal(g, (c["B"], c["H"]), dt))
    t["W"] = [_normal(g, s, dt, 0.02) for s in _shapes(c)]
    t["b"] = [_normal(g, (s[0],), dt, 0.02) for s in _shapes(c)]
    if c["kind"] in ("kv_step", "kv_fill"):
        shape = (c["L"], c["B"], c["ctx"], c["H"])
        t["k"], t["v"] = _normal(g, shape, dt), _normal(g, shape, dt)
    return t


def _pinned(t):
    h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    h.copy_(t)
    return h


def prepare(case, seed):
    c, s = case, State()
    s.case, s.ctx = c, _ctx()
    t = _inputs(c, seed)
    code, dt = DTYPE[c["dtype"]]
    s.code = code
    stream = torch.cuda.current_stream().cuda_stream
    if c["kind"] in ("linear", "tiled"):
        s.x, s.b = t["x"], t["b"]
        s.y = torch.empty((c["B"], c["N"]), dtype=DTYPE[c["out"]][1], device="cuda")
        if c["kind"] == "linear":
            s.W = t["W"]
            s.W_host, s.b_host = _pinned(t["W"]), _pinned(t["b"])
        else:
            s.W = torch.empty(hg.hetegen_tiled_bytes(c["N"], c["K"]) // 2, dtype=torch.int16, device="cuda")
            hg.hetegen_tile_weights(s.ctx, t["W"].data_ptr(), c["N"], c["K"], s.W.data_ptr(), stream)
            torch.cuda.synchronize()
        return s
    s.x = t["x"]
    s.W_host, s.b_host = [_pinned(w) for w in t["W"]], [_pinned(b) for b in t["b"]]
    del t["W"], t["b"]
    L = c["L"]
    # hetero: attention linears in HBM, FFN linears in host memory split by alpha
    alpha = [0.0, 0.0, c["alpha"], c["alpha"]] * L if c["kind"] == "hetero" else [0.0] * (4 * L)
    resident = [1, 1, 0, 0] * L if c["kind"] == "hetero" else [1] * (4 * L)
    s.model = hg.hetegen_model_create(s.ctx, L, c["H"], c["F"], code, [w.data_ptr() for w in s.W_host] * L,
                                      [b.data_ptr() for b in s.b_host] * L, alpha, resident, c["B"])
    s.y = torch.empty((c["B"], c["H"]), dtype=dt, device="cuda")
    if c["kind"] == "kv_step":
        hg.hetegen_model_kv_create(s.ctx, s.model, c["ctx"] + 1, c["D"])
        for l in range(L):
            hg.hetegen_model_kv_write(s.ctx, s.model, l, c["B"], 0, c["ctx"], t["k"][l].data_ptr(),
                                      t["v"][l].data_ptr(), stream)
        torch.cuda.synchronize()
    elif c["kind"] == "kv_fill":
        hg.hetegen_model_kv_create(s.ctx, s.model, c["ctx"] + 128, c["D"])
        s.k, s.v = t["k"], t["v"]
        s.k_out, s.v_out = torch.empty_like(s.k), torch.empty_like(s.v)
    return s


def run(s):
    c = s.case
    stream = torch.cuda.current_stream().cuda_stream
    if c["kind"] == "linear":
        hg.hetegen_linear(s.ctx, s.x.data_ptr(), c["B"], c["K"], s.W_host.data_ptr(), s.W.data_ptr(), c["N"], s.code,
                          s.b_host.data_ptr(), s.b.data_ptr(), 0.0, s.y.data_ptr(), DTYPE[c["out"]][0], stream)
    elif c["kind"] == "tiled":
        hg.hetegen_linear_tiled(s.ctx, s.x.data_ptr(), c["B"], c["K"], s.W.data_ptr(), c["N"], s.code, s.b.data_ptr(),
                                s.y.data_ptr(), DTYPE[c["out"]][0], stream)
    elif c["kind"] in ("step", "hetero"):
        hg.hetegen_decode_step(s.ctx, s.model, s.x.data_ptr(), s.y.data_ptr(), c["B"], stream)
    elif c["kind"] == "kv_step":
        hg.hetegen_decode_step_kv(s.ctx, s.model, s.x.data_ptr(), s.y.data_ptr(), c["B"], c["ctx"], stream)
    else:
        for l in range(c["L"]):
            hg.hetegen_model_kv_write(s.ctx, s.model, l, c["B"], 0, c["ctx"], s.k[l].data_ptr(), s.v[l].data_ptr(),
                                      stream)
            hg.hetegen_model_kv_read(s.ctx, s.model, l, c["B"], 0, c["ctx"], s.k_out[l].data_ptr(),
                                     s.v_out[l].data_ptr(), stream)
        return s.k_out, s.v_out
    return s.y


def work(case):
    c = case
    B = c["B"]
    if c["kind"] in ("linear", "tiled"):
        N, K = c["N"], c["K"]
        ys = 4 if c["out"] == "f32" else 2
        return {"bytes": 2 * (N * K + N + B * K) + ys * B * N, "flops": 2 * B * N * K}
    H, L = c["H"], c["L"]
    if c["kind"] == "kv_fill":  # the prompt's rows read and the cache written, then the reverse
        return {"bytes": 4 * (2 * L * B * c["ctx"] * H * 2), "flops": 0}
    params = sum(n * k for n, k in _shapes(c))
    w = {"bytes": 2 * (L * (params + sum(n for n, _ in _shapes(c))) + 2 * B * H), "flops": 2 * B * L * params}
    if c["kind"] == "kv_step":
        w["bytes"] += 2 * 2 * L * B * (c["ctx"] + 1) * H
        w["flops"] += 4 * L * B * (c["ctx"] + 1) * H
    return w


def tolerance(case):
    c = case
    if c["kind"] == "kv_fill":
        return "exact"
    if c["kind"] in ("linear", "tiled"):
        return {"rel": {"f32": 1e-5, "f16": 1e-3, "bf16": 8e-3}[c["out"]]}
    # activations are rounded to 16 bits after every linear, and the roundings of the layers add
    # up like independent errors (measured against 64 bits: 5.5e-4 after 4 fp16 layers, 3.7e-3
    # and 1.1e-2 after 1 and 24 bf16 layers)
    return {"rel": {"f16": 1e-3, "bf16": 8e-3}[c["dtype"]] * math.sqrt(c["L"])}


def _linear64(x, W, b):
    y = torch.empty((x.shape[0], W.shape[0]), dtype=torch.float64, device=x.device)
    for r in range(0, W.shape[0], 8192):  # in blocks of rows, to bound the 64-bit copies
        y[:, r:r + 8192] = x @ W[r:r + 8192].double().t()
    return y + b.double()


def _norm64(x):
    m = x.mean(1, keepdim=True)
    return (x - m) / torch.sqrt(((x - m) ** 2).mean(1, keepdim=True) + LN_EPS)


def _attend64(c, q, k, v):
    """q [B, H], k and v [B, n, H]: per-head softmax attention."""
    B, n, D, h = c["B"], k.shape[1], c["D"], c["H"] // c["D"]
    q, k, v = q.view(B, 1, h, D), k.view(B, n, h, D), v.view(B, n, h, D)
    p = torch.softmax((q * k).sum(-1) / math.sqrt(D), dim=1)
    return (p.unsqueeze(-1) * v).sum(1).reshape(B, c["H"])


def exact(case, seed):
    c = case
    if c["kind"] == "kv_fill":
        t = _inputs(c, seed)
        return t["k"], t["v"]
    t = _inputs(c, seed)
    if c["kind"] in ("linear", "tiled"):
        return _linear64(t["x"].double(), t["W"], t["b"])
    H = c["H"]
    x = t["x"].double()
    for l in range(c["L"]):
        q = _linear64(_norm64(x), t["W"][0], t["b"][0])
        a = q[:, 2 * H:]
        if c["kind"] == "kv_step":
            k = torch.cat([t["k"][l].double(), q[:, None, H:2 * H]], 1)
            v = torch.cat([t["v"][l].double(), q[:, None, 2 * H:]], 1)
            a = _attend64(c, q[:, :H], k, v)
        x = x + _linear64(a, t["W"][1], t["b"][1])
        f = torch.relu(_linear64(_norm64(x), t["W"][2], t["b"][2]))
        x = x + _linear64(f, t["W"][3], t["b"][3])
    return x
