"""Timed cases of the executor's public entry points.

Each case is one call (or one fixed group of calls) as a user's program
makes it: the kernel classes through ``paper_2206_07896_amd.ops``, a batch of
mixed launches and a chain of dependent launches through ``batch.Batch``, and
the schedule cost model through its C ABI.  Outputs and workspaces that such
a program allocates once are allocated in ``prepare``.

A case's plain values fix every size; the values in the buffers come from the
seed alone.
"""

import math

import numpy as np
import torch

import paper_2206_07896_amd as spmd
from paper_2206_07896_amd import batch as B
from paper_2206_07896_amd import learned
from paper_2206_07896_amd import workload

DEV = "cuda"


def listed():
    return [
        # the smallest configured launch: 2^20 ints summed by 4096 blocks of
        # 256, where the latency of a launch counts
        {"name": "reduce_2e20", "kind": "reduce", "n": 1 << 20, "grid": 4096, "block": 256},
        # the two launches of the headline step: prefix sum of 2^26 ints,
        # 256-bin histogram of 2^27 skewed keys
        {"name": "scan_2e26", "kind": "scan", "n": 1 << 26, "block": 512, "items": 128},
        {"name": "hist_2e27_zipf", "kind": "hist", "n": 1 << 27, "grid": 256, "block": 1024, "alpha": 1.1},
        # a database selection that keeps about half of 2^26 ints
        {"name": "compact_2e26", "kind": "compact", "n": 1 << 26, "block": 1024, "items": 32, "t": 0},
        # one sweep of the configured 8192^2 stencil in 16 x 16 blocks
        {"name": "jacobi_8192", "kind": "jacobi", "nx": 8192, "ny": 8192, "bx": 16, "by": 16, "cells": 1},
        # eight sweeps of the same grid in one launch
        {"name": "jacobi_8192_fused8", "kind": "fused", "nx": 8192, "ny": 8192, "sweeps": 8},
        # an iterative solver: 100 sweeps of a 1024^2 grid as one dependent
        # batch, each sweep reading the one before it
        {"name": "chain_1024_x100", "kind": "chain", "nx": 1024, "ny": 1024, "sweeps": 100, "block": 256, "items": 4,
         "bpf": 0},
        # the configured square product, and an ordinary one of odd sizes at
        # the default tile
        {"name": "gemm_4096_t64", "kind": "gemm", "m": 4096, "n": 4096, "k": 4096, "tile": 64},
        {"name": "gemm_odd", "kind": "gemm", "m": 1000, "n": 901, "k": 1111, "tile": 128},
        # 2000 launches of four classes and of 2^10 to 2^22 elements run from
        # the block queue under the shipped model's schedules
        {"name": "mixed_2000", "kind": "mixed", "count": 2000, "log2_hi": 22.0, "mix": 0xC5F},
        # one full-batch training step of the cost model (forward, gradient,
        # Adam) on the rows of 500 tuned launches
        {"name": "mlp_train_60k", "kind": "train", "n": 60000},
        # schedules for 10 000 launches by a three-model ensemble
        {"name": "mlp_choose_10000", "kind": "choose", "m": 10000, "models": 3, "slack": -1.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes log-uniform, odd ones among
    them."""
    kind = rng.choice(["reduce", "scan", "hist", "compact", "jacobi", "fused", "chain", "gemm", "mixed", "train",
                       "choose"])
    if kind == "reduce":
        return {"kind": kind, "n": _log_int(rng, 1 << 10, 1 << 27), "grid": rng.choice([256, 1024, 4096, 16384]),
                "block": rng.choice([128, 256, 512, 1024])}
    if kind == "scan":
        n = _log_int(rng, 1 << 10, 1 << 26)
        block, items = rng.choice([(512, 16), (256, 8), (256, 16)] if n < 1 << 21 else [(512, 16), (512, 64), (512, 128)])
        return {"kind": kind, "n": n, "block": block, "items": items}
    if kind == "hist":
        return {"kind": kind, "n": _log_int(rng, 1 << 10, 1 << 27), "grid": rng.choice([64, 256, 1024]),
                "block": rng.choice([256, 512, 1024]), "alpha": rng.choice([0.0, 1.1, 2.0])}
    if kind == "compact":
        n = _log_int(rng, 1 << 10, 1 << 26)
        block, items = rng.choice([(256, 16), (512, 16)] if n < 1 << 21 else [(256, 16), (512, 32), (1024, 32)])
        return {"kind": kind, "n": n, "block": block, "items": items, "t": rng.choice([-600, 0, 600])}
    if kind == "jacobi":
        bx, by = rng.choice([(16, 16), (64, 4), (32, 8)])
        return {"kind": kind, "nx": _log_int(rng, 32, 8192), "ny": _log_int(rng, 32, 8192), "bx": bx, "by": by,
                "cells": rng.choice([1, 2, 4])}
    if kind == "fused":
        return {"kind": kind, "nx": 4 * _log_int(rng, 8, 2048), "ny": _log_int(rng, 32, 8192),
                "sweeps": rng.randint(2, 8)}
    if kind == "chain":
        block, items, bpf = rng.choice([(256, 4, 0), (512, 4, 8)])
        return {"kind": kind, "nx": _log_int(rng, 64, 2048), "ny": _log_int(rng, 64, 2048),
                "sweeps": rng.randint(8, 100), "block": block, "items": items, "bpf": bpf}
    if kind == "gemm":
        q = rng.choice([1, 1, 4, 16])
        m, n, k = (max(1, _log_int(rng, 32, 4096) // q) * q for _ in range(3))
        return {"kind": kind, "m": m, "n": n, "k": k, "tile": rng.choice([64, 128, 128, 256])}
    if kind == "mixed":
        return {"kind": kind, "count": _log_int(rng, 50, 2000), "log2_hi": rng.choice([16.0, 18.0, 20.0, 22.0]),
                "mix": rng.randrange(1, 1 << 16)}
    if kind == "train":
        return {"kind": kind, "n": _log_int(rng, 500, 60000)}
    return {"kind": kind, "m": _log_int(rng, 100, 10000), "models": rng.choice([1, 3, 4]),
            "slack": rng.choice([-1.0, 0.2, 1.0])}


# ---- inputs -----------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _ints(g, n, lo, hi):
    return torch.randint(lo, hi + 1, (n,), dtype=torch.int32, device=DEV, generator=g)


def _keys(g, n, alpha):
    """Bounded Zipf(alpha) keys over 256 bins."""
    w = 1.0 / np.power(np.arange(1, 257, dtype=np.float64), alpha)
    cdf = torch.from_numpy((np.cumsum(w) / w.sum()).astype(np.float32)).to(DEV)
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    for lo in range(0, n, 1 << 25):
        hi = min(n, lo + (1 << 25))
        u = torch.rand(hi - lo, device=DEV, generator=g)
        out[lo:hi] = torch.searchsorted(cdf, u, right=True, out_int32=True).clamp_(max=255)
    return out


def _grid_input(case, seed):
    return torch.rand((case["ny"], case["nx"]), device=DEV, generator=_gen(seed))


def _gemm_input(case, seed):
    g = _gen(seed)
    return (torch.randn((case["m"], case["k"]), device=DEV, generator=g),
            torch.randn((case["k"], case["n"]), device=DEV, generator=g))


def _specs(case):
    return workload.mixed_specs(case["count"], seed=case["mix"], log2_hi=case["log2_hi"])


def _pad(n):
    return -(-n // 64) * 64


MIX_KINDS = (spmd.REDUCE_I32, spmd.SCAN_I32, spmd.HIST256_U32, spmd.JACOBI5_F32)


def _mix_layout(specs):
    """Offsets of each launch's input and output in its class's arenas, and
    the arenas' sizes."""
    size_in = dict.fromkeys(MIX_KINDS, 0)
    size_out = dict.fromkeys(MIX_KINDS, 0)
    at = []
    for s in specs:
        k = s["kid"]
        at.append((size_in[k], size_out[k]))
        size_in[k] += _pad(s["n"])
        size_out[k] += {spmd.REDUCE_I32: 64, spmd.HIST256_U32: 256}.get(k, _pad(s["n"]))
    return at, size_in, size_out


def _mix_inputs(sizes, seed):
    g = _gen(seed)
    return {spmd.REDUCE_I32: _ints(g, sizes[spmd.REDUCE_I32], -1000, 1000),
            spmd.SCAN_I32: _ints(g, sizes[spmd.SCAN_I32], 0, 100),
            spmd.HIST256_U32: _keys(g, sizes[spmd.HIST256_U32], 1.1),
            spmd.JACOBI5_F32: torch.rand(sizes[spmd.JACOBI5_F32], device=DEV, generator=g)}


# the 144 schedules' inputs: log2 of the block, the items and the blocks per
# fetch, as the library's candidate table lists them
def _cands():
    return torch.from_numpy(learned.candidate_inputs())


def _features(g, m):
    """Launch features of `m` launches of the mixed workload's kind, and
    their class."""
    kid = torch.randint(0, 4, (m,), device=DEV, generator=g)
    bd = torch.randint(6, 10, (m,), device=DEV, generator=g).float()
    f = torch.zeros((m, 9), device=DEV)
    f[torch.arange(m, device=DEV), kid] = 1.0
    f[:, 4] = 10.0 + 12.0 * torch.rand(m, device=DEV, generator=g)
    f[:, 5] = bd
    shm = torch.stack([2 + bd, torch.log2(4 * torch.exp2(bd - 5) + 4), torch.full_like(bd, 10.0),
                       torch.log2(4 * (torch.exp2(bd - 6) + 2) * 66)], 1)
    bar = torch.stack([bd + 1, torch.full_like(bd, 2.0), torch.full_like(bd, 2.0), torch.full_like(bd, 1.0)], 1)
    f[:, 6] = shm.gather(1, kid[:, None])[:, 0]
    f[:, 7] = bar.gather(1, kid[:, None])[:, 0]
    f[:, 8] = torch.where(kid == 1, 10.0, 0.0)
    return f, kid


def _net(g, models):
    """He-style weights and small biases, one vector per model."""
    def w(*shape, scale):
        return torch.randn(shape, device=DEV, generator=g) * scale
    return torch.stack([torch.cat([w(768, scale=math.sqrt(2 / 12)), w(64, scale=0.1), w(4096, scale=math.sqrt(2 / 64)),
                                   w(64, scale=0.1), w(64, scale=math.sqrt(1 / 64)), w(1, scale=0.1)])
                        for _ in range(models)]).contiguous()


def _norm(x):
    sd = x.std(0)
    return torch.cat([x.mean(0), torch.where(sd > 1e-6, 1 / sd.clamp(min=1e-6), torch.ones_like(sd))]).contiguous()


def _train_input(case, seed):
    g, n = _gen(seed), case["n"]
    f, kid = _features(g, n)
    c = _cands().to(DEV)
    x = torch.cat([f, c[torch.randint(0, c.shape[0], (n,), device=DEV, generator=g)]], 1).contiguous()
    # log-microseconds: a floor, the elements' share, a cost per fetch, noise
    t = torch.log(3 + torch.exp2(x[:, 4] - 14) * (1 + 0.3 * kid) + torch.exp2((x[:, 4] - x[:, 9:].sum(1)) / 2 - 2))
    t = (t + 0.05 * torch.randn(n, device=DEV, generator=g)).contiguous()
    p = _net(g, 1)[0].contiguous()
    return {"x": x, "t": t, "norm": _norm(x), "p": p,
            "m": 1e-3 * torch.randn(p.numel(), device=DEV, generator=g),
            "v": 1e-4 * (0.5 + torch.rand(p.numel(), device=DEV, generator=g))}


def _choose_input(case, seed):
    g = _gen(seed)
    f, kid = _features(g, case["m"])
    c = _cands().to(DEV)
    b, it, bpf = c[:, 0], c[:, 1], c[:, 2]
    # 8 cells per thread at most for the stencil, 32 items for scans alone
    valid = torch.where(kid[:, None] == 3, it <= 3, torch.where(kid[:, None] == 1, it <= 5, it <= 4))
    bpf = torch.where(kid[:, None] == 1, torch.zeros_like(bpf), bpf)
    chunks = torch.ceil(torch.exp2(f[:, 4:5] - b - it - bpf)).clamp(min=1).to(torch.int32)
    chunks = torch.where(valid, chunks, torch.full_like(chunks, -1)).contiguous()
    rows = torch.cat([f.repeat_interleave(2, 0), c[torch.randint(0, c.shape[0], (2 * case["m"],), device=DEV, generator=g)]], 1)
    return {"f": f.contiguous(), "c": c.contiguous(), "valid": valid.to(torch.uint8).contiguous(), "chunks": chunks,
            "norm": _norm(rows), "p": _net(g, case["models"])}


LR, B1, B2, EPS = 3e-3, 0.9, 0.999, 1e-8


# ---- a user's program -------------------------------------------------------

def prepare(case, seed):
    k = case["kind"]
    s = dict(case)
    if k == "reduce":
        s["x"] = _ints(_gen(seed), case["n"], -1000, 1000)
        s["partials"] = torch.empty(case["grid"], dtype=torch.int32, device=DEV)
        s["out"] = torch.empty(1, dtype=torch.int32, device=DEV)
        s["ws"] = spmd.ops.workspace(spmd.REDUCE_I32, case["grid"], case["block"], case["n"])
    elif k == "scan":
        s["x"] = _ints(_gen(seed), case["n"], 0, 100)
        s["y"] = torch.empty_like(s["x"])
        grid = spmd.ops.scan_grid(case["n"], case["block"], case["items"])
        s["ws"] = spmd.ops.workspace(spmd.SCAN_I32, grid, case["block"], case["n"])
    elif k == "hist":
        s["x"] = _keys(_gen(seed), case["n"], case["alpha"])
        s["hist"] = torch.empty(256, dtype=torch.int32, device=DEV)
    elif k == "compact":
        s["x"] = _ints(_gen(seed), case["n"], -1000, 1000)
        s["y"] = torch.zeros_like(s["x"])
        s["count"] = torch.empty(1, dtype=torch.int32, device=DEV)
        grid = spmd.ops.compact_grid(case["n"], case["block"], case["items"])
        s["ws"] = spmd.ops.workspace(spmd.COMPACT_I32, grid, case["block"], case["n"])
    elif k in ("jacobi", "fused"):
        s["u"] = _grid_input(case, seed)
        s["v"] = torch.empty_like(s["u"])
    elif k == "chain":
        u = _grid_input(case, seed)
        s["bufs"] = [u, torch.empty_like(u)]
        n = case["sweeps"]
        items = [(spmd.JACOBI5_F32, case["nx"], case["ny"], 256, s["bufs"][i % 2], s["bufs"][(i + 1) % 2])
                 for i in range(n)]
        s["batch"] = B.Batch(items, [(case["block"], case["items"], case["bpf"])] * n,
                             deps=[None] + list(range(n - 1)))
    elif k == "gemm":
        s["A"], s["B"] = _gemm_input(case, seed)
        s["C"] = torch.empty((case["m"], case["n"]), device=DEV)
    elif k == "mixed":
        specs = _specs(case)
        at, size_in, size_out = _mix_layout(specs)
        src = _mix_inputs(size_in, seed)
        s["out"] = {i: torch.zeros(size_out[i], dtype=torch.float32 if i == spmd.JACOBI5_F32 else torch.int32,
                                   device=DEV) for i in MIX_KINDS}
        items = [(q["kid"], q["nx"], q["ny"], q["block_dim"], src[q["kid"]][i:], s["out"][q["kid"]][o:])
                 for q, (i, o) in zip(specs, at)]
        model = learned.load_default()
        choice = model.choose(specs, slack=model.slack)[0]
        s["src"] = src
        s["batch"] = B.Batch(items, [learned.CANDIDATES[j] for j in choice])
    elif k == "train":
        s.update(_train_input(case, seed))
        n = case["n"]
        s["y"] = torch.empty(n, device=DEV)
        s["h1"], s["h2"] = torch.empty((64, n), device=DEV), torch.empty((64, n), device=DEV)
        s["grad"], s["loss"] = torch.empty_like(s["p"]), torch.empty(1, device=DEV)
        s["ws"] = torch.empty(int(spmd.lib().spmd_mlp_workspace_size(n)), dtype=torch.uint8, device=DEV)
        s["step"] = 100
    else:
        s.update(_choose_input(case, seed))
        m = case["m"]
        s["best"] = torch.empty(m, dtype=torch.int32, device=DEV)
        s["pred"], s["sd"] = torch.empty(m, device=DEV), torch.empty(m, device=DEV)
    return s


def _ok(rc):
    if rc:
        raise spmd.SpmdError(rc)


def run(s):
    k = s["kind"]
    if k == "reduce":
        return spmd.ops.reduce_i32(s["x"], s["grid"], s["block"], s["partials"], s["out"], s["ws"])
    if k == "scan":
        return spmd.ops.scan_i32(s["x"], s["block"], s["items"], y=s["y"], ws=s["ws"])
    if k == "hist":
        return spmd.ops.hist256_u32(s["x"], s["grid"], s["block"], hist=s["hist"])
    if k == "compact":
        return spmd.ops.compact_i32(s["x"], s["t"], s["block"], s["items"], y=s["y"], count=s["count"], ws=s["ws"])
    if k == "jacobi":
        return spmd.ops.jacobi5_f32(s["u"], s["v"], (s["bx"], s["by"]), s["cells"])
    if k == "fused":
        return spmd.ops.jacobi5t_f32(s["u"], s["sweeps"], s["v"])
    if k == "chain":
        s["batch"].graph_launch()
        return s["bufs"]
    if k == "gemm":
        return spmd.ops.gemm_f32(s["A"], s["B"], s["C"], s["tile"])
    if k == "mixed":
        s["batch"].graph_launch()
        return [s["out"][i] for i in MIX_KINDS]
    lib, st = spmd.lib(), torch.cuda.current_stream().cuda_stream
    if k == "train":
        p, nm, x, h1, h2 = (s[i].data_ptr() for i in ("p", "norm", "x", "h1", "h2"))
        n, y, g = s["n"], s["y"].data_ptr(), s["grad"].data_ptr()
        _ok(lib.spmd_mlp_forward(p, nm, x, n, y, h1, h2, st))
        _ok(lib.spmd_mlp_backward(p, nm, x, s["t"].data_ptr(), n, y, h1, h2, g, s["loss"].data_ptr(),
                                  s["ws"].data_ptr(), s["ws"].numel(), st))
        _ok(lib.spmd_mlp_adam(p, g, s["m"].data_ptr(), s["v"].data_ptr(), s["step"], LR, B1, B2, EPS, st))
        s["step"] += 1
        return {i: s[i] for i in ("y", "h1", "h2", "grad", "loss", "p", "m", "v")}
    a = (s["p"].data_ptr(), s["models"], s["norm"].data_ptr(), s["f"].data_ptr(), s["m"], s["c"].data_ptr(),
         s["c"].shape[0], s["valid"].data_ptr())
    o = (s["best"].data_ptr(), s["pred"].data_ptr(), s["sd"].data_ptr(), st)
    if s["slack"] < 0:
        _ok(lib.spmd_mlp_choose(*a, *o))
    else:
        _ok(lib.spmd_mlp_choose_batch(*a, s["chunks"].data_ptr(), s["slack"], *o))
    return {"best": s["best"], "pred": s["pred"], "sd": s["sd"]}


def work(case):
    k = case["kind"]
    if k == "reduce":
        return {"bytes": 4 * case["n"] + 4 * case["grid"] + 4, "flops": 0}
    if k == "scan":
        return {"bytes": 8 * case["n"], "flops": 0}
    if k == "hist":
        return {"bytes": 4 * case["n"] + 1024, "flops": 0}
    if k == "compact":  # int32 uniform on [-1000, 1000]
        return {"bytes": int(4 * case["n"] * (1 + (1000 - case["t"]) / 2001)) + 4, "flops": 0}
    if k in ("jacobi", "fused"):
        c = case["nx"] * case["ny"]
        return {"bytes": 8 * c, "flops": 4 * c * case.get("sweeps", 1)}
    if k == "chain":  # the grid read once, both buffers left written
        c = case["nx"] * case["ny"]
        return {"bytes": 12 * c, "flops": 4 * c * case["sweeps"]}
    if k == "gemm":
        m, n, kk = case["m"], case["n"], case["k"]
        return {"bytes": 4 * (m * kk + kk * n + m * n), "flops": 2 * m * n * kk}
    if k == "mixed":
        specs = _specs(case)
        return {"bytes": sum(workload.algorithmic_bytes(q) for q in specs),
                "flops": sum(4 * q["n"] for q in specs if q["kid"] == spmd.JACOBI5_F32)}
    net = 12 * 64 + 64 * 64 + 64
    if k == "train":  # forward; the error's way back and the weights' gradients
        n = case["n"]
        return {"bytes": n * (4 * 12 + 4 + 4 + 2 * 4 * 64) + 4 * 8 * (net + 129), "flops": 2 * n * (2 * net + 64 * 64)}
    rows = case["m"] * 120  # valid candidates of a launch, averaged over the classes
    return {"bytes": case["m"] * (36 + 144 + 12) + 4 * case["models"] * (net + 129),
            "flops": 2 * rows * case["models"] * net}


# ---- the same in 64 bits ----------------------------------------------------

def _sweep64(u):
    v = u.clone()
    if u.shape[0] > 2 and u.shape[1] > 2:
        v[1:-1, 1:-1] = 0.25 * ((u[:-2, 1:-1] + u[2:, 1:-1]) + (u[1:-1, :-2] + u[1:-1, 2:]))
    return v


def _unpack(p):
    p = p.double()
    return (p[:768].view(12, 64), p[768:832], p[832:4928].view(64, 64), p[4928:4992], p[4992:5056], p[5056])


def _forward64(p, norm, x):
    w1, b1, w2, b2, w3, b3 = _unpack(p)
    xn = (x.double() - norm[:12].double()) * norm[12:].double()
    h1 = torch.relu(xn @ w1 + b1)
    h2 = torch.relu(h1 @ w2 + b2)
    return xn, h1, h2, h2 @ w3 + b3


def exact(case, seed):
    k = case["kind"]
    if k in ("jacobi", "fused", "chain"):
        u = _grid_input(case, seed).double()
        sweeps, before = case.get("sweeps", 1), None
        for _ in range(sweeps):
            before, u = u, _sweep64(u)
        if k != "chain":
            return u
        return [u, before] if sweeps % 2 == 0 else [before, u]
    if k == "gemm":
        a, b = _gemm_input(case, seed)
        return a.double() @ b.double()
    if k == "mixed":
        specs = _specs(case)
        at, size_in, size_out = _mix_layout(specs)
        src = _mix_inputs(size_in, seed)[spmd.JACOBI5_F32]
        out = torch.zeros(size_out[spmd.JACOBI5_F32], dtype=torch.float64, device=DEV)
        for q, (i, o) in zip(specs, at):
            if q["kid"] == spmd.JACOBI5_F32:
                u = src[i:i + q["n"]].view(q["ny"], q["nx"]).double()
                out[o:o + q["n"]] = _sweep64(u).reshape(-1)
        return [None, None, None, out]
    if k == "train":
        s = _train_input(case, seed)
        n = case["n"]
        xn, h1, h2, y = _forward64(s["p"], s["norm"], s["x"])
        _, _, w2, _, w3, _ = _unpack(s["p"])
        e = y - s["t"].double()
        dy = 2 * e / n
        d2 = torch.where(h2 > 0, dy[:, None] * w3, 0.0)
        d1 = torch.where(h1 > 0, d2 @ w2.T, 0.0)
        grad = torch.cat([(xn.T @ d1).reshape(-1), d1.sum(0), (h1.T @ d2).reshape(-1), d2.sum(0), dy @ h2,
                          dy.sum()[None]])
        m = B1 * s["m"].double() + (1 - B1) * grad
        v = B2 * s["v"].double() + (1 - B2) * grad * grad
        p = s["p"].double() - LR * (m / (1 - B1 ** 100)) / (torch.sqrt(v / (1 - B2 ** 100)) + EPS)
        return {"y": y, "h1": h1.T.contiguous(), "h2": h2.T.contiguous(), "grad": grad, "loss": (e * e).mean()[None],
                "p": p, "m": m, "v": v}
    if k == "choose" and case["slack"] < 0:  # the spread belongs to the pick, which a near tie may move
        s = _choose_input(case, seed)
        pred = torch.empty(case["m"], dtype=torch.float64, device=DEV)
        c = s["c"].shape[0]
        for lo in range(0, case["m"], 2000):
            f = s["f"][lo:lo + 2000]
            x = torch.cat([f.repeat_interleave(c, 0), s["c"].repeat(f.shape[0], 1)], 1)
            mean = sum(_forward64(p, s["norm"], x)[3] for p in s["p"]) / case["models"]
            mean = mean.view(-1, c).masked_fill(s["valid"][lo:lo + 2000] == 0, math.inf)
            pred[lo:lo + 2000] = mean.min(1).values
        return {"best": None, "pred": pred, "sd": None}
    return None
