"""What this framework is measured on: the calls a user makes, from one
serving step priced on its own to a whole 70B trace.

A case names the call (``op``), the decoder shape, the record form, the number
of serving steps and spec vectors, and the source of the efficiency factor:

* ``op`` "steps": ks_eval_steps (step latencies; ``outs`` "all": per-kernel
  outputs too); "expand_steps": ks_expand, then ks_eval_steps, as a program
  does that is handed batch descriptors; "kernels": ks_eval_kernels
  (``outs`` "latency": t_kernel; "all": the counts, t_roof, eta, t_kernel);
  "expand": ks_expand alone; "simulate": ks_simulate through
  ``abi.simulate_many``.
* ``form`` "layers": a record per dispatched kernel; "homogeneous": a record
  per kernel that is the same in all layers, with its multiplicity.
* ``head`` "f32" / "bf16" (``inp``-``hid``-``hid``-1 heads) or "one" (eta = 1);
  ``bounded`` / ``grid``: every family on the bounded analytical head, every
  family with a measured grid in front of its other head.

Inputs are synthetic: batch sizes U{1..batch}, lognormal contexts (median
1024, sigma 1) capped at ``ctx``, a prefill chunk U{64..2048} in 30% of the
steps, Dirichlet(0.5) routing for a mixture of experts, hypothetical GPUs over
the ranges of the capacity grid, N(0, 0.1^2) head weights.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2606_28565_amd import abi

FIELDS = ("hidden", "layers", "q_heads", "kv_heads", "head_dim", "ffn", "vocab", "tp", "experts", "top_k",
          "expert_ffn", "kv_write")
SHAPES = {
    "7b": (4096, 32, 32, 32, 128, 11008, 32000, 1, 0, 0, 0, 0),
    "s1": (2048, 24, 16, 8, 128, 5632, 32000, 1, 0, 0, 0, 0),
    "s3": (4096, 32, 32, 8, 128, 14336, 32000, 2, 0, 0, 0, 0),
    "s4": (5120, 40, 40, 8, 128, 13824, 32000, 4, 0, 0, 0, 0),
    "s6": (8192, 80, 64, 8, 128, 28672, 32000, 8, 0, 0, 0, 0),
    "moe": (4096, 32, 32, 8, 128, 0, 32000, 1, 8, 2, 14336, 0),
    "70b": (8192, 80, 64, 8, 128, 28672, 32000, 1, 0, 0, 0, 0),
}
HOST = (4.0e-6, 1.5e-3, 2.5e-3, 3.0e-4, 1.04)   # c_disp, ell, c_ovl, c_tail, body_scale
(GEMM, LM_HEAD, GROUPED, PREFILL, DECODE, RMSNORM, ROPE, SILU, KV_WRITE, EMBED) = range(10)
NFAM = 10
FIELDS_READ = (4, 4, 5, 4, 4, 3, 4, 3, 4, 3)     # record fields a family's formulas read
GRID = {"axes": (1, 2, 6), "lo": (-0.8, 0.0, -0.4), "hi": (0.2, 0.4, 0.6), "n": (8, 8, 8)}


def _case(name, op, shape, form, steps, specs, head, inp=16, hid=128, batch=64, ctx=32768, bounded=False,
          grid=False, outs="sums"):
    c = {"op": op, "shape": shape, "form": form, "steps": steps, "specs": specs, "head": head, "inp": inp,
         "hid": hid, "batch": batch, "ctx": ctx, "bounded": bounded, "grid": grid, "outs": outs}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one serving step priced for one GPU: what a scheduler asks for before
        # every step (latency of the call, launches)
        _case("one step", "expand_steps", "7b", "homogeneous", 1, 1, "f32", 16, 64, ctx=4096),
        # one round of 64 simulations in lockstep: 64 steps x 64 spec vectors
        _case("lockstep round", "expand_steps", "7b", "homogeneous", 64, 64, "f32", 16, 64, batch=256),
        # a 1000-step trace on two datasheets with every per-kernel output: the
        # accuracy study of a small trace
        _case("7b trace, per kernel", "steps", "7b", "layers", 1000, 2, "f32", 16, 64, ctx=4096, outs="all"),
        # capacity planning: two 7B traces against 256 hypothetical GPUs (the
        # default benchmark)
        _case("capacity grid", "steps", "7b", "layers", 1345, 256, "bf16", 16, 128, batch=128),
        # the same question with the widest fp32 heads, layers collapsed
        _case("fp32 grid", "steps", "7b", "homogeneous", 4001, 64, "f32", 32, 128),
        # a dense TP-4 trace, one record per kernel, two datasheets
        _case("dense trace", "steps", "s4", "layers", 20000, 2, "bf16", 16, 128, batch=256),
        # a mixture-of-experts trace: ragged grouped GEMMs, routing per layer
        _case("moe trace", "steps", "moe", "layers", 8000, 2, "bf16", 16, 128),
        # a 70B batch from its batch descriptors, one record per kernel (the
        # largest call)
        _case("70b batch", "expand_steps", "70b", "layers", 40000, 2, "bf16", 32, 256, ctx=131072),
        # a 70B trace from its batch descriptors, layers collapsed
        _case("70b homogeneous", "expand_steps", "70b", "homogeneous", 80000, 2, "bf16", 32, 256, ctx=131072),
        # the pure roofline of every kernel of a large trace
        _case("roofline, per kernel", "kernels", "70b", "layers", 40001, 2, "one", outs="latency", ctx=131072),
        # measured grids with the learned heads behind them (Tier B)
        _case("measured grids", "steps", "s3", "homogeneous", 6001, 16, "bf16", 16, 128, batch=256, grid=True),
        # serving simulation, the scheduler in the loop, 16 GPUs in lockstep
        _case("simulation", "simulate", "7b", "homogeneous", 150, 16, "f32", 16, 64, batch=256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(case):
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / (6e13 if case["head"] == "f32" else 1.2e15)


def draw(rng):
    """One more case of the same ranges: any shape, form, head and output set;
    1 step to a whole trace, 1 to 256 spec vectors."""
    most = max(_cost(c) for c in listed())
    while True:
        op = rng.choice(["steps", "steps", "steps", "expand_steps", "expand_steps", "kernels", "kernels", "expand",
                         "simulate"])
        if op == "simulate":
            return _case(None, op, rng.choice(["7b", "s1", "s3"]), "homogeneous", rng.randint(20, 150),
                         rng.randint(1, 16), "f32", 16, 64, batch=rng.choice([64, 256]))
        head = rng.choice(["f32", "bf16", "bf16", "one"])
        inp = rng.choice([16, 32])
        hid = rng.choice([64, 128] if head == "f32" else [64, 128, 256])
        outs = "sums"
        if op == "kernels":
            outs = rng.choice(["latency", "all"])
        elif op == "steps":
            outs = rng.choice(["sums", "sums", "all"])
        c = _case(None, op, rng.choice(sorted(SHAPES)), rng.choice(["layers", "homogeneous"]),
                  _log_int(rng, 1, 80000), _log_int(rng, 1, 256), head, inp, hid, rng.choice([1, 33, 64, 256]),
                  rng.choice([4096, 32768, 131072]), rng.random() < 0.15, rng.random() < 0.15, outs)
        if op == "expand":
            c.update(head="one", specs=1, bounded=False, grid=False)
        pairs = _rows(c) * c["specs"]
        head_work = pairs * (hid * (inp + hid)) * {"one": 0, "bf16": 1, "f32": 12}[c["head"]]
        routed = c["steps"] * 256 if c["shape"] == "moe" else 0   # routing draws are host work
        if (_cost(c) <= most and _rows(c) <= 30_000_000 and routed <= 2_100_000 and c["steps"] * c["specs"] <= 2_000_000
                and head_work <= 4.0e12 and pairs <= 4.0e8 and (c["outs"] == "sums" or pairs <= 6.0e7)):
            return c


# ------------------------------------------------------------------ inputs
def _shape(case):
    return SimpleNamespace(**dict(zip(FIELDS, SHAPES[case["shape"]])))


def _trace(case, seed):
    rng = np.random.Generator(np.random.PCG64([20260602, int(seed)]))
    S = case["steps"]
    batch = rng.integers(1, case["batch"], size=S, endpoint=True)
    prefill = rng.random(S) < 0.3
    chunk = rng.integers(64, 2048, size=S, endpoint=True)
    off = np.zeros(S + 1, np.int64)
    np.cumsum(batch, out=off[1:])
    h = np.floor(rng.lognormal(math.log(1024.0), 1.0, int(off[-1])))
    h = np.minimum(case["ctx"], np.maximum(1, h)).astype(np.int64)
    q = np.ones(int(off[-1]), np.int64)
    q[off[:-1][prefill]] = chunk[prefill]
    s = _shape(case)
    experts = None
    if s.experts:
        tokens = np.add.reduceat(q, off[:-1])
        copies = np.repeat(s.top_k * tokens, s.layers)
        g = rng.standard_gamma(0.5, (len(copies), s.experts)) + 1e-12
        experts = rng.multinomial(copies, g / g.sum(1, keepdims=True)).reshape(S, s.layers, s.experts)
    return SimpleNamespace(shape=s, n_steps=S, req_off=off, req_q=q, req_h=h, prefill=prefill, experts=experts)


def _specs(case, seed):
    rng = np.random.Generator(np.random.PCG64([20260603, int(seed)]))
    n = case["specs"]

    def logu(lo, hi):
        return np.exp(rng.uniform(math.log(lo), math.log(hi), n))

    return {"peak_flops": logu(0.5e15, 5e15), "hbm_bw": logu(2e12, 10e12), "t0": logu(1e-6, 5e-6),
            "l2_bytes": logu(32 * 2.0 ** 20, 256 * 2.0 ** 20), "ar_alpha0": np.full(n, 8.0e-6),
            "ar_alpha_log2p": np.full(n, 2.0e-6), "ar_beta": logu(100e9, 900e9),
            "n_cu": rng.integers(64, 320, n, endpoint=True)}


def _head(case, seed):
    """Parameters at their storage precision, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 31) + 17)
    I, H = case["inp"], case["hid"]
    dt = torch.bfloat16 if case["head"] == "bf16" else torch.float32
    p = {n: (0.1 * torch.randn(s, generator=g, device="cuda")).to(dt)
         for n, s in (("w1", (NFAM, H, I)), ("w2", (NFAM, H, H)), ("b2", (NFAM, H)), ("w3", (NFAM, H)), ("b3", (NFAM,)))}
    p["bounded"] = 0.5 * torch.randn((NFAM, 2, 16), generator=g, device="cuda")
    if case["grid"]:
        lo, hi, n = GRID["lo"], GRID["hi"], GRID["n"]
        c = torch.meshgrid(*(torch.linspace(lo[d], hi[d], n[d], device="cuda") for d in range(3)), indexing="ij")
        off = 0.5 * torch.rand((NFAM, 1, 1, 1), generator=g, device="cuda")
        v = 1.0 + off + 0.6 * torch.sigmoid(3.0 * c[0] + 2.0) + 0.8 * c[1] + 0.3 * torch.cos(3.0 * c[2])
        v = torch.clamp(v + 0.02 * torch.randn((NFAM,) + n, generator=g, device="cuda"), min=1.0)
        v[torch.rand((NFAM,) + n, generator=g, device="cuda") < 0.08] = float("nan")
        p["grid"] = v.contiguous()
    return p


def _ks_heads(case, p):
    h = abi.ks_heads()
    h.in_dim, h.hidden = case["inp"], case["hid"]
    h.precision = abi.KS_BF16 if case["head"] == "bf16" else abi.KS_F32
    h.mode = abi.KS_ETA_ONE if case["head"] == "one" else abi.KS_ETA_MLP
    for n in ("w1", "w2", "b2", "w3", "b3"):
        setattr(h, n, p[n].data_ptr())
    if case["bounded"]:
        h.bounded_mask, h.bounded = (1 << NFAM) - 1, p["bounded"].data_ptr()
    if case["grid"]:
        h.grid_mask, h.grid = (1 << NFAM) - 1, p["grid"].data_ptr()
        for d in range(3):
            h.grid_axis[d], h.grid_n[d] = GRID["axes"][d], GRID["n"][d]
            h.grid_lo[d], h.grid_hi[d] = GRID["lo"][d], GRID["hi"][d]
    return h


def prepare(case, seed):
    st = SimpleNamespace(op=case["op"], S=case["specs"])
    st.params = _head(case, seed)
    st.heads = _ks_heads(case, st.params)
    st.host = abi.ks_host(*HOST)
    specs = _specs(case, seed)
    if case["op"] == "simulate":
        rng = np.random.Generator(np.random.PCG64([20260604, int(seed)]))
        n = case["steps"]
        group = np.where(rng.random(n) < 0.5, rng.integers(1, 9, n), 0)
        prefix = np.where(group > 0, rng.integers(256, 2048, 9, endpoint=True)[group], 0)
        prompt = np.clip(np.floor(rng.lognormal(math.log(512.0), 1.0, n)), 1, 8192)
        st.requests = {"arrival": np.cumsum(rng.exponential(1.0 / 20.0, n)),
                       "prompt": np.maximum(prompt, prefix).astype(np.uint32),
                       "output": np.clip(np.floor(rng.lognormal(math.log(128.0), 0.8, n)), 1, 2048).astype(np.uint32),
                       "group": group.astype(np.uint32), "prefix": prefix.astype(np.uint32)}
        st.shape, st.specs = _shape(case), specs
        st.sched = abi.ks_sched(case["batch"], 8192, 16, 1, 12500)
        return st
    tr = _trace(case, seed)
    st.stream = abi.current_stream()
    st.batch = abi.DeviceBatch(tr, abi.KS_EXPAND_PER_LAYER if case["form"] == "layers" else abi.KS_EXPAND_HOMOGENEOUS)
    if case["op"] == "expand":
        return st
    if case["op"] != "expand_steps":
        st.batch.expand(st.stream)
    st.specs = torch.from_numpy(abi.pack_specs(specs).view(np.uint8).copy()).cuda()
    st.ws_bytes = abi.ks_workspace_bytes(st.batch.desc, st.S)
    st.ws = torch.empty(st.ws_bytes + 256, dtype=torch.uint8, device="cuda")
    st.ws_ptr = st.ws.data_ptr() + (-st.ws.data_ptr()) % 256
    st.out = {}
    st.kout = None
    if case["op"] != "kernels":
        o, st.sout = abi.step_outputs(case["steps"], st.S)
        st.out.update(o)
    if case["outs"] != "sums":
        every = case["outs"] == "all"
        o, st.kout = abi.kernel_outputs(st.batch.desc.n_rows, st.S, counts=every, t_roof=every, eta=every)
        st.out.update(o)
    return st


def run(st):
    if st.op == "simulate":
        res = abi.simulate_many(st.shape, st.specs, st.heads, st.host, st.sched, st.requests, step_cap=1 << 14,
                                entry_cap=1 << 20)
        return {k: np.stack([r[k] for r in res]) for k in ("ttft", "tpot", "e2e", "clock")}
    b = st.batch
    if st.op in ("expand", "expand_steps"):
        b.expand(st.stream)
        if st.op == "expand":
            return {k: b.t[k] for k in ("step", "m", "n", "k", "a", "b", "mult", "s_n_launch") if k in b.t}
    if st.op == "kernels":
        abi.ks_eval_kernels(b.desc, st.specs.data_ptr(), st.S, st.heads, st.kout, st.ws_ptr, st.ws_bytes, st.stream)
    else:
        abi.ks_eval_steps(b.desc, b.steps, st.specs.data_ptr(), st.S, st.heads, st.host, st.sout, st.kout, st.ws_ptr,
                          st.ws_bytes, st.stream)
    return st.out


# ------------------------------------------------------------------ work
def _templates(s):
    """(family, m source, n, k, a, per layer) of a decoder's kernels, in
    dispatch order; PREFILL stands for the step's attention."""
    H, Hkv, d, D = s.q_heads // s.tp, -(-s.kv_heads // s.tp), s.head_dim, s.hidden
    t = [(GEMM, "T", (H + 2 * Hkv) * d, D, 0, True), (ROPE, "T", H + Hkv, d, 0, True),
         (PREFILL, "0", H, d, Hkv, True), (GEMM, "T", D, H * d, 0, True),
         (RMSNORM, "T", D, 0, 0, True), (RMSNORM, "T", D, 0, 0, True)]
    if s.experts:
        e = s.expert_ffn // s.tp
        t += [(GEMM, "T", s.experts, D, 0, True), (GROUPED, "0", 2 * e, D, s.experts, True),
              (SILU, "K", e, 0, 0, True), (GROUPED, "0", D, e, s.experts, True)]
    else:
        i = s.ffn // s.tp
        t += [(GEMM, "T", 2 * i, D, 0, True), (SILU, "T", i, 0, 0, True), (GEMM, "T", D, i, 0, True)]
    return t + [(EMBED, "T", D, 0, 0, False), (LM_HEAD, "R", s.vocab // s.tp, D, 0, False)]


def _per_step(case):
    """Records of one step by family, in the case's form."""
    s, n = _shape(case), [0] * NFAM
    for f, _, _, _, _, per_layer in _templates(s):
        n[f] += s.layers if per_layer and (case["form"] == "layers" or f == GROUPED) else 1
    return n


def _rows(case):
    return case["steps"] * sum(_per_step(case))


def work(case):
    """Bytes: the record fields that are read and the request lists, once, and
    the outputs.  FLOPs: the head's two matrix layers and output layer for
    every different kernel of a step (the same kernel in another layer has
    the same latency) and spec vector."""
    s, S, N = _shape(case), case["steps"], case["specs"]
    head = 2.0 * (case["inp"] * case["hid"] + case["hid"] ** 2 + case["hid"])
    different = 10 if not s.experts else 9 + 2 * s.layers
    req = 4.0 * S + 8.0 * S * (case["batch"] + 1) / 2
    if case["op"] == "simulate":   # about 128 decode steps per request over about 20 running ones
        steps = case["steps"] * 8
        return {"bytes": 300.0 * steps * N, "flops": head * 10 * steps * N}
    rows = _rows(case)
    b = req + 16.0 * S
    if case["op"] in ("expand", "expand_steps"):
        b += rows * (24.0 if case["form"] == "layers" else 28.0)
    if case["op"] != "expand":
        b += 4.0 * S * sum(n * k for n, k in zip(_per_step(case), FIELDS_READ))
        b += 4.0 * rows if case["form"] == "homogeneous" else 0.0
        b += 4.0 * S * s.layers * s.experts
        b += 24.0 * S * N if case["op"] != "kernels" else 0.0
        b += {"sums": 0.0, "latency": 4.0 * rows * N, "all": 24.0 * rows + 12.0 * rows * N}[case["outs"]]
    if case["op"] == "expand" or case["bounded"] or case["head"] == "one":
        return {"bytes": b, "flops": 0.0}
    return {"bytes": b, "flops": head * different * S * N}


def tolerance(case):
    if case["op"] == "expand":
        return "exact"
    if case["op"] == "simulate":
        # a latency's last bit can move an arrival past a step's start, which
        # moves a few requests of one simulation by one step
        return {"rel": 2e-2}
    if case["head"] == "bf16" and not case["bounded"]:
        # measured against 64 bits: 1e-4 (hidden 128) to 3e-4 (hidden 256)
        return {"rel": 2e-3}
    if case["grid"]:
        # a record within rounding of a cell next to an unmeasured node takes
        # the other source of eta
        return {"rel": 2e-3}
    # measured against 64 bits: 5e-8 to 9e-8
    return {"rel": 1e-6}


# ------------------------------------------------------------------ 64 bits
def _cd(a, b):
    return (a + b - 1) // b


def _records(case, tr):
    """Per family: different records in family order (step, then template),
    as int64 tensors of counts F, Bt, B, M, n, k, the step, and how many
    kernels each stands for (for grouped GEMMs: step, layer, template)."""
    s, dev = tr.shape, "cuda"
    off = torch.from_numpy(tr.req_off).to(dev)
    q, h = torch.from_numpy(tr.req_q).to(dev), torch.from_numpy(tr.req_h).to(dev)

    def per_step(v):
        c = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), torch.cumsum(v, 0)])
        return c[off[1:]] - c[off[:-1]]

    T, R = per_step(q), off[1:] - off[:-1]
    KV, PAIRS, TILES = per_step(q + h), per_step(q * h + q * (q + 1) // 2), per_step(_cd(q, 128))
    pre = torch.from_numpy(tr.prefill).to(dev)
    every = torch.arange(tr.n_steps, device=dev)
    out = {}
    for f in range(NFAM):
        rows = []
        for tf, src, n, k, a, per_layer in _templates(s):
            if tf != f and not (f == DECODE and tf == PREFILL):
                continue
            st = every[pre] if f == PREFILL else every[~pre] if f == DECODE else every
            m = {"T": T, "K": s.top_k * T, "R": R, "0": 0 * T}[src][st]
            if f in (GEMM, LM_HEAD):
                F, Bt, B = 2 * m * n * k, 2 * (m * k + k * n + m * n), _cd(m, 128) * _cd(n, 128)
            elif f == GROUPED:
                me = torch.from_numpy(tr.experts).to(dev)
                m = me.sum(-1)
                F, Bt = 2 * m * n * k, 2 * (m * k + (me > 0).sum(-1) * k * n + m * n)
                B = _cd(me, 128).sum(-1) * _cd(n, 128)
                st = every[:, None].expand(-1, s.layers)
            elif f in (PREFILL, DECODE):
                m, F, B = T[st], 4 * n * k * PAIRS[st], n * TILES[st]
                Bt = 2 * (2 * n * k * m + 2 * a * k * KV[st])
            else:
                F, Bt, B = {RMSNORM: lambda: (4 * m * n, 2 * (2 * m * n + n), m),
                            ROPE: lambda: (3 * m * n * k, 2 * (2 * m * n * k + m * k), m),
                            SILU: lambda: (5 * m * n, 6 * m * n, _cd(m * n, 1024)),
                            KV_WRITE: lambda: (0 * m, 8 * m * n * k, m),
                            EMBED: lambda: (0 * m, 4 * m * n + 4 * m, m)}[f]()
            kk = 0 if f in (RMSNORM, SILU, EMBED) else k
            rows.append([F, Bt, B, m, torch.full_like(m, n), torch.full_like(m, kk), st,
                         torch.full_like(m, 1 if not per_layer or f == GROUPED else s.layers)])
        if rows and rows[0][0].numel():
            out[f] = [torch.stack(c, -1).reshape(-1) for c in zip(*rows)]
            out[f].append((len(rows), rows[0][0].numel() // (s.layers if f == GROUPED else 1)))
    return out


def _eta(case, p, f, x, W):
    if case["bounded"]:
        g, a = p["bounded"][f].double()
        gamma = torch.sigmoid(x @ g)
        eta = 1.0 / (gamma - gamma * torch.sigmoid(x @ a) / W.clamp(min=1.0))
    elif case["head"] == "one":
        eta = torch.ones_like(W)
    else:
        w = {n: p[n][f].double() for n in ("w1", "w2", "b2", "w3", "b3")}
        y = torch.cat([x, x * x], -1) if case["inp"] == 32 else x
        h = torch.relu(torch.relu(y @ w["w1"].T) @ w["w2"].T + w["b2"])
        eta = 1.0 + torch.exp(-(h @ w["w3"] + w["b3"]))
    if case["grid"]:
        v = p["grid"][f].double()
        t = torch.stack([(x[..., GRID["axes"][d]] - GRID["lo"][d]) / (GRID["hi"][d] - GRID["lo"][d])
                         * (GRID["n"][d] - 1) for d in range(3)], -1)
        top = torch.tensor(GRID["n"], device=x.device) - 1
        inside = ((t >= 0) & (t <= top)).all(-1)
        i = torch.minimum(t.floor().clamp(min=0).long(), top - 1)
        fr, e = t - i, torch.zeros_like(eta)
        for c in range(8):
            bit = [(c >> d) & 1 for d in range(3)]
            wt = math.prod((fr[..., d] if bit[d] else 1.0 - fr[..., d]) for d in range(3))
            e = e + wt * v[i[..., 0] + bit[0], i[..., 1] + bit[1], i[..., 2] + bit[2]]
        eta = torch.where(inside & ~e.isnan(), e, eta)
    return eta


def _price(case, p, f, rec, sp):
    """t_roof, eta and t, [specs, records], of one family's records for the
    spec vectors sp (columns of shape [specs, 1])."""
    F, Bt, B, M, n, k = (v.double()[None, :] for v in rec[:6])
    W = torch.ceil(B / sp["n_cu"])
    u = torch.where(B > 0, W * sp["n_cu"] / B.clamp(min=1.0), torch.ones_like(W))
    tc, tm = F * u / sp["peak_flops"], Bt / sp["hbm_bw"]
    tr = torch.maximum(tc, tm)
    if case["head"] == "one" and not case["bounded"] and not case["grid"]:
        return tr, torch.ones_like(tr), torch.maximum(tr, sp["t0"])
    bt1, b1 = Bt.clamp(min=1.0), B.clamp(min=1.0)
    ai, den = F / bt1, tc + tm
    log2 = torch.log2
    x = [log2(ai.clamp(min=2.0 ** -10)) / 16, log2((ai * sp["hbm_bw"] / sp["peak_flops"]).clamp(min=2.0 ** -20)) / 16,
         log2(1 + B / sp["n_cu"]) / 16, 1 / u, log2(1 + W) / 16, (sp["l2_bytes"] / bt1).clamp(max=1.0),
         log2((tr / sp["t0"].clamp(min=1e-9)).clamp(min=2.0 ** -20)) / 16,
         torch.where(den > 0, tc / torch.where(den > 0, den, torch.ones_like(den)), torch.zeros_like(den)),
         log2(1 + F) / 64, log2(1 + Bt) / 48, log2(1 + M) / 24, log2(1 + n) / 24, log2(1 + k) / 24,
         log2(1 + F / b1) / 48, log2(1 + Bt / b1) / 40, torch.ones_like(B)]
    eta = _eta(case, p, f, torch.stack([v.expand_as(tr) for v in x], -1), W)
    return tr, eta, torch.maximum(tr * eta, sp["t0"])


def exact(case, seed):
    """run()'s outputs in 64 bits.  None for the simulation (an event loop of
    thousands of steps for each spec vector)."""
    if case["op"] == "simulate":
        return None
    tr = _trace(case, seed)
    if case["op"] == "expand":
        return None   # whole numbers: compared bit for bit
    s, S, N = tr.shape, case["steps"], case["specs"]
    specs = {k: torch.from_numpy(np.asarray(v, np.float64)).cuda() for k, v in _specs(case, seed).items()}
    p = _head(case, seed)
    recs = _records(case, tr)
    keep = {k: [] for k in ("t_roof", "eta", "t_kernel")} if case["outs"] != "sums" else None
    counts = {k: [] for k in ("flops", "bytes", "blocks")}
    body = torch.zeros(N, S, dtype=torch.float64, device="cuda")

    def spread(v, f, tpl):
        # per different record -> per record of the case's form
        if case["form"] == "layers" and f != GROUPED and recs[f][7][0] > 1:
            nt, ns = tpl
            v = v.reshape(v.shape[:-1] + (ns, 1, nt)).expand(v.shape[:-1] + (ns, s.layers, nt))
            return v.reshape(v.shape[:-3] + (-1,))
        return v

    for f, rec in recs.items():
        n, got = rec[0].numel(), {k: [] for k in keep} if keep else None
        room = max(1, int(2.5e8 / max(case["hid"], 64)))
        for s0 in range(0, N, max(1, room // n)):
            sp = {k: v[s0:s0 + max(1, room // n), None] for k, v in specs.items()}
            parts = [_price(case, p, f, [v[i:i + room] for v in rec[:6]], sp) for i in range(0, n, room)]
            tro, eta, t = (torch.cat(x, -1) for x in zip(*parts))
            # one record of a homogeneous pair of equal kernels stands for a layer's worth each
            body[s0:s0 + t.shape[0]].index_add_(1, rec[6], t * rec[7])
            if keep:
                for k, v in (("t_roof", tro), ("eta", eta), ("t_kernel", t)):
                    got[k].append(spread(v, f, rec[8]).float())
        if keep:
            for k in keep:
                keep[k].append(torch.cat(got[k], 0))
            for k, v in zip(("flops", "bytes", "blocks"), rec[:3]):
                counts[k].append(spread(v, f, rec[8]))
    out = {}
    if case["op"] != "kernels":
        off, q = torch.from_numpy(tr.req_off).cuda(), torch.from_numpy(tr.req_q).cuda()
        c = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(q, 0)])
        msg = (c[off[1:]] - c[off[:-1]]).double() * s.hidden * 2
        comm = torch.zeros_like(body)
        if s.tp > 1:
            comm = 2 * s.layers * (specs["ar_alpha0"] + specs["ar_alpha_log2p"] * math.log2(s.tp))[:, None] \
                + 2 * s.layers * 2 * (s.tp - 1) / s.tp * msg[None] / specs["ar_beta"][:, None]
        c_disp, ell, c_ovl, c_tail, scale = HOST
        gpu = scale * body + comm
        launches = torch.from_numpy(np.where(tr.prefill, s.layers, 0)).cuda().double()
        out = {"t_body": body, "t_gpu": gpu,
               "t_step": (gpu + launches * c_disp).clamp(min=ell) + (c_ovl - gpu).clamp(min=0.0) + c_tail}
    if keep:
        every = case["outs"] == "all"
        for k in ("t_roof", "eta", "t_kernel"):
            if every or k == "t_kernel":
                out[k] = torch.cat(keep[k], 1)
        if every:
            out.update({k: torch.cat(v) for k, v in counts.items()})
    return out
