"""The different records of a call (GPU): calls with enough head work evaluate
equal records once, weight them in the step sums and spread their per-pair
values.  The reference is the same call in a workspace with no room for that,
which evaluates every record.  Both form the same fp32 values for a record, so
per-pair outputs are equal bit for bit; the step sums are compared with the
float64 sum of the reference's t_kernel: the weights (counts times
multiplicities below 2^24) are exact in fp32, so only the order of the float64
sums differs, and with at most 4096 non-negative terms a step that is within
4096 2^-53 < 1e-12."""
import numpy as np
import pytest

from paper_2606_28565_amd import abi
from tests.helpers import make_desc, steprec
from workload import gen

pytestmark = pytest.mark.gpu
TOL = 1e-12


def _wl(rows, reqs, heads, n_specs, mult=None, expert_rows=()):
    d = make_desc(rows, reqs, expert_rows)
    if mult is not None:
        d.mult = np.asarray(mult(d.n_rows), np.uint32)
    return gen.Workload("unique", d, steprec(len(reqs), layers=3, hidden=4096, tp=2, n_launch=1),
                        gen.specs_grid(n_specs, 77), heads, gen.HostConsts())


def _every_record_bytes(wl):
    """The workspace of a call that evaluates every record."""
    up = lambda x: -(-x // 256) * 256
    S, N = wl.desc.n_steps, wl.n_specs
    tiles = sum(-(-int(k) // 64) for k in np.diff(wl.desc.fam_off))
    return 256 + up(64 * N) + up(32 * S) + up(80 * S) + up(80 * N * S) + up(8 * N * tiles)


def _run(wl, room, outs=False, steps=True, grid=None, bounded=None):
    """outs: every per-pair output and the counts (False: none; "pairs": no
    counts).  room: whether the different records have room."""
    import torch
    di = abi.DeviceInputs(wl)
    small = _every_record_bytes(wl)
    assert small < di.ws_bytes
    wsb = di.ws_bytes if room else small
    heads = di.make_heads(wl.heads.precision, wl.heads.in_dim, wl.heads.hidden, abi.KS_ETA_MLP, bounded, grid)
    so_t, so = abi.step_outputs(wl.desc.n_steps, di.n_specs)
    ko_t, ko = abi.kernel_outputs(wl.desc.n_rows, di.n_specs, counts=outs is True) if outs else ({}, None)
    for t in list(so_t.values()) + list(ko_t.values()):
        t.fill_(-1)
    if steps:
        abi.ks_eval_steps(di.desc, di.steps, di.specs_ptr, di.n_specs, heads, di.host, so, ko, di.ws_ptr, wsb,
                          abi.current_stream())
    else:
        abi.ks_eval_kernels(di.desc, di.specs_ptr, di.n_specs, heads, ko, di.ws_ptr, wsb, abi.current_stream())
    torch.cuda.synchronize()
    status = abi.ks_device_status(di.ws_ptr, wsb, abi.current_stream(), check=False)
    got = {k: v.cpu().numpy() for k, v in (list(so_t.items()) if steps else []) + list(ko_t.items())}
    return got, status


def _check(wl, grid=None, tol=TOL, bounded=None):
    ref, _ = _run(wl, False, "pairs", grid=grid, bounded=bounded)
    sums, st = _run(wl, True, grid=grid, bounded=bounded)
    assert st == abi.KS_OK
    d = wl.desc
    w = np.ones(d.n_rows) if getattr(d, "mult", None) is None else d.mult.astype(np.float64)
    for s in range(wl.n_specs):
        body = np.bincount(d.step, weights=ref["t_kernel"][s].astype(np.float64) * w, minlength=d.n_steps)
        np.testing.assert_allclose(sums["t_body"][s], body, rtol=tol)
    for k in ("t_gpu", "t_step"):   # the other path's sums are fp32 within 64-record tiles
        np.testing.assert_allclose(sums[k], ref[k], rtol=1e-6)
    for outs, steps in (("pairs", True), (True, False)):
        every, _ = _run(wl, False, outs, steps, grid, bounded)
        got, _ = _run(wl, True, outs, steps, grid, bounded)
        for k in every:
            if k.startswith("t_") and k not in ("t_roof", "t_kernel"):
                np.testing.assert_allclose(got[k], sums[k], rtol=tol)
            else:
                np.testing.assert_array_equal(got[k], every[k], err_msg=k)


def _reqs(rng, n):
    return [[(int(rng.integers(1, 300)), int(rng.integers(0, 4000))) for _ in range(int(rng.integers(1, 4)))]
            for _ in range(n)]


def _family(rng, f, step, kernels, layers):
    """`layers` repeats of `kernels` different records of family f."""
    m = [int(x) for x in rng.integers(1, 3000, kernels)]
    n = [int(x) for x in rng.integers(1, 200, kernels)]
    return [(f, step, m[i], n[i], 128, 4, 0) for _ in range(layers) for i in range(kernels)]


@pytest.mark.parametrize("kernels", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("layers", [1, 7, 80])
def test_layers_repeat(kernels, layers):
    """Periods 1 to 4 and none (5), pieces that start anywhere in a chunk and
    cross its end, odd family offsets, steps without a family.  More than eight
    records per step without a period do not fit and are all evaluated, their
    sums fp32 within 64-record tiles: at most 6 levels of adds, 6 2^-24."""
    rng = np.random.Generator(np.random.PCG64(kernels * 100 + layers))
    n_steps = max(37, 9000 // (kernels * layers * 3))
    fams = (gen.GEMM, gen.ATTN_DECODE, gen.RMSNORM)
    rows = []
    for j in range(n_steps):
        for f in fams:
            if rng.random() < 0.9:
                rows += _family(rng, f, j, kernels, layers if rng.random() < 0.8 else layers + 1)
    wl = _wl(rows, _reqs(rng, n_steps), gen.make_heads(16, 128, "bf16"), 270)
    _check(wl, tol=6 * 2.0 ** -24 if kernels == 5 and layers > 1 else TOL)


@pytest.mark.parametrize("run", [1, 1023, 1024, 1025, 3000])
def test_one_long_step_and_chunk_edges(run):
    """A step of `run` equal records among steps of one: pieces that end at,
    before and after a chunk's edge, and steps that span several chunks."""
    rng = np.random.Generator(np.random.PCG64(run))
    rows = [(gen.ROPE, 0, 17, 8, 128, 0, 0)]
    rows += [(gen.ROPE, 1, 33, 8, 128, 0, 0)] * run
    rows += [(gen.ROPE, 2 + i, int(rng.integers(1, 64)), 8, 128, 0, 0) for i in range(2100)]
    wl = _wl(rows, _reqs(rng, 2102), gen.make_heads(32, 64, "f32"), 370)
    _check(wl)


@pytest.mark.parametrize("precision,in_dim,hidden,n_specs", [("f32", 16, 64, 120), ("bf16", 32, 256, 72),
                                                             ("bf16", 16, 64, 1000)])
def test_multiplicities_and_shared_slots(precision, in_dim, hidden, n_specs):
    """Multiplicities (equal records with different ones stay apart), and token
    counts a table's size apart, which meet in one slot."""
    rng = np.random.Generator(np.random.PCG64(5))
    rows = []
    for j in range(600):
        for m in (3, 3 + (1 << 15), 3 + (1 << 18), int(rng.integers(1, 9))):
            rows += [(gen.LM_HEAD, j, m, 1000, 4096, 0, 0), (gen.GEMM, j, m, 96, 4096, 0, 0),
                     (gen.GEMM, j, m, 97, 4096, 0, 0)]
    wl = _wl(rows, _reqs(rng, 600), gen.make_heads(in_dim, hidden, precision), n_specs,
             mult=lambda n: rng.integers(0, 3, n) * 40)
    _check(wl)


def test_records_that_do_not_repeat_fall_back():
    """Many records per step, none equal: more entries than there is room for,
    so every record is evaluated; beside a family that repeats."""
    rng = np.random.Generator(np.random.PCG64(6))
    rows = []
    for j in range(24):
        rows += [(gen.GEMM, j, 1 + i + 200 * j, 512, 256, 0, 0) for i in range(200)]
        rows += [(gen.RMSNORM, j, 5 + j, 4096, 0, 0, 0)] * 64
    wl = _wl(rows, _reqs(rng, 24), gen.make_heads(16, 128, "bf16"), 320)
    for outs in (False, "pairs", True):
        ref, _ = _run(wl, False, outs)
        got, st = _run(wl, True, outs)
        assert st == abi.KS_OK
        for k in ref:   # both evaluate every record, alike
            np.testing.assert_array_equal(got[k], ref[k], err_msg=k)


@pytest.mark.parametrize("grids", [False, True])
def test_grouped_gemms_and_grids(grids):
    """Grouped GEMMs keep a record per layer (summed in fp32 within 64-record
    tiles: 6 2^-24) beside families that repeat; with and without measured
    grids."""
    rng = np.random.Generator(np.random.PCG64(7))
    rows, experts = [], []
    for j in range(40):
        for layer in range(16):
            rows += [(gen.GROUPED_GEMM, j, 0, 28672, 4096, 8, len(experts)),
                     (gen.GROUPED_GEMM, j, 0, 4096, 14336, 8, len(experts))]
            experts += [int(x) for x in rng.integers(0, 300, 8)]
        rows += _family(rng, gen.GEMM, j, 3, 16) + _family(rng, gen.SILU_MUL, j, 1, 16)
    wl = _wl(rows, _reqs(rng, 40), gen.make_heads(16, 128, "bf16"), 520, expert_rows=experts)
    _check(wl, grid=gen.make_grid(gen.GRID_ALL) if grids else None, tol=6 * 2.0 ** -24)


def test_bad_steps_are_skipped_and_reported():
    """Records whose step is out of range are left out of the sums and flagged;
    with per-pair outputs every record is evaluated, those too."""
    rng = np.random.Generator(np.random.PCG64(8))
    rows = [(gen.ROPE, j, 1 + j % 50, 8, 128, 0, 0) for j in range(4000)]
    good = _wl(rows, _reqs(rng, 4000), gen.make_heads(16, 128, "bf16"), 360)
    bad = _wl(rows + [(gen.ROPE, 4000 + i, 3, 8, 128, 0, 0) for i in range(1500)], [[(1, 1)]] * 4000,
              gen.make_heads(16, 128, "bf16"), 360)
    bad.desc.req_off, bad.desc.req_q, bad.desc.req_h = good.desc.req_off, good.desc.req_q, good.desc.req_h
    ref, _ = _run(good, True)
    for outs, tol in ((False, TOL), ("pairs", 6 * 2.0 ** -24), (True, 6 * 2.0 ** -24)):
        got, st = _run(bad, True, outs)
        assert st == abi.KS_EINVAL
        for k in ("t_body", "t_gpu", "t_step"):
            np.testing.assert_allclose(got[k], ref[k], rtol=tol)
        if outs:
            every, _ = _run(bad, False, outs)
            for k in every:
                np.testing.assert_array_equal(got[k], every[k], err_msg=k)


@pytest.mark.parametrize("n_specs", [1, 2, 3, 4, 5, 16, 33])
def test_step_sums_by_spec_count(n_specs):
    """The step sums' kernels: up to four specs, more, a tile's remainder."""
    rng = np.random.Generator(np.random.PCG64(9))
    rows = []
    n_steps = 6000 // n_specs + 50
    for j in range(n_steps):
        rows += _family(rng, gen.GEMM, j, 4, 20) + [(gen.ATTN_DECODE, j, 0, 32, 128, 8, 0)] * 20
        rows += [(gen.LM_HEAD, j, 1 + j % 64, 32000, 4096, 0, 0)]
    _check(_wl(rows, _reqs(rng, n_steps), gen.make_heads(32, 128, "f32"), n_specs))


def _trace_wl(n_steps, n_specs):
    rng = np.random.Generator(np.random.PCG64(10))
    rows = []
    for j in range(n_steps):
        rows += _family(rng, gen.GEMM, j, 4, 16) + [(gen.ATTN_DECODE, j, 0, 32, 128, 8, 0)] * 16
        rows += [(gen.RMSNORM, j, 1 + j % 40, 4096, 0, 0, 0)] * 32
    return _wl(rows, _reqs(rng, n_steps), gen.make_heads(16, 128, "bf16"), n_specs)


@pytest.mark.parametrize("bounded", [False, True])
@pytest.mark.parametrize("kind", ["dense", "moe"])
def test_whole_traces(kind, bounded):
    """Every family (KV writes among them), prefill and decode steps; with some
    families on the bounded head.  The mixture of experts' grouped GEMMs are
    summed in fp32 within 64-record tiles (6 2^-24)."""
    import dataclasses
    shape = dataclasses.replace(gen.MIXTRAL if kind == "moe" else gen.LLAMA7B, kv_write=True)
    tr = gen.trace_uniform(shape, 60, 11)
    if kind == "moe":
        tr.experts = gen.route_tokens(tr, 12)
    desc, rec = gen.build([tr])
    wl = gen.Workload("trace", desc, rec, gen.specs_grid(130, 78), gen.make_heads(16, 128, "bf16"), gen.HostConsts())
    _check(wl, tol=6 * 2.0 ** -24 if kind == "moe" else TOL,
           bounded=gen.make_bounded(gen.BOUNDED_MIXED) if bounded else None)


def test_static_entry_at_its_limit():
    """A call whose workspace fits the fixed array only without the different
    records' part is accepted, and evaluates every record."""
    import torch
    wl = _trace_wl(600, 700)
    di = abi.DeviceInputs(wl)
    assert _every_record_bytes(wl) <= abi.KS_STATIC_SCRATCH_BYTES < di.ws_bytes
    so_t, so = abi.step_outputs(600, 700)
    flags = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    abi.ks_eval_steps_static(di.desc, di.steps, di.specs_ptr, di.n_specs, di.heads, di.host, so, None,
                             flags.data_ptr(), abi.current_stream())
    torch.cuda.synchronize()
    ref, _ = _run(wl, False)
    assert int(flags.item()) == 0
    for k in ref:
        np.testing.assert_array_equal(so_t[k].cpu().numpy(), ref[k], err_msg=k)


def test_graph_replays():
    """Captured into a graph and replayed on changed inputs, with eager calls in
    the same workspace between the replays: every replay equals the eager call."""
    import torch
    wl = _trace_wl(300, 300)
    di = abi.DeviceInputs(wl)
    so_t, so = abi.step_outputs(300, 300)
    eo_t, eo = abi.step_outputs(300, 300)

    def call(out):
        abi.ks_eval_steps(di.desc, di.steps, di.specs_ptr, di.n_specs, di.heads, di.host, out, None, di.ws_ptr,
                          di.ws_bytes, abi.current_stream())

    call(so)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(so)
    m = di.t["m"].clone()
    for i in range(4):
        di.t["m"].copy_(m + 37 * i * (torch.arange(len(m), device=m.device) // 64 % 3 == 0))
        for t in so_t.values():
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = {k: v.clone() for k, v in so_t.items()}
        call(eo)
        torch.cuda.synchronize()
        for k in got:
            assert torch.equal(got[k], eo_t[k]), (i, k)
