"""Which kernels a call takes must not show in its results (GPU): calls on both
sides of the rules that choose them, against closed forms and the float64
definition."""
import numpy as np
import pytest

from paper_2606_28565_amd import abi
from tests import gpu_helpers as g
from tests.helpers import make_desc, steprec
from workload import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_steps,per_step,n_specs", [(1, 3, 1), (1, 65537, 1), (64, 5, 1024), (64, 1024, 2), (64, 1025, 2),
                                                      (64, 5, 1025), (65, 126, 2), (65, 127, 2), (128, 64, 2), (128, 65, 2),
                                                      (129, 2, 2)])
def test_request_sums_around_the_prologue_rule(n_steps, per_step, n_specs):
    """The flag reset, spec constants and request sums in one launch or in
    several: attention's counts are whole numbers of the request sums."""
    rng = np.random.Generator(np.random.PCG64(n_steps * per_step))
    q = rng.integers(1, 300, (n_steps, per_step))
    h = rng.integers(0, 4000, (n_steps, per_step))
    H, Hkv, d = 8, 2, 64
    desc = make_desc([(gen.ATTN_DECODE, j, 0, H, d, Hkv, 0) for j in range(n_steps)],
                     [list(zip(q[j], h[j])) for j in range(n_steps)])
    wl = gen.Workload("prologue", desc, steprec(n_steps), gen.specs_grid(n_specs, 3), gen.make_heads(16, 64, "f32"),
                      gen.HostConsts())
    out = g.eval_kernels(wl, eta_one=True)
    pairs = (q * h + q * (q + 1) // 2).sum(1)
    np.testing.assert_array_equal(out["flops"], 4 * H * d * pairs)
    np.testing.assert_array_equal(out["bytes"], 2 * (2 * H * d * q.sum(1) + 2 * Hkv * d * (q + h).sum(1)))
    np.testing.assert_array_equal(out["blocks"], H * ((q + 127) // 128).sum(1))
    sp = wl.specs
    B, N = out["blocks"].astype(np.int64)[None], sp["n_cu"].astype(np.int64)[:, None]
    u = ((B + N - 1) // N * N) / B
    t = np.maximum(np.maximum(out["flops"][None] * u / sp["peak_flops"][:, None], out["bytes"][None] / sp["hbm_bw"][:, None]),
                   sp["t0"][:, None])
    assert g.rel_err(out["t_kernel"], t).max() <= 1e-5


def _steps(wl, room, pairs=False, n_specs=None):
    """Step sums (and t_kernel), the device status and, with room, the families whose
    different records did not fit (a flag each, from word 16 after the record ranges)."""
    import torch
    di = abi.DeviceInputs(wl, n_specs=n_specs)
    up = lambda x: -(-x // 256) * 256
    S, N = wl.desc.n_steps, di.n_specs
    ctl = 256 + up(64 * N) + up(32 * S) + up(80 * S)
    tiles = sum(-(-int(k) // 64) for k in np.diff(wl.desc.fam_off))
    small = ctl + up(80 * N * S) + up(8 * N * tiles)
    assert not room or small < di.ws_bytes
    so_t, so = abi.step_outputs(S, N)
    ko_t, ko = abi.kernel_outputs(wl.desc.n_rows, N, counts=False, t_roof=False, eta=False) if pairs else ({}, None)
    abi.ks_eval_steps(di.desc, di.steps, di.specs_ptr, N, di.heads, di.host, so, ko, di.ws_ptr,
                      di.ws_bytes if room else small, abi.current_stream())
    torch.cuda.synchronize()
    st = abi.ks_device_status(di.ws_ptr, di.ws_bytes, abi.current_stream(), check=False)
    o = ctl + di.ws_ptr - di.ws.data_ptr() + 64
    over = di.ws[o:o + 4 * gen.NFAM].view(torch.int32).cpu().numpy()
    return {k: v.cpu().numpy() for k, v in (so_t | ko_t).items()}, st, [f for f in range(gen.NFAM) if over[f]]


def _layers(kernels, layers, n_steps, odd_step=None):
    """Steps of `layers` repeats of `kernels` GEMMs (one step without repeats),
    norms that repeat and grouped-free rest."""
    rows = []
    for j in range(n_steps):
        m = 3 + 7 * (j % 50)
        n = kernels * layers
        rows += [(gen.GEMM, j, m, 64 * (1 + (i if j == odd_step else i % kernels)), 256, 0, 0) for i in range(n)]
        rows += [(gen.RMSNORM, j, m, 4096, 0, 0, 0)] * (2 * layers) + [(gen.LM_HEAD, j, 1 + j % 9, 32000, 4096, 0, 0)]
    return rows


@pytest.mark.parametrize("precision,in_dim,hidden", [("bf16", 16, 128), ("bf16", 32, 256), ("f32", 32, 128)])
@pytest.mark.parametrize("kernels,layers,odd,over", [(4, 3, None, []), (3, 3, None, []), (4, 4, None, []), (4, 5, None, []),
                                                     (5, 3, None, [gen.GEMM]), (5, 40, None, [gen.GEMM]), (4, 40, None, []),
                                                     (4, 8, 77, []), (4, 60, 77, [gen.GEMM])])
def test_a_family_that_does_not_fit_leaves_the_others(precision, in_dim, hidden, kernels, layers, odd, over):
    """Up to four kernels per layer fit at any number of layers (three layers of
    four are twelve records per step, three entries per eight records); a family of
    five, or with a long step without repeats, is evaluated record by record, and
    only that one.  One step without repeats fits where its entries do (32 here,
    28 more than four).  The reference evaluates every record: fp32 sums within 64-record tiles
    (6 levels of adds) against float64 ones: 6 2^-24."""
    n_steps = max(600, 9000 // (kernels * layers))
    rows = _layers(kernels, layers, n_steps, odd)
    n_specs = 24 if precision == "f32" else 160
    wl = gen.Workload("layers", make_desc(rows, [[(1 + j % 7, 5)] for j in range(n_steps)]), steprec(n_steps),
                      gen.specs_grid(n_specs, 5), gen.make_heads(in_dim, hidden, precision), gen.HostConsts())
    ref, _, _ = _steps(wl, False)
    got, st, seen = _steps(wl, True)
    assert st == abi.KS_OK and seen == over
    for k in ref:
        np.testing.assert_allclose(got[k], ref[k], rtol=6 * 2.0 ** -24)
    again, _, _ = _steps(wl, True)
    for k in got:
        np.testing.assert_array_equal(again[k], got[k])


def test_bad_steps_of_one_family_with_per_pair_outputs():
    """Per-pair outputs of records whose step is out of range come from evaluating
    every record of their family; the other families' are spread from the different
    ones.  Both as every record's evaluation gives them."""
    n_steps = 300
    rows = _layers(4, 20, n_steps)
    rows += [(gen.ROPE, j, 3 + j % 50, 8, 128, 0, 0) for j in range(n_steps) for _ in range(20)]
    rows += [(gen.ROPE, n_steps + i, 3 + i % 5, 8, 128, 0, 0) for i in range(2000)]
    wl = gen.Workload("bad", make_desc(rows, [[(1 + j % 7, 5)] for j in range(n_steps)]), steprec(n_steps),
                      gen.specs_grid(200, 5), gen.make_heads(16, 128, "bf16"), gen.HostConsts())
    ref, st, _ = _steps(wl, False, True)
    assert st == abi.KS_EINVAL
    got, st, seen = _steps(wl, True, True)
    assert st == abi.KS_EINVAL and seen == [gen.ROPE]
    np.testing.assert_array_equal(got["t_kernel"], ref["t_kernel"])
    for k in ("t_body", "t_gpu", "t_step"):   # fp32 within 64-record tiles: 6 levels of adds
        np.testing.assert_allclose(got[k], ref[k], rtol=6 * 2.0 ** -24)


@pytest.mark.parametrize("precision,in_dim,hidden", [("f32", 32, 128), ("bf16", 32, 256), ("bf16", 16, 64)])
@pytest.mark.parametrize("tiles", [250, 290, 700, 1100])
def test_spec_ranges_of_tiles_that_fill_the_grid(precision, in_dim, hidden, tiles):
    """Every record evaluated, the spec vectors in one range or several: a spec's
    outputs are those of a call with that spec alone, bit for bit."""
    n_steps = tiles * 256 // 32
    rows = [(gen.SILU_MUL, j, 1 + j % 900, 64 * (1 + i % 3), 0, 0, 0) for j in range(n_steps) for i in range(32)]
    wl = gen.Workload("ranges", make_desc(rows, [[(1, 5)]] * n_steps), steprec(n_steps), gen.specs_grid(16, 5),
                      gen.make_heads(in_dim, hidden, precision), gen.HostConsts())
    got, st, _ = _steps(wl, False, True)
    one, _, _ = _steps(wl, False, True, n_specs=1)
    two, _, _ = _steps(wl, False, True, n_specs=2)
    assert st == abi.KS_OK
    for k in got:
        np.testing.assert_array_equal(got[k][:1], one[k])
        np.testing.assert_array_equal(got[k][:2], two[k])


@pytest.mark.parametrize("precision,in_dim,hidden,n_specs", [("bf16", 16, 128, 400), ("bf16", 32, 256, 120), ("f32", 32, 128, 120)])
def test_collapsed_mixture_of_experts(precision, in_dim, hidden, n_specs):
    """A mixture of experts with its layers collapsed: one record of multiplicity 16
    per layer-identical kernel, the grouped GEMMs one per layer, evaluated every one
    beside the different ones of the rest (fp32 sums within 64-record tiles: 6
    2^-24)."""
    rng = np.random.Generator(np.random.PCG64(12))
    L, n_steps, rows, experts = 16, 420, [], []
    for j in range(n_steps):
        m = int(rng.integers(1, 40))
        for n in (6144, 4096, 8):
            rows.append((gen.GEMM, j, m, n, 4096, 0, 0))
        for _ in range(L):
            for n, k in ((28672, 4096), (4096, 14336)):
                rows.append((gen.GROUPED_GEMM, j, 0, n, k, 8, len(experts)))
            experts += [int(x) for x in rng.integers(0, 12, 8)]
        rows += [(gen.RMSNORM, j, m, 4096, 0, 0, 0)] * 2 + [(gen.SILU_MUL, j, 2 * m, 14336, 0, 0, 0),
                                                            (gen.ATTN_DECODE, j, 0, 32, 128, 8, 0),
                                                            (gen.LM_HEAD, j, m, 32000, 4096, 0, 0)]
    d = make_desc(rows, [[(1, int(h)) for h in rng.integers(0, 4000, 3)] for _ in range(n_steps)], experts)
    d.mult = np.where(np.isin(d.family(), (gen.GROUPED_GEMM, gen.LM_HEAD)), 1, L).astype(np.uint32)
    wl = gen.Workload("moe", d, steprec(n_steps, layers=L, hidden=4096, tp=2), gen.specs_grid(n_specs, 5),
                      gen.make_heads(in_dim, hidden, precision), gen.HostConsts())
    di = abi.DeviceInputs(wl)
    taken = abi.ks_different_families(di.desc, n_specs, di.heads, None, di.ws_bytes)
    assert taken == sum(1 << f for f in np.unique(d.family()) if f != gen.GROUPED_GEMM)
    ref, _, _ = _steps(wl, False, True)
    got, st, seen = _steps(wl, True)
    assert st == abi.KS_OK and seen == []
    w = d.mult.astype(np.float64)
    for s in range(n_specs):
        body = np.bincount(d.step, weights=ref["t_kernel"][s].astype(np.float64) * w, minlength=n_steps)
        np.testing.assert_allclose(got["t_body"][s], body, rtol=6 * 2.0 ** -24)
    for k in ("t_gpu", "t_step"):
        np.testing.assert_allclose(got[k], ref[k], rtol=12 * 2.0 ** -24)
