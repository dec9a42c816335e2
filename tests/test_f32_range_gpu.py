"""fp32 heads over the whole range of fp32 (GPU): weights and activations near
its top, infinities and NaN give what fp32 arithmetic gives (a sum past the
largest value is infinite, relu(NaN) = max(NaN, 0) = 0 as IEEE's maxNum has it),
though the heads run on bfloat16 pieces, which hold less."""
import dataclasses

import numpy as np
import pytest

from oracle import ks_oracle as o
from tests import gpu_helpers as g
from workload import gen

pytestmark = pytest.mark.gpu
KINDS = [(16, 64), (32, 64), (16, 128), (32, 128)]
TOP = float(np.finfo(np.float32).max)


def _f32(v):
    """Past the largest fp32 value: infinity."""
    return np.where(np.abs(v) > TOP, np.sign(v) * np.inf, v)


def _eta(x, s, f):
    w1, w2, b2, w3 = (s[k][f].astype(np.float64) for k in ("w1", "w2", "b2", "w3"))
    with np.errstate(all="ignore"):
        h1 = np.fmax(_f32(x @ w1.T), 0.0)
        h2 = np.fmax(_f32(h1 @ w2.T + b2), 0.0)
        z = _f32(h2 @ w3 + float(s["b3"][f]))
        return 1.0 + np.exp(-z), np.abs(h2 * w3).sum(-1)


def _top(s, f, I):          # 3.4e38 is above the largest bfloat16 and below the largest fp32 value
    s["w1"][f][0] = 0.0
    s["w1"][f][0, 15] = 3.4e38
    s["w2"][f][:, 0] = np.where(s["w2"][f][:, 0] < 0, -1, 1) * np.float32(2.0 ** -125)


def _overflow(s, f, I):     # h1[0] past fp32; z = +inf, then -inf in odd families
    s["w1"][f][0] = 0.0
    s["w1"][f][0, 8] = s["w1"][f][0, 15] = 3.3e38
    s["w1"][f][0, 9] = 3.3e38
    s["w2"][f][:, 0] = np.where(s["w2"][f][:, 0] < 0, -1, 1) * np.float32(2.0 ** -125)
    s["w3"][f] = np.abs(s["w3"][f]) * (-1 if f % 2 else 1)


def _infinite(s, f, I):     # +-inf times an active unit, and times one that never is
    s["w1"][f][5, 15], s["w1"][f][6, 15] = 50.0, -50.0
    s["w2"][f][3, 5], s["w2"][f][4, 5], s["w2"][f][7, 6] = np.inf, -np.inf, np.inf
    s["w3"][f] = np.abs(s["w3"][f])


def _infinite_dropped(s, f, I):
    s["w1"][f][6, 15] = -50.0
    s["w2"][f][7, 6] = np.inf


def _nan(s, f, I):
    s["w1"][f][9, 2] = np.nan
    s["w2"][f][12, 3] = -np.float32(np.nan)
    s["b2"][f][11] = np.nan


def _bias(s, f, I):
    s["b2"][f][2] = 3.4e38
    s["w3"][f][2] = np.float32(2.0 ** -125)


def _small(s, f, I):
    s["w2"][f][1] *= np.float32(2.0 ** -116)
    s["b2"][f][1] = 0.0
    s["w3"][f][1] *= np.float32(2.0 ** 116)


@pytest.mark.parametrize("in_dim,hidden", KINDS)
@pytest.mark.parametrize("change", [_top, _overflow, _infinite, _infinite_dropped, _nan, _bias, _small])
def test_weights_and_activations_of_any_size(in_dim, hidden, change):
    wl = gen.config1(0, 3).with_heads(gen.make_heads(in_dim, hidden, "f32"))
    ref = o.eval_kernels(wl.desc, wl.specs, wl.heads, keep_features=True)
    plain = g.eval_steps(wl, counts=False)
    stor = {k: v.copy() for k, v in wl.heads.storage.items()}
    changed = (gen.GEMM, gen.ATTN_DECODE, gen.RMSNORM)
    for f in changed:
        change(stor, f, in_dim)
    got = g.eval_steps(wl.with_heads(dataclasses.replace(wl.heads, storage=stor)), counts=False)
    fam = wl.desc.family()
    other = ~np.isin(fam, changed)
    for k in ("eta", "t_kernel"):   # the other families' heads are as they were
        np.testing.assert_array_equal(got[k][:, other], plain[k][:, other])
    for f in changed:
        sel = fam == f
        assert sel.any()
        eta, terms = _eta(ref["x"][:, sel], stor, f)
        e = got["eta"][:, sel].astype(np.float64)
        assert not np.isnan(e).any()
        np.testing.assert_array_equal(np.isinf(e), eta > TOP)
        fin = np.isfinite(e)
        # z is a sum of terms each within 1e-5 of its size
        tol = 1e-5 * (1.0 + terms[fin])
        assert (np.abs(e[fin] - eta[fin]) <= tol * eta[fin]).all()
        t = np.maximum(ref["t_roof"][:, sel][fin] * eta[fin], np.broadcast_to(wl.specs["t0"][:, None], e.shape)[fin])
        assert (np.abs(got["t_kernel"][:, sel][fin] - t) <= 2 * tol * t).all()
        assert np.isposinf(got["t_kernel"][:, sel][~fin]).all()


@pytest.mark.parametrize("in_dim,hidden", KINDS)
def test_roofline_past_fp32(in_dim, hidden):
    """A spec whose t_roof is past fp32: its features are infinite and NaN, every
    unit of the first layer max(NaN, 0) = 0, eta the bias terms' and t infinite;
    the other spec's outputs are those without it."""
    wl = gen.config1(0, 3).with_heads(gen.make_heads(in_dim, hidden, "f32"))
    specs = {k: v.copy() for k, v in wl.specs.items()}
    specs["peak_flops"][1] = 1e-290
    plain = g.eval_steps(wl, counts=False)
    got = g.eval_steps(dataclasses.replace(wl, specs=specs), counts=False)
    for k in got:
        np.testing.assert_array_equal(got[k][0], plain[k][0])
    fam = wl.desc.family()
    s = wl.heads.storage
    for f in np.unique(fam):
        if f in (gen.KV_WRITE, gen.EMBED):   # no FLOPs
            continue
        h2 = np.maximum(s["b2"][f].astype(np.float64), 0.0)
        eta = 1.0 + np.exp(-(h2 @ s["w3"][f].astype(np.float64) + s["b3"][f]))
        assert g.rel_err(got["eta"][1, fam == f], eta).max() <= 1e-5
        assert np.isposinf(got["t_kernel"][1, fam == f]).all()
