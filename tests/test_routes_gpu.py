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
