"""The one-launch order-partitioned stage and the separated step as a chain,
which step graphs of small meshes take, against kernel-by-kernel launches
(which do not): equal bit for bit, for static and re-chosen orders, with and
without open edges, at element counts around the 256-element blocks and on a
mesh beyond the one-launch limit; the base order 2 form against the oracle."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2311_11348_amd import inputs as I
from paper_2311_11348_amd import swe

pytestmark = pytest.mark.gpu


def problem(n, lo, hi, adapt, tidal):
    prob = I.config_c2(n=n, p=hi, seed=n) if tidal else I.config_c3(n=n)
    prob.p_base, prob.p_max = lo, hi
    prob.adapt = 1 if adapt else 0
    prob.adapt_tau = 1e-3
    prob.p = (np.full(prob.mesh.ne, lo) if adapt else np.random.default_rng(n).integers(lo, hi + 1, prob.mesh.ne)
              * (np.arange(prob.mesh.ne) % 7 == 0)).clip(lo, hi).astype(np.int8)
    return prob


CASES = [(2, 1, 2, False, True), (11, 1, 2, False, True), (12, 1, 3, False, False), (16, 2, 3, False, True),
         (23, 1, 3, True, False), (24, 1, 2, True, True), (17, 2, 3, True, False), (250, 1, 2, False, False)]


@pytest.mark.parametrize("separate", [1, 2])
@pytest.mark.parametrize("precision", [swe.SWE_FP64, swe.SWE_FP32_WB])
@pytest.mark.parametrize("n,lo,hi,adapt,tidal", CASES)
def test_graph_equals_launches(n, lo, hi, adapt, tidal, precision, separate):
    if precision == swe.SWE_FP32_WB and separate == 2 and hi == 3:
        pytest.skip("FP32 order-partitioned stepping with p_max = 3 is switched off")
    prob = problem(n, lo, hi, adapt, tidal)
    c0 = I.random_state(prob.mesh, prob.p, hi, 3, prob.hb_vertex, 0.2, 0.5, 0.1)
    dt, steps, got = prob.dt(), 9, []
    for graph in (2, 0):
        with swe.context_for(prob, precision=precision, separate=separate, step_graph=graph) as ctx:
            ctx.set_state(c0)
            ctx.step(steps, dt)
            ctx.sync()
            got.append((ctx.state()[0], ctx.order()))
    assert np.array_equal(got[0][1], got[1][1])
    assert np.array_equal(got[0][0], got[1][0])
    if n == 16 and precision == swe.SWE_FP64:
        ref = Oracle.from_problem(prob).step(c0, steps, dt)
        assert np.linalg.norm(got[0][0] - ref) <= 1e-12 * np.linalg.norm(ref)
