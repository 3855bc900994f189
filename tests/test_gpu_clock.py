"""The step clock of a static order-partitioned graph, advanced by the last
list kernel of the step before: graph replays (of eight steps and of one, over
two calls) against kernel-by-kernel launches, whose stage times come from the
host, on a forced open sea (a clock that is a step off moves the forcing, and
with it the whole surface, by far more than rounding)."""
import numpy as np
import pytest

from paper_2311_11348_amd import inputs as I
from paper_2311_11348_amd import swe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,bound", [(swe.SWE_FP64, 1e-12), (swe.SWE_FP32_WB, 1e-5)])
@pytest.mark.parametrize("n", [6, 40])
def test_static_partitioned_clock(precision, bound, n):
    """bound: the oracle tests' FP64 and FP32 elevation tolerances."""
    prob = I.config_c2(n=n, p=2)
    order = np.ones(prob.mesh.ne, dtype=np.int8)
    order[::16] = 2
    out = []
    for graph in (1, 0):
        with swe.context_for(prob, precision=precision, separate=2, step_graph=graph) as ctx:
            ctx.set_order(order)
            ctx.set_state_fn(prob.ic)
            dt = prob.dt()
            for steps in (11, 16, 1):
                ctx.step(steps, dt)
            ctx.sync()
            c, t = ctx.state()
            out.append((c[:, 0], t))
    (a, ta), (b, tb) = out
    assert ta == tb
    assert np.linalg.norm(b) > 0
    assert np.linalg.norm(a - b) <= bound * np.linalg.norm(b)
