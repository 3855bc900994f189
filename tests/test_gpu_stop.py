"""Where a step graph stops: after the step in which a non-finite value or a
non-positive mean depth first appears, with that step's result as the state,
whatever the graph's form and wherever in a replay of eight steps it happens.
The reference makes the same steps one call at a time, kernel by kernel, and
looks at the failure flag after each.  Runs blow up from a time step far above
the CFL bound; step multiples are scanned so that failures fall on both steps
of a pair."""
import numpy as np
import pytest

from paper_2311_11348_amd import inputs as I
from paper_2311_11348_amd import swe

pytestmark = pytest.mark.gpu

STEPS = 24


def basin(n, lo, hi):
    """Closed (no forcing, whose device clock rounds its own way), orders all hi or mostly lo."""
    prob = I.config_c3(n=n)
    prob.adapt, prob.p_base, prob.p_max = 0, lo, hi
    prob.p = np.where(np.arange(prob.mesh.ne) % 32 == 0, hi, lo).astype(np.int8)
    return prob


def fails(call):
    try:
        call()
    except swe.SweError as e:
        assert e.status == swe.SWE_ESTATE
        return True
    return False


def expected(make, c0, dt):
    """(step that fails, counted from 1, state after it), or None if STEPS steps pass."""
    with make(0) as ctx:
        ctx.set_state(c0)
        for k in range(1, STEPS + 1):
            ctx.step(1, dt)
            if fails(ctx.sync):
                return k, ctx.state()[0]
    return None


def stopped(make, c0, dt):
    with make(2) as ctx:
        ctx.set_state(c0)
        ctx.step(STEPS, dt)
        assert fails(ctx.sync)
        return ctx.state()[0]


@pytest.mark.parametrize("precision", [swe.SWE_FP64, swe.SWE_FP32_WB])
@pytest.mark.parametrize("n,p", [(12, 2), (130, 1), (150, 2)])     # roles; roles, two tiles a CU; one group of waves
def test_uniform_stop(n, p, precision):
    prob = basin(n, p, p)
    c0 = I.random_state(prob.mesh, prob.p, p, 3, prob.hb_vertex, 0.2, 0.5, 0.1)
    make = lambda graph: swe.context_for(prob, precision=precision, step_graph=graph)
    seen = set()
    for k in range(12):
        dt = prob.dt() * 3.0 * 1.35 ** k
        want = expected(make, c0, dt)
        if want is None:
            continue
        seen.add(want[0] % 2)
        assert np.array_equal(stopped(make, c0, dt), want[1], equal_nan=True), (k, want[0])
    assert seen == {0, 1}


def first_stage_passes(prob, precision, c, dt):
    """Whether c + dt L(c) is finite with a positive mean depth in every element."""
    with swe.context_for(prob, precision=precision) as ctx:
        c1 = c + dt * ctx.rhs(0.0, c)
    H = c1[:, 0, 0] / np.sqrt(prob.mesh.areas()) + prob.hb_vertex[prob.mesh.tri].mean(axis=1)
    return bool(np.all(np.isfinite(c1)) and np.all(H > 0.0))


# The order-partitioned graphs whose clock advances in the list kernel of the
# step before, while the rest of that step's last stage may still find a
# failure: each stage in one launch, and (more than 448 base blocks in FP64,
# 1,536 in FP32) its kernels on branches.  c0 of a step that first fails in its
# second stage is made by the scan over time steps.
@pytest.mark.parametrize("precision,n,lo", [(swe.SWE_FP64, 20, 1), (swe.SWE_FP32_WB, 20, 1), (swe.SWE_FP64, 20, 0),
                                            (swe.SWE_FP64, 260, 1), (swe.SWE_FP32_WB, 480, 1)])
def test_partitioned_stop(precision, n, lo):
    prob = basin(n, lo, 2)
    order = prob.p
    c0 = I.random_state(prob.mesh, prob.p, 2, 3, prob.hb_vertex, 0.2, 0.5, 0.1)

    def make(graph):
        ctx = swe.context_for(prob, precision=precision, separate=2, step_graph=graph)
        ctx.set_order(order)
        return ctx

    small = n < 100
    seen, second = set(), 0
    for k in range(16 if small else 6):
        dt = prob.dt() * (3.0 * 1.2 ** k if small else 7.0 * 1.25 ** k)
        want = expected(make, c0, dt)
        if want is None:
            continue
        step, state = want
        seen.add(step)
        with make(0) as ctx:
            ctx.set_state(c0)
            for _ in range(step - 1):
                ctx.step(1, dt)
            before = ctx.state()[0]
        second += first_stage_passes(prob, precision, before, dt)
        for _ in range(3):
            assert np.array_equal(stopped(make, c0, dt), state, equal_nan=True), (k, step)
    assert len(seen) > 1 and second > 0
