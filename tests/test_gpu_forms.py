"""Which form a several-step call takes, on both sides of each switch, and the
forms that small meshes never take: step graphs with branches, over several
replays, on a forced open sea against kernel-by-kernel launches (whose stage
times come from the host)."""
import numpy as np
import pytest

from paper_2311_11348_amd import inputs as I
from paper_2311_11348_amd import swe
from tests.test_gpu_transfer import strip

pytestmark = pytest.mark.gpu

F64, F32 = swe.SWE_FP64, swe.SWE_FP32_WB
S, T, R = swe.FORM_STAGES, swe.FORM_STEP, swe.FORM_STEP_ROLES


def isolated():
    k = np.arange(400)
    x, y = (k % 20) * 300.0, (k // 20) * 300.0
    vxy = np.stack([np.stack([x, x + 200.0, x], 1), np.stack([y, y, y + 150.0], 1)], -1).reshape(-1, 2)
    return I.Mesh(vxy=vxy, tri=np.arange(1200, dtype=np.int32).reshape(-1, 3), tag=np.full((400, 3), -1, np.int8))


# mesh, order, precision -> form, groups of edge waves (256 compute units).  A
# strip of this jitter is scattered by the storage order: beyond one tile its
# rings are as large as its tiles, and it is refused.
UNIFORM = [(45, 1, F64, R, 2), (45, 1, F32, R, 2), (45, 2, F64, R, 1), (45, 2, F32, R, 2), (45, 3, F32, R, 2),
           (45, 3, F64, T, 0), (170, 1, F64, R, 1), (170, 1, F32, R, 1), (235, 1, F32, T, 0), (170, 2, F32, T, 0),
           (170, 2, F64, T, 0), (235, 2, F64, S, 0), (290, 2, F64, T, 0), (170, 3, F32, T, 0), (235, 3, F64, S, 0), (20, 0, F64, S, 0),
           ("strip 95", 2, F64, R, 1), ("isolated", 2, F64, R, 1), ("strip 385", 2, F64, S, 0)]


@pytest.mark.parametrize("mesh,p,precision,form,groups", UNIFORM)
def test_uniform_form_and_two_launches_agree(mesh, p, precision, form, groups):
    if isinstance(mesh, int):
        prob = I.config_c2(n=mesh, p=p, seed=mesh)
    else:
        m = isolated() if mesh == "isolated" else strip(int(mesh.split()[1]))
        prob = I._problem(mesh, m, I.bathy_flat(30.0), I.ic_rest(0.0), p, p, p)
    c0 = I.random_state(prob.mesh, prob.p, p, 3, prob.hb_vertex, 0.2, 0.5, 0.1)
    out = []
    with swe.context_for(prob, precision=precision) as ctx:
        for calls in ((2,), (1, 1)):
            ctx.set_state(c0)
            for k in calls:
                ctx.step(k, prob.dt())
            ctx.sync()
            out.append(ctx.state()[0])
        got, tile, g = ctx.step_form()
    assert (got, g) == (form, groups) and (tile > 0) == (form != S)
    assert np.array_equal(out[0], out[1])


# n, scheme, lowest order, precision -> form; the larger are above 448 / 1,536
# base blocks (partitioned) and 1,024 / 1,536 blocks (separated)
STATIC = [(40, 2, 1, F64, swe.FORM_STAGE_ONE), (40, 2, 1, F32, swe.FORM_STAGE_ONE), (40, 1, 1, F64, swe.FORM_CHAIN),
          (40, 2, 0, F64, swe.FORM_BRANCHES), (260, 2, 1, F64, swe.FORM_BRANCHES), (480, 2, 1, F32, swe.FORM_BRANCHES),
          (380, 1, 1, F64, swe.FORM_BRANCHES), (460, 1, 1, F32, swe.FORM_BRANCHES), (260, 2, 0, F32, swe.FORM_BRANCHES)]


@pytest.mark.parametrize("n,separate,lo,precision,form", STATIC)
def test_static_form_and_launches_agree(n, separate, lo, precision, form):
    """Bounds: the oracle tests' FP64 and FP32 elevation tolerances."""
    prob = I.config_c2(n=n, p=2)
    prob.p_base = lo
    order = np.full(prob.mesh.ne, lo, dtype=np.int8)
    order[::16 if n < 100 else 32] = 2
    out = []
    for graph in (1, 0):
        with swe.context_for(prob, precision=precision, separate=separate, step_graph=graph) as ctx:
            ctx.set_order(order)
            ctx.set_state_fn(prob.ic)
            if graph:
                assert ctx.step_form()[0] == form
            for steps in (11, 16, 1):
                ctx.step(steps, prob.dt())
            ctx.sync()
            c, t = ctx.state()
            out.append((c[:, 0], t))
    (a, ta), (b, tb) = out
    assert ta == tb
    assert np.linalg.norm(b) > 0
    assert np.linalg.norm(a - b) <= (1e-12 if precision == F64 else 1e-5) * np.linalg.norm(b)


def test_steps_under_capture():
    """The first several-step call on a stream that is being captured (it has
    no tiles yet, and must not make them there), then with tiles; replayed with
    eager work and synchronisations between, each replay against plain calls."""
    import torch
    prob = I.config_c3(n=20)
    prob.adapt, prob.p_base, prob.p_max = 0, 2, 2
    prob.p[:] = 2
    c0 = I.random_state(prob.mesh, prob.p, 2, 3, prob.hb_vertex, 0.2, 0.5, 0.1)
    dt = prob.dt()
    want = []
    with swe.context_for(prob) as ctx:
        ctx.set_state(c0)
        for _ in range(7):
            ctx.step(2, dt)
            want.append(ctx.state()[0])
    s = torch.cuda.Stream()
    with swe.context_for(prob, stream_base=s.cuda_stream) as ctx:
        ctx.set_state(c0)
        done = 0
        for tiles in (False, True):
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                ctx.step(2, dt)
            assert (ctx.step_form()[1] > 0) == tiles
            for _ in range(3):
                with torch.cuda.stream(s):
                    g.replay()
                ctx.sync()
                torch.zeros(1000, device="cuda").sum().item()
                assert np.array_equal(ctx.state()[0], want[done])
                done += 1
            if not tiles:
                ctx.step(2, dt)
                assert np.array_equal(ctx.state()[0], want[done])
                done += 1
