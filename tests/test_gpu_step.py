"""The one-launch step (both stages of a tile of elements in one kernel)
against stage-by-stage launches: advancing two steps in one call takes it,
the same two steps in two calls do not, and the results must be equal bit for
bit.  Element counts around its tiles (192 owned elements, fewer on meshes
whose tiles have long rings), all land, open edges and an extra source, odd
step counts, and a mesh whose triangles share no edge, which it does not
take."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2311_11348_amd import inputs as I
from paper_2311_11348_amd import swe
from tests.test_gpu_transfer import strip

pytestmark = pytest.mark.gpu


def both(prob, precision, steps, source=False):
    c0 = I.random_state(prob.mesh, prob.p, prob.p_max, 3, prob.hb_vertex, 0.2, 0.5, 0.1)
    dt = prob.dt()
    src = I.random_state(prob.mesh, prob.p, prob.p_max, 4, prob.hb_vertex, 1e-3, 1e-3) if source else None
    got = []
    for one_by_one in (False, True):
        with swe.context_for(prob, precision=precision) as ctx:
            ctx.set_source(src)
            ctx.set_state(c0)
            for _ in range(steps if one_by_one else 1):
                ctx.step(1 if one_by_one else steps, dt)
            ctx.sync()
            got.append(ctx.state()[0])
    assert np.all(np.isfinite(got[0])) and not np.array_equal(got[0], c0)
    return c0, dt, got


@pytest.mark.parametrize("precision", [swe.SWE_FP64, swe.SWE_FP32_WB])
@pytest.mark.parametrize("p", [1, 2, 3])
@pytest.mark.parametrize("ne", [1, 2, 95, 96, 97, 191, 193, 385])
def test_strip_bitwise(ne, p, precision):
    prob = I._problem("strip", strip(ne), I.bathy_shelf(4.0e4, 40.0, 20.0), I.ic_rest(0.0), p, p, p,
                      f_coriolis=1e-4, friction=I.FRICTION_LINEAR, friction_coef=1e-3)
    _, _, (a, b) = both(prob, precision, 4)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", [swe.SWE_FP64, swe.SWE_FP32_WB])
@pytest.mark.parametrize("p", [1, 2, 3])
@pytest.mark.parametrize("n,steps", [(9, 2), (13, 5), (45, 3), (130, 2), (170, 3), (235, 2)])   # 130: 256 tiles; 235: > 512
def test_open_sea_bitwise(n, steps, p, precision):
    prob = I.config_c2(n=n, p=p, seed=n)
    c0, dt, (a, b) = both(prob, precision, steps, source=n == 13)
    assert np.array_equal(a, b)
    if n == 9 and precision == swe.SWE_FP64:
        ref = Oracle.from_problem(prob).step(c0, steps, dt)
        assert np.linalg.norm(a - ref) <= 1e-12 * np.linalg.norm(ref)


def test_isolated_triangles_bitwise():
    """No two triangles share an edge: three land items each and no ring."""
    k = np.arange(400)
    x, y = (k % 20) * 300.0, (k // 20) * 300.0
    vxy = np.stack([np.stack([x, x + 200.0, x], 1), np.stack([y, y, y + 150.0], 1)], -1).reshape(-1, 2)
    mesh = I.Mesh(vxy=vxy, tri=np.arange(1200, dtype=np.int32).reshape(-1, 3), tag=np.full((400, 3), -1, np.int8))
    prob = I._problem("isolated", mesh, I.bathy_flat(30.0), I.ic_rest(0.0), 2, 2, 2)
    _, _, (a, b) = both(prob, swe.SWE_FP64, 4)
    assert np.array_equal(a, b)
