"""State read and written through the device's packing kernels: the caller's
layout and element order against the numbers themselves, at element counts
around the kernels' 64-element blocks and the two halves of an FP32 transfer,
and what a refused state leaves behind."""
import numpy as np
import pytest

from paper_2311_11348_amd import inputs as I
from paper_2311_11348_amd import swe

pytestmark = pytest.mark.gpu


def strip(ne):
    """ne triangles in a row (jittered), each sharing an edge with the next."""
    rng = np.random.default_rng(ne)
    i = np.arange(ne + 2)
    vxy = np.stack([i * 100.0, (i % 2) * 150.0 + rng.uniform(-20.0, 20.0, ne + 2)], 1)
    tri = np.array([[e, e + 1, e + 2] if e % 2 else [e, e + 2, e + 1] for e in range(ne)], np.int32)
    perm = rng.permutation(ne)                       # the caller's order is not the storage order
    m = I.Mesh(vxy=vxy, tri=np.ascontiguousarray(tri[perm]), tag=np.full((ne, 3), -1, np.int8))
    assert np.all(m.areas() > 0)
    return m


@pytest.mark.parametrize("precision", [swe.SWE_FP64, swe.SWE_FP32_WB])
@pytest.mark.parametrize("p,ne", [(0, 1), (1, 63), (2, 64), (3, 65), (2, 129), (3, 257), (1, 1000)])
def test_state_round_trip(p, ne, precision):
    mesh = strip(ne)
    prob = I._problem("strip", mesh, I.bathy_flat(30.0), I.ic_rest(0.0), p, 0, p)
    prob.p = np.random.default_rng(1).integers(0, p + 1, ne).astype(np.int8)
    c0 = I.random_state(mesh, np.full(ne, p), p, 5, prob.hb_vertex)
    keep = np.arange(I.K_OF_P[p])[None, :] < np.array(I.K_OF_P)[prob.p][:, None]
    with swe.context_for(prob, precision=precision) as ctx:
        bad = c0.copy()
        bad[ne // 2, 1, 0] = np.inf
        ctx.set_state(c0, 3.0)
        with pytest.raises(swe.SweError):
            ctx.set_state(bad, 4.0)                  # refused: the state and time before stay
        got, t = ctx.state()
        # one multiplication by 1 / s and one by s, each within half an ulp
        # (and the stored value in FP32): at most two FP64 ulps, one FP32 ulp
        tol = 2.0 ** -51 if precision == swe.SWE_FP64 else 2.0 ** -23
        ref = c0 * keep[:, None, :]
        assert t == 3.0
        assert np.all(np.abs(got - ref) <= tol * np.abs(ref))
        if p > 0 and (~keep).any():
            e = int(np.argmax((~keep).any(1)))
            c1 = c0.copy()
            c1[e, 2, -1] = np.nan                    # a mode above the element's order is not looked at
            ctx.set_state(c1)
            assert np.array_equal(ctx.state()[0], got)
        ctx.set_source(c0)
        with pytest.raises(swe.SweError):
            ctx.set_source(bad)
        r0 = ctx.rhs(0.0, np.zeros_like(c0))
        ctx.set_source(None)
        r1 = ctx.rhs(0.0, np.zeros_like(c0))
        assert np.all(np.abs((r0 - r1) - ref) <= 4 * tol * (np.abs(ref) + np.abs(r1)) + 1e-300)
        assert np.array_equal(ctx.state()[0], got)


@pytest.mark.parametrize("precision,p,n", [(swe.SWE_FP32_WB, 2, 70), (swe.SWE_FP64, 1, 200), (swe.SWE_FP64, 3, 141)])
def test_large_read_back_threads(precision, p, n):
    """Read-backs of a few parts of the pinned ring, by two threads on two
    contexts at once: the bytes of a read alone (the round trip's tolerance
    against what was set)."""
    import threading
    prob = I.config_c3(n=n)
    prob.p[:], prob.p_base, prob.p_max, prob.adapt = p, p, p, 0
    c0 = I.random_state(prob.mesh, prob.p, p, 9, prob.hb_vertex)
    tol = 2.0 ** -51 if precision == swe.SWE_FP64 else 2.0 ** -23
    with swe.context_for(prob, precision=precision) as a, swe.context_for(prob, precision=precision) as b:
        a.set_state(c0)
        b.set_state(2.0 * c0)
        alone, alone2 = a.state()[0], b.state()[0]
        assert np.all(np.abs(alone - c0) <= tol * np.abs(c0))
        assert np.array_equal(alone2, 2.0 * alone)
        bad = []

        def read(ctx, ref):
            for _ in range(4):
                if not np.array_equal(ctx.state()[0], ref):
                    bad.append(ctx)
        th = [threading.Thread(target=read, args=x) for x in ((a, alone), (b, alone2))]
        for t in th:
            t.start()
        for t in th:
            t.join()
        assert not bad
