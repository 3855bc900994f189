"""Host-side behaviour on the stand-in runtime (no GPU)."""
import pytest

from tests import host_runtime


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("host"))


def test_read_back_memory_is_coherent_by_its_own_flags(lib):
    """Kernels write read-backs into pinned memory that host threads then read:
    its coherence does not hang on the environment."""
    host_runtime.run(lib, """
        with swe.context_for(I.config_c2(n=160, p=2)) as ctx:      # 51,200 elements, 7.4 MB
            ctx.state()
            assert count("pinned allocations") == 1
            assert count("pinned allocations not coherent") == 0
    """)


def test_read_back_without_host_memory_does_not_throw(lib):
    """An exception that leaves the C entry ends the process."""
    host_runtime.run(lib, """
        with swe.context_for(I.config_c2(n=160, p=2)) as ctx:
            out, t = np.empty((ctx.ne, 3, ctx.K)), ctypes.c_double()
            for _ in range(2):                                     # the ring's first use, then a later one
                L.fake_refuse_new(1)
                st = L.swe_get_state(ctx.h, swe._d(out), ctypes.byref(t))
                L.fake_refuse_new(0)
                assert st == swe.SWE_OK, st
            assert count("pinned allocations") == 1
    """)


def test_step_graphs_are_built_and_destroyed_one_at_a_time_and_at_rest(lib):
    """Contexts with static order maps (whose graphs have branches) in several
    threads, beside a batch whose members come and go."""
    host_runtime.run(lib, """
        def contexts(seed):
            for i in range(4):
                prob = I.config_dambreak(n=12 + 2 * i, seed=seed)
                with swe.context_for(prob, separate=1 + i % 2) as ctx:
                    for shift in range(3):
                        ctx.set_order(np.roll(prob.p, shift))
                        ctx.step(20, 1e-5)
                    ctx.sync()

        def batch():
            with swe.Batch(budget_bytes=64 << 20, max_instances=8) as b:
                members = []
                for i in range(12):
                    p = 1 + i % 3
                    m = swe.context_for(I.config_c2(n=10, p=p))
                    members.append((b.admit(m, 100, 1.0), m))
                    b.tick(17)
                    if len(members) > 3:
                        slot, m = members.pop(0)
                        b.retire(slot)
                        m.close()
                for slot, m in members:
                    b.retire(slot)
                    m.close()

        errors = []
        def guarded(f, *a):
            try:
                f(*a)
            except BaseException as e:
                errors.append(e)

        threads = [threading.Thread(target=guarded, args=(contexts, s)) for s in range(4)]
        threads.append(threading.Thread(target=guarded, args=(batch,)))
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors
        assert count("graphs built") > 20
        assert count("graphs destroyed in flight") == 0
        assert count("graph calls at once") == 1, count("graph calls at once")
        assert count("other calls beside graph calls") == 0, count("other calls beside graph calls")
    """)


def test_tiles_are_built_by_the_call_that_uses_them(lib):
    """Not for a context that only goes through a batch, nor when it comes back
    from one; by the first call of several steps, once."""
    host_runtime.run(lib, """
        prob = I.config_c2(n=40, p=2)
        with swe.Batch(budget_bytes=64 << 20, max_instances=8) as b, swe.context_for(prob) as ctx:
            ctx.set_state(np.zeros((ctx.ne, 3, ctx.K)))
            slot = b.admit(ctx, 50, 1.0)
            b.tick(50)
            b.retire(slot)
            assert count("tile builds") == 0
            ctx.step(1, 1.0)
            assert count("tile builds") == 0
            ctx.step(5, 1.0)
            ctx.step(4, 1.0)
            assert count("tile builds") == 1 and count("one-launch steps") == 8
            slot = b.admit(ctx, 50, 1.0)
            b.retire(slot)
            ctx.step(2, 1.0)
            assert count("tile builds") == 2 and count("one-launch steps") == 10
    """)


# swe_footprint_bytes before the one-launch step and the device-side transfers,
# for ne x p = 0..3 x (FP64, FP32): a request admitted then is admitted now.
FOOTPRINTS = {
    288: [89068, 68588, 189784, 115700, 349528, 189784, 562520, 296280],
    22050: [4396892, 3506012, 8511636, 5555384, 15460500, 8511636, 24725652, 13144212],
    65536: [12956044, 10334604, 25054528, 16364940, 45501760, 25054528, 72764736, 38686016],
    260642: [51490588, 41056028, 99688132, 65059592, 181077700, 99688132, 289597124, 153947844],
}


def test_footprints_are_no_larger_than_they_were(lib):
    host_runtime.run(lib, f"""
        for ne, old in {FOOTPRINTS!r}.items():
            new = [swe.swe_footprint_bytes(ne, p, prec) for p in range(4) for prec in (0, 1)]
            assert all(a <= b for a, b in zip(new, old)), (ne, new, old)
            assert all(a >= 0.85 * b for a, b in zip(new, old)), (ne, new, old)
    """)


def test_footprints_bound_what_is_held(lib):
    """Alone after set_mesh and set_state, and resident in an empty batch."""
    host_runtime.run(lib, """
        for p in range(4):
            for prec in (0, 1):
                prob = I.config_c2(n=21, p=p)
                bound = swe.swe_footprint_bytes(prob.mesh.ne, p, prec)
                before = count("bytes")
                with swe.context_for(prob, precision=prec) as ctx:
                    ctx.set_state(np.zeros((ctx.ne, 3, ctx.K)))
                    assert 0 < count("bytes") - before <= bound, (p, prec)
                    with swe.Batch(precision=prec, budget_bytes=64 << 20, max_instances=2) as b:
                        empty = count("bytes")
                        b.admit(ctx, 5, 1.0)
                        b.tick(5)
                        assert b.free_bytes() >= (64 << 20) - bound
                        # the batch's own fixed arrays came before, the context's state buffers went
                        own = 2 * 1024
                        assert count("bytes") - before <= bound + own, (p, prec)
                        b.retire(0)
                        assert count("bytes") == empty and b.free_bytes() == 64 << 20
                    ctx.step(4, 1.0)
    """)


def test_reading_and_stepping_leave_captures_elsewhere_alone(lib):
    """A read-back and a step made no allocation when both were host loops and
    stage launches; those they make now must not break a stream capture that
    another thread (or this one, on another stream) has under way."""
    host_runtime.run(lib, """
        with swe.context_for(I.config_c2(n=160, p=2)) as ctx:
            ctx.set_state(np.zeros((ctx.ne, 3, ctx.K)))
            before = count("allocations a capture elsewhere forbids")
            ctx.step(4, 1.0)
            ctx.state()
            assert count("tile builds") == 1 and count("pinned allocations") == 1
            assert count("allocations a capture elsewhere forbids") == before
    """)


def test_no_entry_throws_when_host_memory_runs_out(lib):
    """Every call that takes host memory is refused with SWE_ENOMEM (or goes on
    without it); with memory again the same objects work."""
    host_runtime.run(lib, """
        def refused(call):
            L.fake_refuse_new(1)
            st = call()
            L.fake_refuse_new(0)
            assert st in (swe.SWE_OK, swe.SWE_ENOMEM), st
            return st == swe.SWE_ENOMEM

        prob = I.config_dambreak(n=12)
        m = prob.mesh
        p32, p8 = ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int8)
        vxy, tri, tag = (np.ascontiguousarray(a) for a in (m.vxy, m.tri.astype(np.int32), m.tag.astype(np.int8)))
        order = np.ascontiguousarray(prob.p)
        names = []
        with swe.context_for(prob, separate=2) as ctx, swe.context_for(I.config_c2(n=9, p=2)) as member:
            c, hb = np.zeros((ctx.ne, 3, ctx.K)), np.ascontiguousarray(prob.hb_vertex)
            pts, t = np.zeros((ctx.ne, swe.SWE_NQP, 3)), ctypes.c_double()
            d = swe._d
            calls = {
                "mesh": lambda: L.swe_set_mesh(ctx.h, len(vxy), d(vxy), ctx.ne, tri.ctypes.data_as(p32), tag.ctypes.data_as(p8)),
                "bathymetry": lambda: L.swe_set_bathymetry(ctx.h, d(hb)),
                "order": lambda: L.swe_set_order(ctx.h, order.ctypes.data_as(p8)),
                "points": lambda: L.swe_set_state_points(ctx.h, 0.0, d(pts)),
                "state": lambda: L.swe_set_state(ctx.h, 0.0, d(c)),
                "source": lambda: L.swe_set_source(ctx.h, d(c)),
                "step": lambda: L.swe_step(ctx.h, 9, 1e-5),
                "sync": lambda: L.swe_sync(ctx.h),
                "get": lambda: L.swe_get_state(ctx.h, d(c), ctypes.byref(t)),
                "rhs": lambda: L.swe_rhs(ctx.h, 0.0, d(c), d(c.copy())),
            }
            for name, call in calls.items():
                if refused(call):
                    names.append(name)
                    assert b"no host memory" in L.swe_last_error(ctx.h)
                assert call() == swe.SWE_OK, name
            slot, n = ctypes.c_int32(), ctypes.c_int()
            with swe.Batch(budget_bytes=64 << 20, max_instances=4) as b:
                refused(lambda: L.swe_batch_admit(b.h, member.h, 9, 1.0, ctypes.byref(slot)))
                if L.swe_batch_resident(b.h) == 0:
                    assert L.swe_batch_admit(b.h, member.h, 9, 1.0, ctypes.byref(slot)) == swe.SWE_OK
                refused(lambda: L.swe_batch_tick(b.h, 9))
                slots = (ctypes.c_int32 * 4)()
                refused(lambda: L.swe_batch_poll(b.h, slots, (ctypes.c_int32 * 4)(), 4, ctypes.byref(n)))
                refused(lambda: L.swe_batch_tune(b.h, 1))
                L.fake_refuse_new(1)
                L.swe_batch_destroy(b.h)
                L.fake_refuse_new(0)
                b.h = None
            member.step(2, 1.0)
        assert {"mesh", "order", "points", "step"} <= set(names), names
    """)
