"""Host-side behaviour on the stand-in runtime (no GPU)."""
import pytest

from tests import host_runtime


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("host"))


def test_read_back_memory_is_coherent_by_its_own_flags(lib):
    """Kernels write read-backs into pinned memory that host threads then read:
    its coherence and the events' release do not hang on the environment."""
    host_runtime.run(lib, """
        with swe.context_for(I.config_c2(n=160, p=2)) as ctx:      # 51,200 elements, 7.4 MB
            ctx.state()
            assert count("pinned allocations") == 1
            assert count("pinned allocations not coherent") == 0
            assert count("host waits on events without a system release") == 0
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
