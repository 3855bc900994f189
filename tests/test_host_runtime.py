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
