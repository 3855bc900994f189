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
