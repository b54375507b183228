"""CPU-only: the binding's own allocations."""
import os
import types

import pytest


@pytest.fixture
def bi():
    import paper_2607_28897_amd as m
    if not os.path.exists(m.LIB_PATH):
        pytest.skip("library not built")
    m.lib()
    return m


class NoMemory(Exception):
    pass


@pytest.mark.parametrize("fails", [False, True])
def test_workspace_is_on_the_device_of_the_stream(bi, monkeypatch, fails):
    """The calls run on the current device's current stream, wherever their
    operands are; a workspace of another device would go back to that device's
    allocator, ordered on another stream, while the call still uses it."""
    asked = []

    def empty(n, dtype, device):
        asked.append((n, dtype, device))
        if fails:
            raise NoMemory
        return "buffer"

    fake = types.SimpleNamespace(empty=empty, uint8="u8", cuda=types.SimpleNamespace(OutOfMemoryError=NoMemory))
    monkeypatch.setattr(bi, "_torch", lambda: fake)
    for ws, size in (bi._mul_ws(16384, 16384, 3),
                     bi._workspace(bi.lib().bigint_divmod_workspace_size, "divmod", 2048, 1024, 16)):
        n, dtype, device = asked.pop(0)
        assert n > 0 and dtype == "u8" and device == "cuda"      # no index: the current device
        assert (ws, size) == ((None, 0) if fails else ("buffer", n))
    assert bi._mul_ws(1024, 1024, 3) == (None, 0) and not asked
