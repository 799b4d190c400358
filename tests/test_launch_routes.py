"""Which launches the host side chooses for a call, without a GPU (see tests/recorder)."""

import pytest

from tests.recorder import record


def _uneven(pairs, long):
    """Kept lengths of a cache with one dense head in eight, the others sparse."""
    return [long if p % 8 == 0 else long // 20 for p in range(pairs)]


# ------------------------------------------------------------------ gapless numbering
@pytest.mark.parametrize("call", [["step"], ["attend"], ["static"], ["score", [4] * 16]])
def test_unanswered_capture_query_leaves_no_error_behind(call):
    """The runtime may refuse to say whether a stream is being captured (the legacy stream while
    another one is: error 906).  The call must go on, and must not find that error when it asks
    whether its own launches went well."""
    setup = [["append", [8192] * 16], ["lengths", _uneven(128, 6000)], ["attend"], ["capture", 0, 906]]
    got = record(dict(batch=16), setup + [call])[-1]
    assert got.rc == 0
    assert "compact" in got.launches[0][0]           # the route that asks
