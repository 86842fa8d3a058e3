"""Host-side checks of the path whose waves share one decode of the weight: which calls take it."""
from test_midtok_host import _run_check, pytestmark  # noqa: F401


def test_forward_route_follows_from_the_shape(tmp_path):
    out = _run_check(tmp_path, "fwd_route_check")
    assert out.startswith("OK "), out
    assert int(out.split()[1]) == 40000 and int(out.split()[2]) > 2000
