"""Host-side checks of the path whose waves share one decode of the weight: which calls take it."""
from test_midtok_host import _run_check, pytestmark  # noqa: F401


def test_forward_route_follows_from_the_shape(tmp_path):
    out = _run_check(tmp_path, "fwd_route_check")
    assert out.startswith("OK "), out
    assert int(out.split()[1]) == 40000 and int(out.split()[2]) > 2000


def test_backward_modes_are_kept_and_restored():
    """The default is mode 2; a mode set returns the one before; queries change nothing; other values select the fused form."""
    import paper_2305_14314_amd as ql
    f = ql.qlora_bwd_fused_dequant
    assert f(-1) == 2
    try:
        assert f(0) == 2 and f(-1) == 0 and f(1) == 0 and f(7) == 1 and f(2) == 1 and f(-5) == 2
    finally:
        f(2)


def test_shared_decode_plans_and_choice(tmp_path):
    out = _run_check(tmp_path, "wide_choice_check")
    assert out.startswith("OK 37 "), out
    assert int(out.split()[2]) > 15000
