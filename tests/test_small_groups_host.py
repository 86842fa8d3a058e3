"""Host-side check of how dL1 and dL2 are split among groups of waves: the measured calls get the split that was the faster one."""
import ctypes
import os

import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2305_14314_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    return ctypes.CDLL(binding.LIB_PATH)


def _tiles(h, o, r):
    """64 x 64 output tiles of dL1 (h x r) and dL2 (r x o)."""
    up = lambda n: (n + 63) // 64
    return up(h) * up(r), up(r) * up(o)


# 0: partials and a finalize launch; else the groups of waves that share a tile's tokens and finish it
@pytest.mark.parametrize("tokens,h,o,r,groups", [
    (64, 1024, 1024, 16, 1), (65, 1024, 1024, 16, 2), (128, 4096, 4096, 64, 2), (256, 4096, 4096, 64, 4), (256, 5120, 13824, 64, 1),
    (257, 5120, 13824, 64, 2), (262, 3072, 14080, 16, 2), (512, 4096, 4096, 64, 4), (512, 4096, 11008, 256, 1), (1024, 2048, 2048, 64, 0), (1024, 2560, 2560, 64, 4),
    (1024, 8192, 8192, 64, 4), (1400, 3584, 3584, 64, 0), (1400, 4608, 4608, 64, 0), (2048, 5120, 5120, 64, 4), (3000, 8192, 8192, 64, 4),
    (600, 9216, 9216, 64, 2), (4096, 9216, 9216, 64, 0), (4096, 10240, 10240, 64, 0), (4096, 8192, 22016, 64, 2), (4096, 11008, 4096, 256, 1)])
def test_measured_calls(lib, tokens, h, o, r, groups):
    f = lib._ZN5qlora12small_groupsEiii
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int] * 3
    t1, t2 = _tiles(h, o, r)
    assert f(tokens, t1 + t2, min(t1, t2)) == groups


def test_groups_have_kernels(lib):
    """Whatever the tokens and tiles: 0, or a number of groups that the launch takes; several only where a tile's tokens are several K-steps."""
    f = lib._ZN5qlora12small_groupsEiii
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int] * 3
    for tokens in (1, 16, 63, 64, 65, 128, 129, 192, 193, 256, 257, 320, 500, 512, 513, 640, 1000, 1024, 1025, 2048, 4096, 1 << 20, 1 << 30):
        for tiles in (1, 2, 16, 79, 80, 149, 150, 255, 256, 257, 399, 400, 511, 512, 513, 2000, 100000):
            for least in {1, min(tiles, 128), min(tiles, 256), tiles}:
                n = f(tokens, tiles, least)
                assert n in (0, 1, 2, 4) and (n <= 1 or tokens > 64), (tokens, tiles, least)


# partials that share a launch are the faster form where they are few, under dropout sooner; without the room for that the groups stay
@pytest.mark.parametrize("tokens,h,o,r,dropout,groups", [
    (481, 256, 64, 16, True, 0), (494, 320, 64, 64, True, 0), (894, 448, 4544, 16, True, 0), (1537, 192, 9728, 16, True, 0), (2090, 3776, 7296, 16, True, 0),
    (509, 128, 64, 64, False, 0), (378, 512, 64, 32, False, 4), (449, 192, 4160, 64, True, 4), (512, 4096, 4096, 64, True, 4), (512, 4096, 4096, 64, False, 4), (577, 1664, 1600, 16, False, 0),
    (577, 1664, 1600, 16, True, 0), (640, 3072, 3136, 96, True, 4), (330, 4160, 2048, 256, True, 2), (1500, 3072, 3136, 128, True, 4), (256, 1024, 1024, 16, False, 4)])
def test_layer_by_partials_or_groups(lib, tokens, h, o, r, dropout, groups):
    f = lib._ZN5qlora12layer_groupsElllimb
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.c_size_t, ctypes.c_bool]
    assert f(tokens, h, o, r, 1 << 40, dropout) == groups
    if groups == 0:
        assert f(tokens, h, o, r, 0, dropout) == 4


# all layers' gradients in one launch, or, with little room where the weights will lie, a launch per layer: then its own tiles count
@pytest.mark.parametrize("tokens,h,outs,r,groups", [
    (2000, 5120, (5120, 5120, 5120), 64, (2, 2, 2)), (512, 1024, (1024, 1024), 64, (4, 4)),
    (1938, 448, (4288, 3712, 576, 4416), 64, (0, 0, 0, 0)), (780, 640, (256, 768, 1536), 64, (0, 0, 0)),
    (1647, 448, (2624, 3776, 320, 5504), 64, (0, 0, 0, 0)), (1132, 320, (1088, 4480, 1152, 4288), 64, (0, 0, 0, 0)),
    (757, 128, (4416, 768), 256, (2, 4)), (755, 192, (576, 256), 256, (4, 4)), (3787, 320, (6080,), 256, (2,)), (194, 640, (128, 128), 64, (4, 4))])
def test_stacked_layers(lib, tokens, h, outs, r, groups):
    f = lib._ZN5qlora12stack_groupsElilPKlPKii
    f.restype = ctypes.c_int
    n = len(outs)
    o, ranks = (ctypes.c_int64 * n)(*outs), (ctypes.c_int32 * n)(*[r] * n)
    assert tuple(f(ctypes.c_int64(tokens), n, ctypes.c_int64(h), o, ranks, l) for l in range(n)) == groups
