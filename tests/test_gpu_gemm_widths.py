"""GPU parity of the main product in every way its output is cut -- tile columns of 256, 192 or 128, two widths beside each other,
tiles of 128 x 128 with rings of five and nine slots: fewer tiles than compute units, outputs just past a full round, and widths
that leave every kind of remainder of a last column."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import dev_bf16, host_bits, upload_quant
from test_gpu_linear import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,h,o,r", [(513, 64, 64, 0), (700, 192, 448, 16), (520, 64, 10944, 16), (1000, 64, 8256, 16),
                                     (1000, 128, 8320, 0), (1025, 64, 8384, 16), (800, 320, 16448, 16), (4100, 64, 3904, 16)])
def test_widths(oracle, synth, M, h, o, r):
    _widths(oracle, synth, M, h, o, r)


class _Cut(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("wide", "rest", "rest_width", "half", "slots")]


def _cut(M, K, N, r):
    """How the product of M x K and K x N is cut (both directions of _widths): (256-wide columns?, width of the rest, ring slots)."""
    from paper_2305_14314_amd import binding
    f = ctypes.CDLL(binding.LIB_PATH)._ZN5qlora8gemm_cutEiii
    f.restype, f.argtypes = _Cut, [ctypes.c_int] * 3
    c = f(M, N, K // 64 + (r + 63) // 64)
    return c.wide > 0, c.rest_width if c.rest else 0, c.slots


# one K-step, up to ten (one turn of the nine-slot ring and the segment switch), ragged rows and columns, up to one workgroup per
# compute unit and just above
@pytest.mark.parametrize("M,h,o,r,slots", [(513, 64, 128, 16, 9), (640, 128, 192, 0, 9), (641, 512, 320, 16, 9), (769, 576, 64, 32, 9),
                                           (1025, 640, 3520, 16, 9), (700, 704, 5504, 0, 5), (1100, 320, 4224, 16, 5),
                                           (1300, 768, 3520, 48, 5), (2300, 832, 2368, 64, 5)])
def test_half_tiles(oracle, synth, M, h, o, r, slots):
    """Tiles of 128 x 128 by the kernel that the shape is meant for."""
    assert _cut(M, h, o, r) == (False, 0, slots)
    _widths(oracle, synth, M, h, o, r)


@pytest.mark.parametrize("kt,r", [(15, 16), (16, 144), (17, 64), (18, 16), (19, 256), (20, 16), (21, 80), (22, 16), (23, 48), (33, 128)])
def test_nine_slot_ring(oracle, synth, kt, r):
    """The nine-slot ring in its steady state, which fifteen K-steps of the weight reach: one turn of it and two (33), the number of
    steps in every residue of the ring, then the adapter's segment of one to four."""
    assert _cut(520, 64 * kt, 320, r) == (False, 0, 9)
    _widths(oracle, synth, 520, 64 * kt, 320, r)


@pytest.mark.parametrize("M,h,o,r,cut", [(1000, 640, 15296, 16, (True, 0, 0)), (2049, 1216, 1984, 48, (False, 128, 0)),
                                         (1500, 1280, 3200, 16, (False, 128, 0)), (1000, 64, 8256, 16, (False, 192, 0)), (4096, 640, 13376, 16, (True, 192, 0)),
                                         (4100, 640, 12544, 16, (True, 128, 0))])
def test_each_cut(oracle, synth, M, h, o, r, cut):
    """256-wide columns alone, narrower ones alone, and both beside each other."""
    assert _cut(M, h, o, r) == cut
    _widths(oracle, synth, M, h, o, r)


def _widths(oracle, synth, M, h, o, r):
    """Forward (output width o) and, with the sides swapped, backward (output width o again, and the adapter's segment)."""
    import paper_2305_14314_amd as ql
    print(f"case widths M={M} h={h} o={o} r={r}", flush=True)
    s, rows = 0.5, np.unique(np.concatenate([np.arange(0, M, 97), [255, 256, 511, 512, M - 1]]))
    for fwd in (True, False):
        shape = (h, o) if fwd else (o, h)
        q = oracle.nf4_quantize(synth.normal_f32(shape, synth.SIGMA_W, 9500 + M))
        What, Wq = oracle.nf4_dequant(q), upload_quant(q)
        A = synth.normal_bf16((M, h), 1.0, 9501 + M)
        L1 = synth.normal_bf16((shape[0], r), 0.05, 9502) if r else None
        L2 = synth.normal_bf16((r, shape[1]), 0.05, 9503) if r else None
        dL = [dev_bf16(L) if r else None for L in (L1, L2)]
        if fwd:
            got = ql.qlora_linear_fwd(dev_bf16(A), Wq, dL[0], dL[1], s)
            ref = oracle.linear_fwd(A, What, L1, L2, s, rows=rows)
        else:
            got, _, _ = ql.qlora_linear_bwd(dev_bf16(A), None, Wq, dL[0], dL[1], s, need_dL=False)
            ref = oracle.linear_bwd_dx(A, What, L1, L2, s, rows=rows)
        torch.cuda.synchronize()
        _check(host_bits(got)[rows], ref, "Y" if fwd else "dX")
