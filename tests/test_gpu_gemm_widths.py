"""GPU parity of the main product where its output is cut into tile columns of 256, 192 or 128: fewer tiles than compute
units, outputs just past a full round, and widths that leave every kind of remainder of a 192- or 128-wide last column."""
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


@pytest.mark.parametrize("M,h,o,r", [(513, 64, 128, 16), (640, 128, 192, 0), (641, 512, 320, 16), (769, 576, 64, 32), (1025, 640, 3520, 16),
                                     (700, 704, 5504, 0), (2049, 1216, 1984, 48)])
def test_half_tiles(oracle, synth, M, h, o, r):
    """Tiles of 128 x 128: one K-step, one to two turns of the nine-slot ring and the segment switch in each of its places, just
    below and above one workgroup per compute unit, ragged rows and columns."""
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
