"""Forward and input gradient at tens to hundreds of tokens, where the weight is decoded inside a product that is split
along its contraction: against the fp64 oracle at the edges of its tiles (16 tokens, groups of at most 128, slabs of 128
outputs, steps of 32 / 128), with and without an adapter, under dropout, for the other 4-bit types and for weights
without Double Quantization."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import dev_bf16, dev_f32, host_bits, upload_quant
from test_boundary import accepted_workspace
from test_gpu_dropout import _mask
from test_gpu_fused_bwd import _dx, _gemm_launches, fused  # noqa: F401
from test_gpu_linear import _check

pytestmark = pytest.mark.gpu


class _Plan(ctypes.Structure):
    _fields_ = ([("ok", ctypes.c_bool), ("pack", ctypes.c_bool)] + [(n, ctypes.c_int) for n in ("MF", "KW", "n_tg", "n_slabs", "steps", "n_lparts",
                "chunk", "max_contrib", "units", "ups", "wgs")] + [(n, ctypes.c_size_t) for n in ("part_floats", "lpart_floats", "pack_elems")] +
                [("us", ctypes.c_double)])


def _plan(M, h, o, r):
    """The plan of a forward call that brings the reported workspace (the library's internal struct)."""
    from paper_2305_14314_amd import binding
    f = ctypes.CDLL(binding.LIB_PATH)._ZN5qlora8mid_planEblllimb
    f.restype, f.argtypes = _Plan, [ctypes.c_bool, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t, ctypes.c_bool]
    return f(False, M, h, o, r, max((h + (r + 63) // 64 * 64) * o * 2, 32 << 20), False)


# token tiles 2 .. 8 per group, one to five groups, a remainder of one token; h and o with a 64-wide remainder (half a slab
# forward and backward, half a step backward), one step, many splits; ranks none, below 32, above 64, the largest
@pytest.mark.parametrize("M,h,o,r", [(17, 64, 64, 16), (33, 320, 192, 16), (48, 1024, 1088, 64), (49, 192, 128, 0),
                                      (64, 2048, 320, 48), (65, 128, 448, 32), (81, 576, 1024, 64), (97, 64, 2112, 16),
                                      (112, 320, 320, 80), (113, 1088, 64, 64), (128, 512, 704, 256), (129, 448, 512, 64),
                                      (257, 2048, 1024, 64), (334, 320, 1536, 0), (511, 704, 192, 144), (512, 1024, 1024, 64)])
def test_midtok_forward_backward(oracle, synth, M, h, o, r):
    import paper_2305_14314_amd as ql
    s = 0.5
    q = oracle.nf4_quantize(synth.normal_f32((h, o), synth.SIGMA_W, 500 + M))
    What, Wq = oracle.nf4_dequant(q), upload_quant(q)
    X, dY = synth.normal_bf16((M, h), 1.0, 501 + M), synth.normal_bf16((M, o), 1.0, 502 + M)
    L1 = synth.normal_bf16((h, r), 0.05, 503 + M) if r else None
    L2 = synth.normal_bf16((r, o), 0.05, 504 + M) if r else None
    d = lambda a: None if a is None else dev_bf16(a)
    print(f"case mid M={M} h={h} o={o} r={r}", flush=True)
    ws = ql.workspace_alloc(max(ql.qlora_linear_fwd_sizes(M, h, o, r), ql.qlora_linear_bwd_sizes(M, h, o, r)) + 4096)
    ws[ql.binding.WORKSPACE_HEADER_BYTES:].fill_(0x7F)          # stale contents: NaN-ish everywhere
    fb, bb = ql.qlora_linear_fwd_sizes(M, h, o, r), ql.qlora_linear_bwd_sizes(M, h, o, r)
    T = torch.full((M, 2 * r), float("nan"), dtype=torch.bfloat16, device="cuda") if r else None
    Y = ql.qlora_linear_fwd(d(X), Wq, d(L1), d(L2), s, T_save=T, workspace=ws[:fb])
    assert int((ws[fb:] != 0x7F).sum()) == 0                    # nothing behind the reported size
    dX, dL1, dL2 = ql.qlora_linear_bwd(d(dY), d(X), Wq, d(L1), d(L2), s, T_saved=T, workspace=ws[:bb])
    assert int((ws[max(fb, bb):] != 0x7F).sum()) == 0
    torch.cuda.synchronize()
    _check(host_bits(Y), oracle.linear_fwd(X, What, L1, L2, s), "Y")
    _check(host_bits(dX), oracle.linear_bwd_dx(dY, What, L1, L2, s), "dX")
    if r:
        r1, r2 = oracle.linear_bwd_dl(dY, X, L1, L2, s)
        _check(host_bits(dL1), r1, "dL1", few_terms=M < 64)
        _check(host_bits(dL2), r2, "dL2", few_terms=M < 64)


# Contractions long enough, either way, for the product that decodes the weight (the small layers above may be dequantised
# instead): the same edges, and no launch of the main GEMM.
@pytest.mark.parametrize("M,h,o,r", [(49, 1088, 1024, 0), (64, 2048, 1088, 48), (65, 1024, 2112, 32), (81, 1600, 1088, 64),
                                      (97, 1600, 2112, 16), (112, 2048, 1344, 80), (113, 1088, 2048, 64),
                                      (128, 2752, 3136, 256), (129, 2048, 1088, 64), (334, 1536, 2112, 0),
                                      (511, 2752, 3136, 144), (512, 2112, 1600, 64)])
def test_midtok_is_reached(oracle, synth, M, h, o, r):
    import paper_2305_14314_amd as ql
    s = 0.5
    q = oracle.nf4_quantize(synth.normal_f32((h, o), synth.SIGMA_W, 800 + M))
    What, Wq = oracle.nf4_dequant(q), upload_quant(q)
    X, dY = synth.normal_bf16((M, h), 1.0, 801 + M), synth.normal_bf16((M, o), 1.0, 802 + M)
    L1 = synth.normal_bf16((h, r), 0.05, 803 + M) if r else None
    L2 = synth.normal_bf16((r, o), 0.05, 804 + M) if r else None
    d = lambda a: None if a is None else dev_bf16(a)
    print(f"case mid reached M={M} h={h} o={o} r={r}", flush=True)
    Y, n = _gemm_launches(ql, lambda: ql.qlora_linear_fwd(d(X), Wq, d(L1), d(L2), s))
    (dX, dL1, dL2), m = _gemm_launches(ql, lambda: ql.qlora_linear_bwd(d(dY), d(X), Wq, d(L1), d(L2), s))
    assert n == 0 and m == 0
    _check(host_bits(Y), oracle.linear_fwd(X, What, L1, L2, s), "Y")
    _check(host_bits(dX), oracle.linear_bwd_dx(dY, What, L1, L2, s), "dX")
    if r:
        r1, r2 = oracle.linear_bwd_dl(dY, X, L1, L2, s)
        _check(host_bits(dL1), r1, "dL1", few_terms=M < 64)
        _check(host_bits(dL2), r2, "dL2", few_terms=M < 64)


@pytest.mark.parametrize("M,h,o,r,p", [(3, 320, 192, 16, 0.5), (40, 448, 320, 64, 0.1), (130, 192, 576, 48, 0.1),
                                        (512, 320, 448, 64, 0.3)])
def test_midtok_dropout(oracle, synth, M, h, o, r, p):
    """The mask enters T and, in the input gradient, the adapter's term only -- exactly: one rounding per element."""
    import paper_2305_14314_amd as ql
    q = oracle.nf4_quantize(synth.normal_f32((h, o), synth.SIGMA_W, 600 + M))
    What, Wq = oracle.nf4_dequant(q), upload_quant(q)
    X, dY = synth.normal_bf16((M, h), 1.0, 601 + M), synth.normal_bf16((M, o), 1.0, 602 + M)
    L1, L2 = synth.normal_bf16((h, r), 0.2, 603 + M), synth.normal_bf16((r, o), 0.2, 604 + M)
    keep, dmask = _mask(M, h, p, 605 + M)
    D = oracle.dropout_multipliers(keep, p)
    print(f"case mid dropout M={M} h={h} o={o} r={r} p={p}", flush=True)
    Y = ql.qlora_linear_fwd_dropout(dev_bf16(X), Wq, dev_bf16(L1), dev_bf16(L2), 1.0, dmask, p)
    dX, _, _ = ql.qlora_linear_bwd_dropout(dev_bf16(dY), dev_bf16(X), Wq, dev_bf16(L1), dev_bf16(L2), 1.0, dmask, p)
    torch.cuda.synchronize()
    _check(host_bits(Y), oracle.linear_fwd(X, What, L1, L2, 1.0, D=D), "Y")
    ref = oracle.linear_bwd_dx(dY, What, L1, L2, 1.0, D=D)
    _check(host_bits(dX), ref, "dX")
    got = (host_bits(dX).astype(np.uint32) << 16).view(np.float32).astype(np.float64).reshape(ref.shape)
    # half a bf16 step (2^-8 of the value at most), plus the fp32 sums and the 16 bits U keeps; two roundings would be twice that
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 2e-4 * np.sqrt((ref ** 2).mean()))


@pytest.mark.parametrize("kind,dtype,dq", [("nf4", 0, 0), ("fp4_e2m1", 1, 256), ("int4", 3, 0)])
@pytest.mark.parametrize("M", [2, 60, 200])
def test_midtok_types(oracle, synth, kind, dtype, dq, M):
    import paper_2305_14314_amd as ql
    if M == 2 and dq:
        M = 18                                                  # double-quantised weights take the streaming kernels up to 16
    h, o, r, s = 320, 448, 32, 1.0
    table = oracle.codebook4(kind)
    W = synth.normal_f32((h, o), synth.SIGMA_W, 700)
    q = oracle.nf4_quantize(W, dq_blocksize=dq, table=table)
    What = oracle.nf4_dequant(q)
    Wq = ql.qlora_nf4_quantize(dev_f32(W), dq_blocksize=dq, dtype=dtype)
    X, dY = synth.normal_bf16((M, h), 1.0, 701), synth.normal_bf16((M, o), 1.0, 702)
    L1, L2 = synth.normal_bf16((h, r), 0.05, 703), synth.normal_bf16((r, o), 0.05, 704)
    print(f"case mid {kind} dq={dq} M={M}", flush=True)
    Y = ql.qlora_linear_fwd(dev_bf16(X), Wq, dev_bf16(L1), dev_bf16(L2), s)
    dX, _, _ = ql.qlora_linear_bwd(dev_bf16(dY), dev_bf16(X), Wq, dev_bf16(L1), dev_bf16(L2), s)
    torch.cuda.synchronize()
    _check(host_bits(Y), oracle.linear_fwd(X, What, L1, L2, s), "Y")
    _check(host_bits(dX), oracle.linear_bwd_dx(dY, What, L1, L2, s), "dX")


# The fused backward GEMM is reached above 512 tokens only: its ragged shapes there, the same bits as the two-kernel form
@pytest.mark.parametrize("M,h,o,r", [(520, 64, 64, 0), (600, 320, 1536, 0), (529, 704, 128, 16), (513, 320, 64, 0)])
def test_fused_backward_above_mid(oracle, synth, fused, M, h, o, r):  # noqa: F811
    ql = fused
    L = synth.make_layer(0, 0, M=M, h=h, o=o, r=max(r, 1))
    q = oracle.nf4_quantize(L["W"])
    Wq, X, dY = upload_quant(q), dev_bf16(L["X"]), dev_bf16(L["dY"])
    L1, L2 = (dev_bf16(L["L1"]), dev_bf16(L["L2"])) if r else (None, None)
    print(f"fused bwd: M {M} h {h} o {o} r {r}", flush=True)
    a, b = _dx(ql, 0, dY, X, Wq, L1, L2, L["s"]), _dx(ql, 1, dY, X, Wq, L1, L2, L["s"])
    ref = oracle.linear_bwd_dx(L["dY"], oracle.nf4_dequant(q), L["L1"] if r else None, L["L2"] if r else None, L["s"])
    _check(host_bits(b), ref, "fused dX")
    if r == 0:
        assert torch.equal(a, b)


@pytest.mark.parametrize("M,h,o,r", [(256, 1024, 1024, 64), (64, 4096, 448, 16), (512, 1088, 2048, 48), (200, 1600, 1088, 0)])
def test_smallest_accepted_workspace(oracle, synth, M, h, o, r):
    """With the bytes of the dequantise + GEMM plan and no more the calls split less or take that plan: the oracle's values,
    and nothing written behind them."""
    import paper_2305_14314_amd as ql
    s, L = 0.5, ql.binding.lib()
    nf, nb = accepted_workspace(L, False, M, h, o, r), accepted_workspace(L, True, M, h, o, r)
    assert nf < ql.qlora_linear_fwd_sizes(M, h, o, r) or nb < ql.qlora_linear_bwd_sizes(M, h, o, r)
    q = oracle.nf4_quantize(synth.normal_f32((h, o), synth.SIGMA_W, 900 + M))
    What, Wq = oracle.nf4_dequant(q), upload_quant(q)
    X, dY = synth.normal_bf16((M, h), 1.0, 901 + M), synth.normal_bf16((M, o), 1.0, 902 + M)
    L1 = synth.normal_bf16((h, r), 0.05, 903 + M) if r else None
    L2 = synth.normal_bf16((r, o), 0.05, 904 + M) if r else None
    d = lambda a: None if a is None else dev_bf16(a)
    print(f"case smallest workspace M={M} h={h} o={o} r={r}: {nf} {nb}", flush=True)
    for n, bwd in ((nf, False), (nb, True)):
        ws = ql.workspace_alloc(n + 4096)
        ws[ql.binding.WORKSPACE_HEADER_BYTES:].fill_(0x7F)
        if not bwd:
            Y = ql.qlora_linear_fwd(d(X), Wq, d(L1), d(L2), s, workspace=ws[:n])
            _check(host_bits(Y), oracle.linear_fwd(X, What, L1, L2, s), "Y")
        else:
            dX, dL1, dL2 = ql.qlora_linear_bwd(d(dY), d(X), Wq, d(L1), d(L2), s, workspace=ws[:n])
            _check(host_bits(dX), oracle.linear_bwd_dx(dY, What, L1, L2, s), "dX")
            if r:
                r1, r2 = oracle.linear_bwd_dl(dY, X, L1, L2, s)
                _check(host_bits(dL1), r1, "dL1", few_terms=M < 64)
                _check(host_bits(dL2), r2, "dL2", few_terms=M < 64)
        assert int((ws[n:] != 0x7F).sum()) == 0


@pytest.mark.parametrize("M", [52, 90, 113, 160, 333, 500])
@pytest.mark.parametrize("h,o", [(4096, 11008), (1088, 1344)])
def test_midtok_forward_packed_or_not(synth, M, h, o):
    """The forward's token operand packed by a launch of its own (the large weight, but for 90 tokens) and read as it lies, in
    several groups of tokens (the small one), against fp64 products with the dequantised weight; the same with T saved, bit for bit."""
    import paper_2305_14314_amd as ql
    r, s = 48, 0.5
    plan = _plan(M, h, o, r)
    assert plan.ok and plan.pack == (o == 11008 and M != 90) and (plan.pack or plan.n_tg > 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(4000 + M)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    Wq = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 4100 + M))
    X, L1, L2 = bf(M, h), bf(h, r, sd=0.05), bf(r, o, sd=0.05)
    Y = ql.qlora_linear_fwd(X, Wq, L1, L2, s)
    T = torch.empty((M, 2 * r), dtype=torch.bfloat16, device="cuda")
    Y2 = ql.qlora_linear_fwd(X, Wq, L1, L2, s, T_save=T)
    t = X.double() @ L1.double()
    ref = X.double() @ ql.qlora_nf4_dequant(Wq).double() + s * t @ L2.double()
    _check(host_bits(Y), ref.cpu().numpy(), f"Y M={M}")
    assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))
    got = T[:, :r].double() + T[:, r:].double()               # 16 significant bits
    assert (got - t).abs().max() <= 2.0 ** -14 * t.abs().max() + 1e-6


@pytest.mark.parametrize("M", [3, 9, 11, 12, 16])
@pytest.mark.parametrize("h,o,r", [(1024, 1024, 0), (1088, 1344, 48), (1024, 1024, 128), (2048, 4096, 64), (1344, 1088, 48), (1024, 1024, 144),
                                   (2304, 2368, 0), (448, 1344, 48), (320, 1344, 80)])
def test_few_tokens_forward_decoded_once(synth, M, h, o, r):
    """Up to 16 tokens on a small weight, forward: with the reported workspace (from 12 tokens on decoded once for all of them, if the
    contraction is long enough and no longer than the outputs and the rank up to 128) and with the smallest that the streaming kernel takes, both
    against fp64 products with the dequantised weight.  Which of the two ran shows in how much of the workspace was written.
    T is a sum of h terms of which neither path drops bits, so the two agree to one rounding of the result and the order of the
    sums: a unit in the last place, 2^-7 of the value at most, and h 2^-24 of the largest."""
    import paper_2305_14314_amd as ql
    s = 2.0
    g = torch.Generator(device="cuda")
    g.manual_seed(5000 + M + r)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    Wq = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 5100 + M))
    X, L1, L2 = bf(M, h), (bf(h, r, sd=0.05) if r else None), (bf(r, o, sd=0.05) if r else None)
    small, head = accepted_workspace(ql.binding.lib(), False, M, h, o, r), ql.binding.WORKSPACE_HEADER_BYTES
    T = torch.empty((M, 2 * r), dtype=torch.bfloat16, device="cuda") if r else None

    def run(n, **kw):                                          # the output, and the bytes behind the header up to the last one written
        ws = ql.workspace_alloc(ql.qlora_linear_fwd_sizes(M, h, o, r))
        ws[head:].fill_(0x7F)
        Y = ql.qlora_linear_fwd(X, Wq, L1, L2, s, workspace=ws[:n], **kw)
        assert int(ws[:head].max()) == 0
        return Y, int((ws[head:] != 0x7F).nonzero().max()) + 1

    Y, used = run(None, T_save=T)
    Ys, streamed = run(small)
    plan = _plan(M, h, o, r)
    align = lambda b: (b + 255) // 256 * 256
    decoded = align(plan.part_floats * 4) + plan.lpart_floats * 4 if r else plan.part_floats * 4
    assert abs(decoded - streamed) > 256                       # the two can be told apart
    once = M >= 12 and h <= o and r <= 128 and (h >= (512 if r <= 64 else 256) if r else M * h > 32768)
    assert abs(used - (decoded if once else streamed)) < 16
    ref = X.double() @ ql.qlora_nf4_dequant(Wq).double()
    if r:
        t = X.double() @ L1.double()
        ref = ref + s * t @ L2.double()
        got = T[:, :r].double() + T[:, r:].double()
        assert (got - t).abs().max() <= 2.0 ** -14 * t.abs().max() + 1e-6
    _check(host_bits(Y), ref.cpu().numpy(), f"Y M={M}")
    _check(host_bits(Ys), ref.cpu().numpy(), f"Y, smallest workspace, M={M}")
    assert ((Y.double() - Ys.double()).abs() <= 2.0 ** -7 * Ys.double().abs() + h * 2.0 ** -24 * ref.abs().max()).all()


@pytest.mark.parametrize("M,h,o,r", [(2, 4096, 320, 256), (5, 1600, 1088, 112), (9, 320, 64, 80), (17, 1600, 1088, 256), (31, 1088, 2112, 128),
                                      (40, 512, 704, 208), (33, 1600, 11008, 144)])
def test_finalize_sums_every_quadruple(synth, M, h, o, r):
    """T of several quadruples of ranks per thread, of one to eight partials, tokens that do not fill the last tile of 16, on few
    workgroups and on many (the widest output): forward without Double Quantization and dX, against fp64 products.  T_save is
    checked too: 16 significant bits of sums of h terms."""
    import paper_2305_14314_amd as ql
    s = 0.5
    g = torch.Generator(device="cuda")
    g.manual_seed(6000 + M)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    Wq = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 6100 + M), dq_blocksize=0)
    What = ql.qlora_nf4_dequant(Wq).double()
    X, dY, L1, L2 = bf(M, h), bf(M, o), bf(h, r, sd=0.05), bf(r, o, sd=0.05)
    print(f"case finalize M={M} h={h} o={o} r={r}", flush=True)
    T = torch.full((M, 2 * r), float("nan"), dtype=torch.bfloat16, device="cuda")
    Y = ql.qlora_linear_fwd(X, Wq, L1, L2, s, T_save=T)
    dX, _, _ = ql.qlora_linear_bwd(dY, None, Wq, L1, L2, s, need_dL=False)
    t = X.double() @ L1.double()
    _check(host_bits(Y), (X.double() @ What + s * t @ L2.double()).cpu().numpy(), "Y")
    _check(host_bits(dX), (dY.double() @ What.T + s * (dY.double() @ L2.double().T) @ L1.double().T).cpu().numpy(), "dX")
    got = T[:, :r].double() + T[:, r:].double()
    assert (got - t).abs().max() <= 2.0 ** -14 * t.abs().max() + 1e-6
