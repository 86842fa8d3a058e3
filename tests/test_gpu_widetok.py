"""Forward and input gradient by the kernels whose waves share one decode of the weight: every tile shape in both directions, with tokens,
outputs and contractions that do not fill a tile, a slab or a step, against fp64 products with the dequantised weight."""
import ctypes

import pytest
import torch

from gpu_util import host_bits
from test_gpu_fused_bwd import _gemm_launches
from test_gpu_linear import _check

pytestmark = pytest.mark.gpu


class _Plan(ctypes.Structure):
    _fields_ = ([("ok", ctypes.c_bool)] + [(n, ctypes.c_int) for n in ("MF", "BN", "n_tg", "n_slabs", "steps", "k_pad", "n_lparts", "chunk")] +
                [(n, ctypes.c_size_t) for n in ("lpart_floats", "pack_elems")] + [("us", ctypes.c_double)])


def _plan(bwd, M, h, o, r):
    """The plan of a call with room for it (the library's internal struct)."""
    from paper_2305_14314_amd import binding
    f = ctypes.CDLL(binding.LIB_PATH)._ZN5qlora9wide_planEblllim
    f.restype, f.argtypes = _Plan, [ctypes.c_bool, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t]
    return f(bwd, M, h, o, r, h * o * 2 if bwd else 1 << 40)   # the dequantised weight's place; forward the reported size brings what it needs


# A step is 128 elements of the contraction with slabs of 128 outputs, else 256: contractions that end in a quarter, half or three
# quarters of one; a single step, odd and even numbers of them; the last slab of 128 half empty; ranks none, below 32, above 64 (several
# passes), the largest; a few tokens in the last tile, and a full one
@pytest.mark.parametrize("tile,bwd,M,h,o,r,dtype,dq,drop", [
    ((1, 64), False, 390, 5248, 1728, 64, "NF4", 256, 0.0), ((1, 64), True, 244, 2112, 1664, 48, "NF4", 256, 0.0),
    ((2, 64), False, 481, 2880, 2496, 80, "NF4", 256, 0.0), ((2, 64), True, 159, 7488, 2176, 32, "NF4", 0, 0.3),
    ((3, 64), False, 377, 1920, 6976, 16, "FP4_E2M1", 256, 0.0), ((3, 64), True, 472, 4928, 7616, 96, "NF4", 256, 0.2),
    ((4, 64), False, 411, 5696, 6464, 64, "NF4", 256, 0.1), ((4, 64), True, 419, 7360, 1728, 48, "INT4", 256, 0.0),
    ((1, 128), False, 198, 1408, 6208, 160, "NF4", 256, 0.0), ((1, 128), True, 138, 9536, 384, 48, "NF4", 256, 0.5),
    ((2, 128), False, 457, 1664, 6592, 80, "NF4", 0, 0.0), ((2, 128), True, 199, 13248, 1728, 128, "NF4", 256, 0.0),
    ((3, 128), False, 278, 2176, 11328, 0, "NF4", 256, 0.0), ((3, 128), True, 361, 11584, 1984, 0, "NF4", 256, 0.0),
    ((1, 128), False, 63, 128, 1472, 0, "NF4", 256, 0.0), ((1, 128), True, 34, 1728, 128, 32, "NF4", 256, 0.0),
    ((3, 128), False, 333, 5120, 13824, 128, "NF4", 256, 0.2), ((4, 64), False, 512, 8192, 8192, 256, "NF4", 256, 0.0),
    ((3, 128), False, 768, 8192, 8192, 64, "NF4", 256, 0.0),
    ((2, 64), True, 512, 4096, 4096, 64, "NF4", 256, 0.1),
    # up to the most tokens; from the third on more tiles than compute units
    ((2, 64), False, 1412, 5952, 1280, 32, "NF4", 256, 0.0), ((1, 64), False, 1252, 9984, 256, 64, "NF4", 256, 0.0),
    ((2, 64), False, 808, 4864, 4672, 0, "NF4", 256, 0.0), ((2, 64), True, 896, 4672, 11008, 16, "NF4", 256, 0.1),
    ((3, 128), True, 1618, 6848, 512, 64, "NF4", 256, 0.2), ((2, 128), True, 1376, 5632, 896, 64, "NF4", 0, 0.1),
    ((4, 64), True, 1760, 4672, 1280, 64, "NF4", 256, 0.1), ((3, 128), True, 1126, 5120, 6656, 0, "NF4", 256, 0.0),
    ((3, 128), True, 2048, 8192, 640, 64, "NF4", 256, 0.1)])
def test_widetok(synth, tile, bwd, M, h, o, r, dtype, dq, drop):
    import paper_2305_14314_amd as ql
    s = 0.5
    g = torch.Generator(device="cuda")
    g.manual_seed(7000 + M)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    Wq = ql.qlora_quantize_4bit(synth.normal_f32_device((h, o), synth.SIGMA_W, 7100 + M), getattr(ql, dtype), dq_blocksize=dq)
    What = ql.qlora_nf4_dequant(Wq).double()
    X, dY = bf(M, h), bf(M, o)
    L1, L2 = (bf(h, r, sd=0.05), bf(r, o, sd=0.05)) if r else (None, None)
    keep = torch.rand((M, h), device="cuda", generator=g) >= drop
    mask, D = ql.pack_keep_mask(keep), keep.double() / (1.0 - drop)
    plan, head = _plan(bwd, M, h, o, r), ql.binding.WORKSPACE_HEADER_BYTES
    assert plan.ok and (plan.MF, plan.BN) == tile
    need = (max(ql.qlora_linear_dropout_sizes(M, h, o, r)) if drop else
            (ql.qlora_linear_bwd_sizes if bwd else ql.qlora_linear_fwd_sizes)(M, h, o, r))
    ws = ql.workspace_alloc(need + 4096)
    ws[head:].fill_(0x7F)                                      # stale contents: NaN-ish everywhere
    T = torch.full((M, 2 * r), float("nan"), dtype=torch.bfloat16, device="cuda") if r else None
    print(f"case wide {tile} bwd={bwd} M={M} h={h} o={o} r={r} {dtype} dq={dq} drop={drop}", flush=True)

    def call():
        if bwd and drop:
            return ql.qlora_linear_bwd_dropout(dY, X, Wq, L1, L2, s, mask, drop, need_dL=False, workspace=ws[:need])[0]
        if bwd:
            return ql.qlora_linear_bwd(dY, X, Wq, L1, L2, s, need_dL=False, workspace=ws[:need])[0]
        if drop:
            return ql.qlora_linear_fwd_dropout(X, Wq, L1, L2, s, mask, drop, T_save=T, workspace=ws[:need])
        return ql.qlora_linear_fwd(X, Wq, L1, L2, s, T_save=T, workspace=ws[:need])

    out, n = _gemm_launches(ql, call)
    torch.cuda.synchronize()
    assert n == 0 and int((ws[need:] != 0x7F).sum()) == 0
    # which path ran shows in how much of the workspace was written: the partials of T, and behind them the packed operand
    used = int((ws[head:need] != 0x7F).nonzero().max()) + 1
    assert abs(used - ((plan.lpart_floats * 4 + 255) // 256 * 256 + plan.pack_elems * 2)) < 16
    x, y = X.double(), dY.double()
    if bwd:
        ref = y @ What.T
        if r:
            ref = ref + s * (D if drop else 1.0) * ((y @ L2.double().T) @ L1.double().T)
    else:
        ref = x @ What
        if r:
            t = (x * (keep if drop else 1.0)) @ L1.double()
            ref = ref + s / (1.0 - drop) * (t @ L2.double())
            got = T[:, :r].double() + T[:, r:].double()        # 16 significant bits
            assert (got - t).abs().max() <= 2.0 ** -14 * t.abs().max() + 1e-6
    _check(host_bits(out), ref.cpu().numpy(), "dX" if bwd else "Y")
    # half a bf16 step (2^-8 of the value at most), the fp32 sums and the 16 bits that T keeps: one rounding, under dropout too
    err, rms = (out.double() - ref).abs(), ref.square().mean().sqrt()
    assert (err <= 2.0 ** -8 * ref.abs() + 2e-4 * rms).all()
    assert torch.equal(call().view(torch.int16), out.view(torch.int16))      # the same bits again, on a used workspace


def test_widetok_infinite_t(synth):
    """A U that overflows makes its token's outputs infinite, with the outer matrix' sign, as an fp32 product would."""
    import paper_2305_14314_amd as ql
    M, h, o, r = 250, 2112, 1664, 64
    assert _plan(True, M, h, o, r).ok
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    Wq = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 8))
    dY, L1 = bf(M, o), torch.zeros((h, r), dtype=torch.bfloat16, device="cuda")
    L2 = torch.full((r, o), 3e38, dtype=torch.bfloat16, device="cuda")
    dY[5] = 1.0
    L1[:] = torch.where(torch.arange(h, device="cuda") % 2 == 0, 1.0, -1.0).bfloat16()[:, None]
    dX = ql.qlora_linear_bwd(dY, None, Wq, L1, L2, 1.0, need_dL=False)[0]
    assert torch.equal(dX[5].float(), L1[:, 0].float() * float("inf"))


def test_widetok_infinite_t_forward_and_under_dropout(synth):
    """The same in the forward pass, and under dropout where an input element is kept; a dropped one gets the frozen product alone."""
    import paper_2305_14314_amd as ql
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    signs = lambda n: torch.where(torch.arange(n, device="cuda") % 2 == 0, 1.0, -1.0).bfloat16()
    big = lambda *shape: torch.full(shape, 3e38, dtype=torch.bfloat16, device="cuda")
    M, h, o, r = 1412, 5952, 1280, 32
    Wq, X, L2 = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 14)), bf(M, h), signs(o).repeat(r, 1)
    X[5] = 1.0
    Y, n = _gemm_launches(ql, lambda: ql.qlora_linear_fwd(X, Wq, big(h, r), L2, 1.0))
    assert n == 0 and torch.equal(Y[5].float(), signs(o).float() * float("inf"))
    M, h, o, r = 1618, 6848, 512, 64
    Wq, dY, L1 = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 15)), bf(M, o), signs(h)[:, None].repeat(1, r)
    dY[5] = 1.0
    keep = torch.rand((M, h), device="cuda", generator=g) >= 0.3
    dX, n = _gemm_launches(ql, lambda: ql.qlora_linear_bwd_dropout(dY, None, Wq, L1, big(r, o), 1.0, ql.pack_keep_mask(keep), 0.3, need_dL=False)[0])
    assert n == 0 and torch.equal(dX[5][keep[5]].float(), signs(h)[keep[5]].float() * float("inf"))
    frozen = (dY[5].double() @ ql.qlora_nf4_dequant(Wq).double().T)[~keep[5]]
    assert ((dX[5][~keep[5]].double() - frozen).abs() <= 2.0 ** -8 * frozen.abs() + 2e-4 * frozen.square().mean().sqrt()).all()


@pytest.mark.parametrize("M,h,o,r,drop", [(639, 12480, 9280, 64, 0.0), (1376, 5632, 896, 64, 0.1), (1212, 1472, 1792, 16, 0.0), (1131, 1600, 9600, 32, 0.0)])
def test_adapter_gradient_from_the_u_it_leaves(synth, M, h, o, r, drop):
    """dL1 of a call whose dX takes this path: the [hi | lo] pair of U that the first slab's workgroups write."""
    import paper_2305_14314_amd as ql
    s = 0.5
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    Wq = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 16))
    X, dY, L1, L2 = bf(M, h), bf(M, o), bf(h, r, sd=0.05), bf(r, o, sd=0.05)
    keep = torch.rand((M, h), device="cuda", generator=g) >= drop
    if drop:
        call = lambda: ql.qlora_linear_bwd_dropout(dY, X, Wq, L1, L2, s, ql.pack_keep_mask(keep), drop)
    else:
        call = lambda: ql.qlora_linear_bwd(dY, X, Wq, L1, L2, s)
    print(f"case M={M} h={h} o={o} r={r} drop={drop}", flush=True)
    (dX, dL1, dL2), n = _gemm_launches(ql, call)
    assert n == 0
    x, y, a, b = X.double() * keep / (1.0 - drop), dY.double(), L1.double(), L2.double()
    U = y @ b.T
    da = s * (U @ a.T)
    _check(host_bits(dX), (y @ ql.qlora_nf4_dequant(Wq).double().T + (da * keep / (1.0 - drop))).cpu().numpy(), "dX")
    ref = s * (x.T @ U)
    _check(host_bits(dL1), ref.cpu().numpy(), "dL1")
    # half a bf16 step, fp32 sums, and the 16 significant bits of U's pair
    assert ((dL1.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2e-4 * ref.square().mean().sqrt()).all()
    _check(host_bits(dL2), (s * ((x @ a).T @ y)).cpu().numpy(), "dL2")


@pytest.mark.parametrize("M,h,o,r,here", [(1536, 8192, 1024, 64, False), (2000, 4096, 1024, 64, False), (1412, 5952, 1280, 32, True),
                                           (700, 8192, 512, 0, True), (1252, 9984, 256, 64, True)])
def test_forward_bits_do_not_follow_the_workspace(synth, M, h, o, r, here):
    """Fewer outputs than tokens, so that the packed operand is larger than the dequantised weight: the same bits with the reported
    workspace, with a larger one, and behind a wider layer whose workspace both share (`here`: by this path)."""
    import paper_2305_14314_amd as ql
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    W = [ql.qlora_nf4_quantize(synth.normal_f32_device((h, n), synth.SIGMA_W, 11 + n)) for n in (o, 4 * o)]
    X = bf(M, h)
    L = [(bf(h, r, sd=0.05), bf(r, n, sd=0.05)) if r else (None, None) for n in (o, 4 * o)]
    print(f"case M={M} h={h} o={o} r={r}", flush=True)
    need = ql.qlora_linear_fwd_sizes(M, h, o, r)
    want, n = _gemm_launches(ql, lambda: ql.qlora_linear_fwd(X, W[0], *L[0], 0.5, workspace=ql.workspace_alloc(need)))
    assert n == (0 if here else 1)
    for more in (256, 16 << 20, 64 << 20):
        got = ql.qlora_linear_fwd(X, W[0], *L[0], 0.5, workspace=ql.workspace_alloc(need + more))
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), more
    got = ql.qlora_linear_fwd_multi(X, W, [l[0] for l in L], [l[1] for l in L], [0.5, 0.5])[0]
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    _check(host_bits(want), (X.double() @ ql.qlora_nf4_dequant(W[0]).double() +
                             (0.5 * (X.double() @ L[0][0].double()) @ L[0][1].double() if r else 0.0)).cpu().numpy(), "Y")


@pytest.mark.parametrize("M,h,o,here", [(768, 1024, 8192, (0, 16)), (1024, 4096, 4096, (0,)), (768, 8192, 8192, (0, 16)), (640, 960, 2048, (0, 16))])
def test_backward_modes_above_512_tokens(synth, M, h, o, here):
    """Modes 0 and 1 dequantise and decode inside the GEMM, one launch of it each, and give the same bits without an adapter whatever the
    weight's size; the default, mode 2, takes this path where it is estimated faster (`here`: with these ranks)."""
    import paper_2305_14314_amd as ql
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    Wq, dY, L1, L2 = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 12)), bf(M, o), bf(h, 16, sd=0.05), bf(16, o, sd=0.05)
    What = ql.qlora_nf4_dequant(Wq).double()
    out = {}
    for mode in (2, 0, 1):
        prev = ql.qlora_bwd_fused_dequant(mode)
        try:
            for r in (0, 16):
                print(f"case M={M} h={h} o={o} r={r} mode={mode}", flush=True)
                a = (L1, L2, 0.5) if r else (None, None, 0.0)
                out[mode, r], n = _gemm_launches(ql, lambda: ql.qlora_linear_bwd(dY, None, Wq, *a, need_dL=False)[0])
                assert n == (0 if mode == 2 and r in here else 1)
                ref = dY.double() @ What.T + (0.5 * (dY.double() @ L2.double().T) @ L1.double().T if r else 0.0)
                _check(host_bits(out[mode, r]), ref.cpu().numpy(), f"dX mode {mode}")
        finally:
            ql.qlora_bwd_fused_dequant(prev)
        assert prev == 2
    assert torch.equal(out[0, 0].view(torch.int16), out[1, 0].view(torch.int16))


@pytest.mark.parametrize("M,h,o,r", [(512, 4096, 4096, 64), (1555, 5504, 128, 64)])
def test_mask_at_any_address(synth, M, h, o, r):
    """The keep-bits are bytes: dX, and U with it (dL1), have the same bits wherever the mask lies."""
    import paper_2305_14314_amd as ql
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    bf = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g).bfloat16()
    Wq = ql.qlora_nf4_quantize(synth.normal_f32_device((h, o), synth.SIGMA_W, 13))
    X, dY, L1, L2 = bf(M, h), bf(M, o), bf(h, r, sd=0.05), bf(r, o, sd=0.05)
    mask = ql.pack_keep_mask(torch.rand((M, h), device="cuda", generator=g) >= 0.1).flatten()
    room = torch.zeros(mask.numel() + 16, dtype=torch.uint8, device="cuda")
    want = None
    for at in (0, 1, 3, 4, 6):
        print(f"case M={M} h={h} o={o} mask at {at}", flush=True)
        m = room[at:at + mask.numel()]
        m.copy_(mask)
        got, n = _gemm_launches(ql, lambda: ql.qlora_linear_bwd_dropout(dY, X, Wq, L1, L2, 0.5, m, 0.1))
        assert m.data_ptr() % 8 == at and n == 0
        got = [t.view(torch.int16) for t in got]
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), at
