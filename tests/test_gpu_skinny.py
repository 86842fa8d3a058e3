"""GPU parity of the skinny adapter products where their batching changes course: eight products and twelve finalize jobs
of four layers in a launch, layers too small to lend their weight's place (one layer at a time), the largest contraction
that finishes in the product's own epilogue (256 tokens) and the smallest that does not, ranks that are padded."""
import numpy as np
import pytest
import torch

from gpu_util import bits_f64, dev_bf16, host_bits, upload_quant
from test_gpu_linear import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("save", [False, True])
@pytest.mark.parametrize("M,h,outs,ranks", [(520, 704, [1024, 320, 768, 64], [16, 96, 80, 32]),
                                            (1500, 64, [64, 128], [16, 48]), (256, 192, [64, 320, 128], [64, 0, 144]),
                                            (257, 192, [64, 320, 128], [64, 0, 144]), (700, 128, [192], [256])])
def test_stacked_batches(oracle, synth, M, h, outs, ranks, save):
    import paper_2305_14314_amd as ql
    n, ss = len(outs), [0.5, 1.0, 0.25, 2.0][:len(outs)]
    print(f"case skinny batches M={M} h={h} o={outs} r={ranks} save={save}", flush=True)
    hX, hdY = synth.normal_bf16((M, h), 1.0, 9000 + M), synth.normal_bf16((M, sum(outs)), 1.0, 9001 + M)
    Wqs, Whats, hL1, hL2 = [], [], [], []
    for l, (o, r) in enumerate(zip(outs, ranks)):
        q = oracle.nf4_quantize(synth.normal_f32((h, o), synth.SIGMA_W, 9100 + l))
        Wqs.append(upload_quant(q))
        Whats.append(oracle.nf4_dequant(q))
        hL1.append(synth.normal_bf16((h, r), 0.05, 9200 + l) if r else None)
        hL2.append(synth.normal_bf16((r, o), 0.05, 9300 + l) if r else None)
    L1s = [dev_bf16(a) if a is not None else None for a in hL1]
    L2s = [dev_bf16(a) if a is not None else None for a in hL2]
    X, dY = dev_bf16(hX), dev_bf16(hdY)
    Ts = [torch.empty((M, 2 * r), dtype=torch.bfloat16, device="cuda") if r else None for r in ranks]
    ws = ql.workspace_alloc(ql.qlora_linear_fwd_stacked_sizes(M, h, outs, ranks))
    ws[ql.binding.WORKSPACE_HEADER_BYTES:].fill_(0x7F)
    Y = ql.qlora_linear_fwd_stacked(X, Wqs, L1s, L2s, ss, T_saves=Ts, workspace=ws)
    ws = ql.workspace_alloc(ql.qlora_linear_bwd_stacked_sizes(M, h, outs, ranks))
    ws[ql.binding.WORKSPACE_HEADER_BYTES:].fill_(0x7F)
    dX, dL1s, dL2s = ql.qlora_linear_bwd_stacked(dY, X, Wqs, L1s, L2s, ss, T_saveds=Ts if save else None, workspace=ws)
    torch.cuda.synchronize()
    Yh, n0, ref_dx = host_bits(Y), 0, 0.0
    for l, (o, r) in enumerate(zip(outs, ranks)):
        dYl = np.ascontiguousarray(hdY[:, n0:n0 + o])
        _check(Yh[:, n0:n0 + o], oracle.linear_fwd(hX, Whats[l], hL1[l], hL2[l], ss[l]), f"layer {l} Y")
        ref_dx = ref_dx + oracle.linear_bwd_dx(dYl, Whats[l], hL1[l], hL2[l], ss[l])
        if r:
            t = host_bits(Ts[l])
            want = bits_f64(hX) @ bits_f64(hL1[l])
            # hi + lo: 16 significant bits, and an fp32 sum of h terms
            assert np.abs(bits_f64(t[:, :r]) + bits_f64(t[:, r:]) - want).max() <= 2.0 ** -14 * np.abs(want).max() + 1e-6
            r1, r2 = oracle.linear_bwd_dl(dYl, hX, hL1[l], hL2[l], ss[l])
            _check(host_bits(dL1s[l]), r1, f"layer {l} dL1")
            _check(host_bits(dL2s[l]), r2, f"layer {l} dL2")
        n0 += o
    _check(host_bits(dX), ref_dx, "dX")


@pytest.mark.parametrize("kind,M,h", [("nf4", 4000, 256), ("nf4", 4000, 64), ("int8", 500, 256), ("stacked", 4000, 256)])
def test_saving_t_does_not_change_y(synth, kind, M, h):
    """Inference and training forward give the same bits: the order in which T = X L1 is summed does not depend on whether
    the call saves it (four K-steps and fewer, where a product without splits is possible)."""
    import paper_2305_14314_amd as ql
    o, r = 512, 64
    W = torch.from_numpy(synth.normal_f32((h, o), synth.SIGMA_W, 9500)).cuda()
    Wq = ql.qlora_quantize_int8(W) if kind == "int8" else ql.qlora_nf4_quantize(W)
    X = dev_bf16(synth.normal_bf16((M, h), 1.0, 9501))
    L1, L2 = dev_bf16(synth.normal_bf16((h, r), 0.5, 9502)), dev_bf16(synth.normal_bf16((r, o), 0.5, 9503))
    T = torch.empty((M, 2 * r), dtype=torch.bfloat16, device="cuda")
    print(f"case Y with and without T_save: {kind} M={M} h={h}", flush=True)
    if kind == "stacked":
        f = lambda t: ql.qlora_linear_fwd_stacked(X, [Wq, Wq], [L1, L1], [L2, L2], [1.0, 1.0], T_saves=[t, None])
    else:
        f = lambda t: ql.qlora_linear_fwd(X, Wq, L1, L2, 1.0, T_save=t)
    a, b = f(None), f(T)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


# dL1 and dL2 in one launch with a floor under the smaller one's workgroups; in launches of their own with a shared launch's
# splits (short chains) and with their own; finished in the epilogue
@pytest.mark.parametrize("M,h,o,r", [(1024, 2048, 2048, 64), (640, 320, 1088, 64), (2048, 2048, 64, 256), (2048, 64, 2048, 256),
                                      (200, 320, 1088, 48)])
def test_gradients_alone_and_together(oracle, synth, M, h, o, r):
    """Each gradient against the oracle, and the same bits whether the call wants the other or not."""
    import paper_2305_14314_amd as ql
    s = 0.5
    hX, hdY = synth.normal_bf16((M, h), 1.0, 9600), synth.normal_bf16((M, o), 1.0, 9601)
    hL1, hL2 = synth.normal_bf16((h, r), 0.05, 9602), synth.normal_bf16((r, o), 0.05, 9603)
    Wq = upload_quant(oracle.nf4_quantize(synth.normal_f32((h, o), synth.SIGMA_W, 9604)))
    X, dY, L1, L2 = (dev_bf16(a) for a in (hX, hdY, hL1, hL2))
    print(f"case gradients alone and together M={M} h={h} o={o} r={r}", flush=True)
    _, dL1, dL2 = ql.qlora_linear_bwd(dY, X, Wq, L1, L2, s)
    got = []
    for want in ((True, True), (True, False), (False, True)):
        a1 = torch.zeros((h, r), device="cuda") if want[0] else None
        a2 = torch.zeros((r, o), device="cuda") if want[1] else None
        ql.qlora_linear_bwd_acc(dY, X, Wq, L1, L2, s, a1, a2)
        got.append((a1, a2))
    torch.cuda.synchronize()
    r1, r2 = oracle.linear_bwd_dl(hdY, hX, hL1, hL2, s)
    _check(host_bits(dL1), r1, "dL1")
    _check(host_bits(dL2), r2, "dL2")
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[2][1])
