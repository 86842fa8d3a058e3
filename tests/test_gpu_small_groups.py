"""dL1 and dL2 finished in their products' launch: every number of groups of waves to a tile (1, 2 and 4), with tokens, outputs
and ranks that end inside a tile, groups that get fewer K-steps than others or none, and each rule on either side of its line."""
import numpy as np
import pytest
import torch

from gpu_util import bits_f64, dev_bf16, host_bits, upload_quant

pytestmark = pytest.mark.gpu


# 65 tokens two groups; 129 and 200 four, one of them idle; 257 and 300 four of two K-steps, the last idle; 449 and 512; 577 with 51 and 48
# tiles by partials; 640 and 1500 with 194 in four groups; 330, 577 and 1500 with more tiles than CUs (two groups; one from 512 on); 200 with 544 (one)
@pytest.mark.parametrize("M,h,o,r", [(65, 64, 192, 16), (129, 320, 64, 48), (200, 1088, 320, 80), (257, 64, 64, 16), (300, 1088, 448, 112),
                                      (449, 192, 4160, 64), (512, 256, 256, 256), (577, 1664, 1600, 16), (577, 1536, 1536, 16),
                                      (577, 2112, 2240, 256), (1500, 4160, 4096, 256), (200, 4352, 4352, 256), (1025, 3584, 2048, 144),
                                      (640, 3072, 3136, 96), (330, 4160, 2048, 256), (1500, 3072, 3136, 128)])
@pytest.mark.parametrize("dropout", [False, True])
def test_gradients_in_groups(synth, M, h, o, r, dropout):
    """Both gradients in bf16 and added to fp32 sums, with T saved and recomputed, against float64 on the same bf16 operands.  Their
    exact value within (2^-16 + (n + M) 2^-24) of the sum of its terms' magnitudes: T and U enter as [hi | lo] pairs of 16 significant
    bits and are fp32 sums of n = h or o terms, the gradients fp32 sums of M; bf16 rounds once more."""
    import paper_2305_14314_amd as ql
    s, p = 0.5, 0.25
    hX, hdY = synth.normal_bf16((M, h), 1.0, 9700), synth.normal_bf16((M, o), 1.0, 9701)
    hL1, hL2 = synth.normal_bf16((h, r), 0.05, 9702), synth.normal_bf16((r, o), 0.05, 9703)
    X, dY, L1, L2 = (dev_bf16(a) for a in (hX, hdY, hL1, hL2))
    Wq = ql.qlora_nf4_quantize(torch.from_numpy(synth.normal_f32((h, o), synth.SIGMA_W, 9704)).cuda())
    print(f"case gradients in groups M={M} h={h} o={o} r={r} dropout={dropout}", flush=True)
    keep = np.ones((M, h))
    T = torch.empty((M, 2 * r), dtype=torch.bfloat16, device="cuda")
    a1, a2 = torch.ones((h, r), device="cuda"), torch.ones((r, o), device="cuda")
    if dropout:
        keep = np.random.default_rng(9705).random((M, h)) >= p
        mask = torch.from_numpy(np.packbits(keep.reshape(-1), bitorder="little")).cuda()
        ql.qlora_linear_fwd_dropout(X, Wq, L1, L2, s, mask, p, T_save=T)
        got = [ql.qlora_linear_bwd_dropout(dY, X, Wq, L1, L2, s, mask, p, T_saved=t)[1:] for t in (T, None)]
        ql.qlora_linear_bwd_dropout(dY, X, Wq, L1, L2, s, mask, p, T_saved=T, dL1_acc=a1, dL2_acc=a2)
        s /= 1.0 - p
    else:
        ql.qlora_linear_fwd(X, Wq, L1, L2, s, T_save=T)
        got = [ql.qlora_linear_bwd(dY, X, Wq, L1, L2, s, T_saved=t)[1:] for t in (T, None)]
        ql.qlora_linear_bwd_acc(dY, X, Wq, L1, L2, s, a1, a2, T_saved=T)
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0])                 # dL1 does not read T
    X64, dY64, A64, B64 = bits_f64(hX) * keep, bits_f64(hdY), bits_f64(hL1), bits_f64(hL2)
    want = (s * X64.T @ (dY64 @ B64.T), s * (X64 @ A64).T @ dY64)
    mags = (s * np.abs(X64).T @ (np.abs(dY64) @ np.abs(B64).T), s * (np.abs(X64) @ np.abs(A64)).T @ np.abs(dY64))
    for i, (n, acc) in enumerate(((o, a1), (h, a2))):
        bound = (2.0 ** -16 + (n + M) * 2.0 ** -24) * mags[i]
        err = np.abs(acc.cpu().double().numpy() - 1.0 - want[i])
        assert (err <= bound + 2.0 ** -23 * (1.0 + np.abs(want[i]))).all(), (i, "fp32 sum", float((err / bound).max()))
        for form in (0, 1):
            err = np.abs(bits_f64(host_bits(got[form][i])) - want[i])
            assert (err <= bound + 2.0 ** -8 * np.abs(want[i])).all(), (i, form, float((err / bound).max()))


# two groups and four, four and none, none; a rank of 0 between
@pytest.mark.parametrize("M,h,outs,ranks", [(757, 128, [4416, 768], [256, 256]), (450, 128, [2048, 64, 4416], [256, 0, 256]),
                                            (780, 640, [256, 768, 1536], [64, 64, 64]), (300, 64, [64, 192], [64, 48])])
def test_stacked_layers_one_by_one(synth, M, h, outs, ranks):
    """The gradients of stacked layers with too little room for one launch, each layer's in the groups of its own launch; T saved and recomputed.
    The bound is the one above."""
    import paper_2305_14314_amd as ql
    ss = [0.5 + l for l in range(len(outs))]
    hX, hdY = synth.normal_bf16((M, h), 1.0, 9800), synth.normal_bf16((M, sum(outs)), 1.0, 9801)
    hL = [(synth.normal_bf16((h, max(r, 1)), 0.05, 9810 + l), synth.normal_bf16((max(r, 1), o), 0.05, 9820 + l)) for l, (o, r) in enumerate(zip(outs, ranks))]
    Wqs = [ql.qlora_nf4_quantize(torch.from_numpy(synth.normal_f32((h, o), synth.SIGMA_W, 9830 + l)).cuda()) for l, o in enumerate(outs)]
    L1s, L2s = ([dev_bf16(p[i]) if r else None for p, r in zip(hL, ranks)] for i in (0, 1))
    Ts = [torch.empty((M, 2 * r), dtype=torch.bfloat16, device="cuda") if r else None for r in ranks]
    print(f"case stacked one by one M={M} h={h} o={outs} r={ranks}", flush=True)
    X, dY = dev_bf16(hX), dev_bf16(hdY)
    ql.qlora_linear_fwd_stacked(X, Wqs, L1s, L2s, ss, T_saves=Ts)
    for saved in (Ts, None):
        _, dL1s, dL2s = ql.qlora_linear_bwd_stacked(dY, X, Wqs, L1s, L2s, ss, T_saveds=saved)
        torch.cuda.synchronize()
        X64, n0 = bits_f64(hX), 0
        for l, (o, r) in enumerate(zip(outs, ranks)):
            g, n0 = bits_f64(hdY)[:, n0:n0 + o], n0 + o
            if not r:
                continue
            a, b, s = bits_f64(hL[l][0]), bits_f64(hL[l][1]), ss[l]
            want = (s * X64.T @ (g @ b.T), s * (X64 @ a).T @ g)
            mags = (s * np.abs(X64).T @ (np.abs(g) @ np.abs(b).T), s * (np.abs(X64) @ np.abs(a)).T @ np.abs(g))
            for i, (n, got) in enumerate(((o, dL1s[l]), (h, dL2s[l]))):
                err = np.abs(bits_f64(host_bits(got)) - want[i])
                assert (err <= (2.0 ** -16 + (n + M) * 2.0 ** -24) * mags[i] + 2.0 ** -8 * np.abs(want[i])).all(), (l, i)
