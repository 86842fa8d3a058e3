"""Adapter products whose inner sum overflows: T = X L1 (U = dY L2^T) is infinite for one token although every input is finite.
The term s T L2 is then infinite, as the product of the fp32 value is, whatever number of bf16 terms a path multiplies T in; the
other tokens stay what they are.  Up to 16 tokens, where T is multiplied whole, also a finite T that rounds to an infinite bf16 value."""
import pytest
import torch

from test_boundary import accepted_workspace
from test_gpu_fused_bwd import _gemm_launches

pytestmark = pytest.mark.gpu

N, R, S = 768, 48, 0.5


def _case(M, bwd, seed, whole, K=512):
    """Token operand A (M x K), inner P (K x R) and outer Q (R x N) matrix, weight; token 1: an infinite T[0]; token 2: T[1] just
    below fp32's largest value, above the largest finite bf16 value's rounding bound."""
    import paper_2305_14314_amd as ql
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rnd = lambda *shape, sd=1.0: torch.empty(shape, device="cuda").normal_(0, sd, generator=g)
    A, P, Q = rnd(M, K), rnd(K, R, sd=0.05), rnd(R, N, sd=0.05)
    Q[0] = torch.where(Q[0] >= 0, 0.05, -0.05)
    A[:, :2], P[:2] = 0, 0
    A[1, 0] = P[0, 0] = 2.0 ** 100
    if whole:
        A[2, 1], P[1, 1] = 181 / 128 * 2.0 ** 63, 181 / 128 * 2.0 ** 64   # T[2, 1] = 1.9996 * 2^127
        Q[1] *= 2.0 ** -50
    A, P, Q = A.bfloat16(), P.bfloat16(), Q.bfloat16()
    Wf = rnd(*((N, K) if bwd else (K, N)), sd=0.02)
    Wq = ql.qlora_nf4_quantize(Wf)
    What = ql.qlora_nf4_dequant(Wq).double()
    ref = A.double() @ (What.T if bwd else What) + S * (A.double() @ P.double()) @ Q.double()
    return Wq, A, P, Q, ref


def _check(out, Q, ref, tag):
    out = out.double()
    assert torch.equal(out[1], Q[0].double().sign() * float("inf")), tag
    keep = [m for m in range(out.shape[0]) if m != 1]
    for m in keep:                                            # per token: one is of another magnitude
        assert (out[m] - ref[m]).abs().max() <= 2.0 ** -7 * ref[m].abs().max(), (tag, m)


@pytest.mark.parametrize("bwd", [False, True])
@pytest.mark.parametrize("M", [4, 11, 16, 40])
def test_overflowing_adapter_sum(M, bwd):
    """One layer; up to 16 tokens with the workspace that the streaming kernels take (as well)."""
    import paper_2305_14314_amd as ql
    Wq, A, P, Q, ref = _case(M, bwd, 70 + M, M <= 16, 512 if M <= 16 else 2048)
    h, o = Wq.rows, Wq.cols
    sizes = [None] if M > 16 else [None, accepted_workspace(ql.binding.lib(), bwd, M, h, o, R)]
    for n in sizes:
        print(f"case overflow M={M} bwd={bwd} workspace={n}", flush=True)
        ws = None if n is None else ql.workspace_alloc(n)
        if bwd:
            call = lambda: ql.qlora_linear_bwd(A, None, Wq, Q.T.contiguous(), P.T.contiguous(), S, need_dL=False, workspace=ws)[0]
        else:
            call = lambda: ql.qlora_linear_fwd(A, Wq, P, Q, S, workspace=ws)
        out, gemms = _gemm_launches(ql, call)
        assert gemms == 0                                     # the streaming kernels, or the product that decodes the weight
        _check(out, Q, ref, (M, bwd, n))


@pytest.mark.parametrize("M", [4, 16])
def test_overflowing_adapter_sum_several_layers(M):
    import paper_2305_14314_amd as ql
    for bwd in (False, True):
        print(f"case overflow list M={M} bwd={bwd}", flush=True)
        cases = [_case(M, bwd, 90 + M + l, True) for l in range(3)]
        As, Ws, ss = [c[1] for c in cases], [c[0] for c in cases], [S] * 3
        if bwd:
            outs = ql.qlora_linear_bwd_list(As, Ws, [c[3].T.contiguous() for c in cases], [c[2].T.contiguous() for c in cases], ss)
        else:
            outs = ql.qlora_linear_fwd_list(As, Ws, [c[2] for c in cases], [c[3] for c in cases], ss)
        for out, c in zip(outs, cases):
            _check(out, c[3], c[4], ("list", M, bwd))
    Wq, A, P, Q, ref = _case(M, False, 99 + M, True)
    for out in ql.qlora_linear_fwd_multi(A, [Wq, Wq], [P, P], [Q, Q], [S, S]):
        _check(out, Q, ref, ("multi", M))
