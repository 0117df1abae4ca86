"""The autograd layer on the GPU (bf16 parameters and activations, HIP
recurrence) against the same layer in fp64 on the CPU with the recurrence
computed by the oracle: output and the gradients of the input and of every
parameter, normwise (max|got-ref|/max|ref|) within the bf16 tolerance; the
scalar gate-bias gradient, a sum over every (token, head), relative to the
sum of its summands' magnitudes."""
import copy

import pytest
import torch

from paper_2606_08804_amd import layer
from tests import oracle_binding
from tests.gpu_helpers import TOL, normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_decay,varlen,fixed_lambda", [(True, False, None), (False, True, None),
                                                          (True, False, 0.0), (True, True, 0.5)])
def test_layer_matches_oracle_layer(monkeypatch, use_decay, varlen, fixed_lambda):
    torch.manual_seed(41)
    m = layer.QDeltaLayer(d_model=256, n_heads=2, head_dk=128, head_dv=128, use_decay=use_decay,
                          fixed_lambda=fixed_lambda)
    m = m.to(torch.bfloat16)
    ref = copy.deepcopy(m).double()
    g = torch.Generator().manual_seed(42)
    B, T = (1, 270) if varlen else (2, 150)
    h = torch.randn(B, T, 256, generator=g).to(torch.bfloat16)
    dy = torch.randn(B, T, 256, generator=g).to(torch.bfloat16)
    cu = torch.tensor([0, 70, 71, 270], dtype=torch.int32) if varlen else None

    mg = m.cuda()
    hg = h.cuda().requires_grad_()
    y = mg(hg, cu_seqlens=None if cu is None else cu.cuda())
    y.backward(dy.cuda())
    torch.cuda.synchronize()

    monkeypatch.setattr(layer, "_binding", oracle_binding)
    # the reference's lambda bias, broadcast to one copy per (token, head), so
    # that its gradient holds the summands of the scalar bias gradient
    if fixed_lambda is None:
        ref.lambda_bias = torch.nn.Parameter(ref.lambda_bias.detach().expand(B, T, ref.H).clone())
    hr = h.double().requires_grad_()
    yr = ref(hr, cu_seqlens=cu)
    yr.backward(dy.double())

    tol = TOL["bf16"]
    assert normwise(y.detach().cpu().double().numpy(), yr.detach().numpy()) <= tol
    assert normwise(hg.grad.cpu().double().numpy(), hr.grad.numpy()) <= tol
    for (name, p), (_, pr) in zip(mg.named_parameters(), ref.named_parameters()):
        if name == "lambda_bias":
            # a sum over every (token, head) with cancellation: its error is
            # measured against the sum of the summands' magnitudes
            terms = pr.grad
            err = abs(float(p.grad) - float(terms.sum())) / float(terms.abs().sum())
        else:
            err = normwise(p.grad.cpu().double().numpy(), pr.grad.numpy())
        assert err <= tol, (name, err)


def test_layer_continuation_with_carried_state():
    """Running a sequence in two calls, the second from the first's final
    state, equals one call over the whole sequence (output and final state)."""
    torch.manual_seed(43)
    m = layer.QDeltaLayer(d_model=256, n_heads=2, head_dk=128, head_dv=128).to(torch.bfloat16).cuda()
    g = torch.Generator().manual_seed(44)
    h = torch.randn(2, 200, 256, generator=g).to(torch.bfloat16).cuda()
    with torch.no_grad():
        y, S = m(h, output_final_state=True)
        y1, S1 = m(h[:, :77].contiguous(), output_final_state=True)
        y2, S2 = m(h[:, 77:].contiguous(), initial_state=S1, output_final_state=True)
    torch.cuda.synchronize()
    tol = TOL["bf16"]
    assert normwise(torch.cat([y1, y2], 1).float().cpu().numpy(), y.float().cpu().numpy()) <= tol
    assert normwise(S2.cpu().numpy(), S.cpu().numpy()) <= tol


@pytest.mark.parametrize("dt,D", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 128),
                                  (torch.float32, 64)])
def test_l2norm_kernels_match_normalize(dt, D):
    """Row normalisation of a strided slice of a fused projection (1001 rows,
    one of them zero, so clamped) against F.normalize and its gradient in fp64."""
    from paper_2606_08804_amd import qdelta
    g = torch.Generator().manual_seed(45)
    fused = torch.randn(7, 11, 13, 2 * D + 64, generator=g)
    fused[3, 4, 5] = 0.0
    fused = fused.to(dt)
    dy = torch.randn(7, 11, 13, D, generator=g).to(dt)
    x_cpu = fused[..., D:2 * D]                         # the k slice: strided rows
    xr = x_cpu.double().requires_grad_()
    yr = torch.nn.functional.normalize(xr, dim=-1, eps=1e-12)
    yr.backward(dy.double())
    x = fused.cuda()[..., D:2 * D]
    y, rn = qdelta.l2norm_fwd(x)
    dx = qdelta.l2norm_bwd(y, rn, dy.cuda())
    torch.cuda.synchronize()
    tol = TOL["bf16"] if dt == torch.bfloat16 else TOL["f32"]
    assert normwise(y.double().cpu().numpy(), yr.detach().numpy()) <= tol
    assert normwise(dx.double().cpu().numpy(), xr.grad.numpy()) <= tol
    assert float(rn[3, 4, 5]) < 0 and torch.all(y[3, 4, 5] == 0)


@pytest.mark.parametrize("dt,dk,dv,lengths", [(torch.bfloat16, 128, 128, None), (torch.bfloat16, 64, 256, None),
                                              (torch.bfloat16, 128, 64, [70, 0, 1, 199]), (torch.float32, 64, 128, None),
                                              (torch.float32, 64, 64, [64, 206])])
def test_fused_rows_equal_separate_tensors(dt, dk, dv, lengths):
    """The recurrence on the projection's rows in place against the same rows split into q, k and v tensors: equal
    outputs, gate and state gradients; the gradient of the rows (one row of q and one of k zero, so clamped) but for
    the order of the normalisation's sums y . dy, from the same rounded dq and dk.  128 products in another order
    differ by 2^-17 at most, so that one bf16 value in 2^8 may round the other way, by 2^-8: 2^-12 in the 2-norm."""
    g = torch.Generator().manual_seed(47)
    B, T, H = (1, 270, 3) if lengths else (2, 135, 3)
    N = len(lengths) if lengths else B
    cu = torch.tensor([0] + lengths, dtype=torch.int32).cumsum(0).to(torch.int32).cuda() if lengths else None
    qkv = torch.randn(B, T, H, 2 * dk + dv, generator=g)
    qkv[0, 5, 1, :dk] = 0.0
    qkv[0, 9, 2, dk:2 * dk] = 0.0
    qkv = qkv.to(dt).cuda()
    gates = [torch.sigmoid(torch.randn(B, T, H, generator=g)).cuda(), torch.sigmoid(torch.randn(B, T, H, generator=g)).cuda(),
             torch.nn.functional.logsigmoid(torch.randn(B, T, H, generator=g)).cuda()]
    S0 = (0.1 * torch.randn(N, H, dv, dk, generator=g)).cuda()
    do = torch.randn(B, T, H, dv, generator=g).to(dt).cuda()
    dS = torch.randn(N, H, dv, dk, generator=g).cuda()

    def grads(f):
        xs = [t.clone().requires_grad_() for t in (qkv, *gates, S0)]
        o, Sf = f(*xs)
        return (o, Sf) + torch.autograd.grad((o, Sf), xs, (do, dS))

    def separate(x, b, lam, la, s):
        q, k, v = x.split([dk, dk, dv], dim=-1)
        return layer.qdelta_chunk(layer.L2NormFunction.apply(q), layer.L2NormFunction.apply(k), v.contiguous(), b, lam,
                                  la, s, cu)

    fused = grads(lambda x, b, lam, la, s: layer.QKVChunkFunction.apply(x, b, lam, la, s, cu, dk, dv))
    apart = grads(separate)
    torch.cuda.synchronize()
    for i in (0, 1, 3, 4, 5, 6):
        assert torch.equal(fused[i], apart[i]), i
    tol = 2.0 ** -8 if dt == torch.bfloat16 else 1e-6
    assert normwise(fused[2].double().cpu().numpy(), apart[2].double().cpu().numpy()) <= tol
    if dt == torch.bfloat16:
        assert float((fused[2].double() - apart[2].double()).norm() / apart[2].double().norm()) <= 2.0 ** -12
    assert torch.equal(fused[2][..., 2 * dk:], apart[2][..., 2 * dk:])


@pytest.mark.parametrize("dt,use_decay,fixed_lambda", [(torch.bfloat16, True, None), (torch.float32, False, None),
                                                       (torch.float32, True, 0.5), (torch.bfloat16, False, 0.0)])
@pytest.mark.parametrize("B,T,H", [(1, 1, 1), (2, 65, 3), (3, 1001, 16)])
def test_gate_kernels_match_gates(dt, use_decay, fixed_lambda, B, T, H):
    """The gate kernels against gates() itself in fp64 on the same logits (a saturated one of each sign among them):
    values and logit gradients to the rounding of fp32 (bf16 gradients: 2^-8), the bias's gradient relative to the
    sum of its summands' magnitudes."""
    m = layer.QDeltaLayer(d_model=8, n_heads=H, head_dk=64, head_dv=64, use_decay=use_decay, fixed_lambda=fixed_lambda)
    g = torch.Generator().manual_seed(48)
    n = m.w_gates.out_features
    x = torch.randn(B, T, n, generator=g)
    x[0, 0, 0], x[-1, -1, -1] = 40.0, -40.0
    x = x.to(dt)
    bias = torch.tensor(-0.8, dtype=dt) if fixed_lambda is None else None
    dy = [torch.randn(B, T, H, generator=g) for _ in range(3)]

    xr = x.double().requires_grad_()
    br = None if bias is None else bias.double().expand(B, T, H).clone().requires_grad_()
    if br is not None:
        m.lambda_bias = torch.nn.Parameter(br.detach().clone())
    ref = m._split_gates(xr, torch.float64)
    xg = x.cuda().requires_grad_()
    bg = None if bias is None else bias.cuda().requires_grad_()
    got = layer.GatesFunction.apply(xg, bg, H, use_decay)
    live = [(a, b, d) for a, b, d in zip(got, ref, dy) if a is not None]
    torch.autograd.backward([a for a, _, _ in live], [d.cuda() for _, _, d in live])
    torch.autograd.backward([b for _, b, _ in live], [d.double() for _, _, d in live])
    torch.cuda.synchronize()
    for a, b, _ in live:
        assert torch.allclose(a.cpu().double(), b.detach(), rtol=1e-6, atol=1e-30)
    tol = dict(rtol=2.0 ** -8, atol=1e-30) if dt == torch.bfloat16 else dict(rtol=2e-6, atol=1e-7)
    assert torch.allclose(xg.grad.cpu().double(), xr.grad, **tol)
    if bias is not None:
        terms = m.lambda_bias.grad
        err = abs(float(bg.grad) - float(terms.sum())) / float(terms.abs().sum())
        assert err <= (2.0 ** -8 if dt == torch.bfloat16 else 1e-6)
