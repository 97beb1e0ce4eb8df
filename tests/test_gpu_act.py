"""The derivative of the feed-forward block's nonlinearity, bit for bit: dx is multiplied by s + v (s (1 - s)) d, each product and
difference rounded on its own (d and the last sum are one operation each).  In another order bf16 gradients behind it round differently."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

F = np.float32


def _fma(a, b, c):
    return (a.astype(np.float64) * b + c).astype(F)  # the product is exact in 64 bits


def _gates(v, y):
    """(5, n) fp32 values s next to y / v, and which of them give y = v s: one of them is the kernel's."""
    near = (y.astype(np.float64) / v).astype(F)
    s = np.stack([(near.view(np.int32) + d).view(F) for d in range(-2, 3)])
    return s, v * s == y


def _gradients(v, s, fused=False):
    d = _fma(np.full_like(v, 0.21406445), v * v, np.full_like(v, 1.5957692))
    return _fma(v * (_fma(-s, s, s) if fused else s * (F(1) - s)), np.broadcast_to(d, s.shape), s)


V = np.arange(-128, 128).astype(F) / 16
V[128] = 2.0 ** -10   # where y = v s says nothing of s


def _disagree(v, y, grad):
    s, is_gate = _gates(v, y)
    assert is_gate.any(0).all()
    return int((~((_gradients(v, s) == grad) & is_gate).any(0)).sum())


def test_the_check_sees_another_order():
    s = (1 / (1 + np.exp(-V.astype(np.float64) * (1.5957691 + 0.0713548 * V.astype(np.float64) ** 2)))).astype(F)
    assert _disagree(V, V * s, _gradients(V, s)) == 0
    assert _disagree(V, V * s, _gradients(V, s, fused=True)) >= 8


@pytest.mark.gpu
def test_derivative_is_rounded_in_its_order():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    m, n = 16, 256
    v = torch.from_numpy(V).cuda()
    zero, one = torch.zeros((m, m, m), device="cuda"), torch.eye(m, device="cuda").expand(m, m, m).contiguous()
    ones = torch.ones((3, n), device="cuda")
    pre, y = B.monarch_fwd_bias_gelu(ones, zero, zero, v)   # gelu(0 + v)
    assert torch.equal(pre, v.expand(3, n))
    x = torch.zeros((3, n), device="cuda")
    dx = B.monarch_bwd_bias_gelu_in(ones, x, pre, one, one)[0]   # identity blocks: 1 in every place before the nonlinearity's factor
    for row in range(3):
        wrong = _disagree(V, y[row].cpu().numpy(), dx[row].cpu().numpy())
        assert wrong == 0, wrong
