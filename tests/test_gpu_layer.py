"""MonarchLinear and the binding's checks around it: what a call without gradients keeps."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding
    return binding


def layer_of(p, q, s, k=4, dtype=torch.bfloat16, bias=True):
    from paper_2204_00595_amd import autograd
    torch.manual_seed(5)
    layer = autograd.MonarchLinear(k * p, k * s, nblocks=k, q=q, bias=bias, device="cuda", dtype=dtype)
    if bias:
        torch.nn.init.normal_(layer.bias)
    return layer


# a shape with a packed forward, and one of the shape-generic contractions; both keep the vector in a training step
@pytest.mark.parametrize("bias", [True, False], ids=["bias", "no_bias"])
@pytest.mark.parametrize("dims", [(192, 192, 192), (49, 33, 64)], ids=str)
def test_layer_without_gradients_keeps_nothing(B, dims, bias):
    p, q, s = dims
    rows = 3000
    layer = layer_of(p, q, s, bias=bias)
    x = torch.randn((rows, 4 * p), device="cuda").bfloat16()
    saved = B.monarch_saved_bytes(rows, 4 * p, 4, q, s, B.MONARCH_BF16)
    assert saved > 0
    if bias:
        want = B.monarch_fwd_bias(x, layer.R.detach(), layer.L.detach(), layer.bias.detach())
    else:
        want = B.monarch_fwd_ws(x, layer.R.detach(), layer.L.detach())

    def peak():
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        y = layer(x)
        torch.cuda.synchronize()
        return y, torch.cuda.max_memory_allocated() - before

    y, most = peak()   # a training step's forward: y and the vector
    assert y.requires_grad and most >= y.numel() * 2 + saved
    room = y.numel() * 2 + B.monarch_fwd_workspace_bytes(rows, 4 * p, 4, q, s, B.MONARCH_BF16) + 2048  # the allocator rounds up to 512
    del y
    for guard in (torch.no_grad, torch.inference_mode):
        with guard():
            y, most = peak()
        assert torch.equal(y, want) and most <= room
        del y
    for par in layer.parameters():
        par.requires_grad_(False)
    y, most = peak()   # a frozen layer
    assert not y.requires_grad and torch.equal(y, want) and most <= room


# what is not (..., width) is refused, however it lies in memory
@pytest.mark.parametrize("shape", [(10, 384), (384, 10), (10, 2, 384), (5, 2, 768, 1), (10, 769), (10, 1536)], ids=str)
def test_layer_refuses_inputs_of_another_width(B, shape):
    layer = layer_of(192, 192, 192)
    x = torch.randn(shape, device="cuda").bfloat16()
    for t in (x, x.transpose(0, 1).contiguous().transpose(0, 1), x.requires_grad_(True)):
        assert tuple(t.shape) == shape
        with pytest.raises((RuntimeError, ValueError)):
            layer(t)


def test_layer_takes_any_leading_dimensions_and_strides(B):
    layer = layer_of(192, 192, 576)
    x = torch.randn((6, 768), device="cuda").bfloat16()
    want = layer(x)
    views = [(x[:1].reshape(768), want[:1].reshape(2304)), (x.reshape(3, 2, 768), want.reshape(3, 2, 2304)),
             (x.t().contiguous().t(), want), (x.reshape(2, 3, 768).transpose(0, 1), want.reshape(2, 3, 2304).transpose(0, 1)),
             (x[:0], want[:0]), (x[:0].reshape(0, 5, 768), want[:0].reshape(0, 5, 2304))]
    for view, y in views:
        view = view.detach().requires_grad_(True)
        out = layer(view)
        assert out.shape == y.shape and torch.equal(out, y)
        out.backward(torch.ones_like(out))
        assert view.grad.shape == view.shape


# dims (p, q, s), k, dtype: shapes whose calls never find packed weights take the flag without a workspace and ignore it
@pytest.mark.parametrize("case", [((49, 33, 64), 4, "f32"), ((49, 33, 64), 4, "bf16"), ((96, 96, 384), 4, "bf16"), ((7, 5, 9), 3, "f32"),
                                  ((16, 16, 16), 16, "f32")], ids=str)
def test_packed_flag_without_a_workspace_is_ignored_where_it_means_nothing(B, case):
    (p, q, s), k, dtype = case
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    layer = layer_of(p, q, s, k=k, dtype=dt)
    x = torch.randn((33, k * p), device="cuda").to(dt)
    R, L, bias = (t.detach() for t in (layer.R, layer.L, layer.bias))
    assert torch.equal(B.monarch_fwd_ws(x, R, L, flags=B.MONARCH_FLAG_WS_PACKED), B.monarch_fwd_ws(x, R, L))
    assert torch.equal(B.monarch_fwd_bias(x, R, L, bias, flags=B.MONARCH_FLAG_WS_PACKED), B.monarch_fwd_bias(x, R, L, bias))
    with pytest.raises(B.MonarchError):
        B.monarch_fwd_save(x, R, L, flags=B.MONARCH_FLAG_WS_PACKED)


@pytest.mark.parametrize("case", [((192, 192, 192), 4, "bf16"), ((64, 64, 64), 64, "bf16"), ((32, 32, 32), 3, "f32")], ids=str)
def test_packed_flag_without_a_workspace_is_refused_where_one_is_needed(B, case):
    (p, q, s), k, dtype = case
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    layer = layer_of(p, q, s, k=k, dtype=dt)
    x = torch.randn((33, k * p), device="cuda").to(dt)
    with pytest.raises(ValueError):
        B.monarch_fwd_ws(x, layer.R.detach(), layer.L.detach(), flags=B.MONARCH_FLAG_WS_PACKED)


@pytest.mark.parametrize("bias", [True, False], ids=["bias", "no_bias"])
def test_traced_layer_computes(B, bias):
    """torch.jit.trace records the multiply itself: the traced layer follows its input, its weights and their gradients."""
    layer = layer_of(192, 192, 576, bias=bias)
    x, other, dy = (torch.randn(shape, device="cuda").bfloat16() for shape in ((2, 5, 768), (2, 5, 768), (2, 5, 2304)))
    traced = torch.jit.trace(layer, x)
    with torch.no_grad():
        layer.R.mul_(0.5)
        tn = torch.jit.trace(layer, x)
        assert torch.equal(tn(other), layer(other))
    a, b = (other.clone().requires_grad_(True) for _ in range(2))
    ya, yb = traced(a), layer(b)
    assert torch.equal(ya, yb)
    pars = list(layer.parameters())
    for g, w in zip(torch.autograd.grad(ya, [a] + pars, dy), torch.autograd.grad(yb, [b] + pars, dy)):
        assert torch.equal(g, w)
    with pytest.raises((RuntimeError, ValueError)):
        torch.jit.trace(layer, torch.randn((20, 384), device="cuda").bfloat16())
