"""Backward of the square matrix of 64 blocks of 64: rows at the edges of a 32-row step, of a pair of steps, of the bf16 partial
sums and of the number of batch chunks."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [1, 31, 33, 64, 97, 256, 257, 2049, 2113])
def test_backward_at_the_edges(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2204_00595_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(rows)
    x, dy, R, L = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
                   for shape in ((rows, 4096), (rows, 4096), (64, 64, 64), (64, 64, 64)))
    # whatever the kernels' buffers held before must not show in the rows past the last one
    B.monarch_bwd(torch.full_like(dy, float("nan")), torch.full_like(x, float("nan")), R, L)
    guard = torch.full((rows + 1, 4096), 7.0, device="cuda", dtype=torch.bfloat16)
    want = oracle.bwd(*(a.float().cpu().numpy().astype(np.float64) for a in (dy, x, R, L)))
    for flags in (0, B.MONARCH_FLAG_WGRAD_F32):
        got = B.monarch_bwd(dy, x, R, L, dx=guard[:rows], flags=flags)
        assert bool((guard[rows] == 7.0).all())
        for name, g, w in zip(("dx", "dR", "dL"), got, want):
            # two bf16 roundings of 2^-9 at most: the vector between the factors, and the result or the chunks' sums
            err = np.linalg.norm(g.float().cpu().numpy() - w) / np.linalg.norm(w)
            assert err <= 2.0 ** -8, (name, rows, flags, err)
        again = B.monarch_bwd(dy, x, R, L, flags=flags)
        assert all(torch.equal(g, a) for g, a in zip(got, again))


# The layer, which keeps the vector between the factors, against the calls that recompute it: the same bits, with a bias and without,
# and the bias gradient from the sums of the weight gradient's fragments against 64 bits (fp32 sums of 8 rows, then of a chunk's).
@pytest.mark.gpu
@pytest.mark.parametrize("bias", (False, True), ids=("no_bias", "bias"))
@pytest.mark.parametrize("rows", [1, 31, 64, 97, 257, 2113])
def test_layer_keeps_the_vector(rows, bias):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import autograd
    from paper_2204_00595_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(50 + rows)
    x, dy, R, L, b = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
                      for shape in ((rows, 4096), (rows, 4096), (64, 64, 64), (64, 64, 64), (4096,)))
    code = B.MONARCH_BF16
    assert B.lib().monarch_kept_bytes(rows, 4096, 64, 64, 64, code, 0) >= rows * 8192
    assert B.lib().monarch_kept_bytes(rows, 4096, 64, 64, 64, code, B.MONARCH_FLAG_GENERIC) == 0
    layer = autograd.MonarchLinear(4096, 4096, nblocks=64, bias=bias, q=64, device="cuda", dtype=torch.bfloat16)
    with torch.no_grad():
        layer.R.copy_(R)
        layer.L.copy_(L)
        if bias:
            layer.bias.copy_(b)
    xg = x.clone().requires_grad_(True)
    y = layer(xg)
    y.backward(dy)
    want = B.monarch_fwd_ws(x, R, L)
    if bias:
        want = (want.float() + b.float()).to(torch.bfloat16)
        assert torch.equal(B.monarch_fwd_bias(x, R, L, b), want)
    assert torch.equal(y, want)
    for got, ref in zip((xg.grad, layer.R.grad, layer.L.grad), B.monarch_bwd(dy, x, R, L)):
        assert torch.equal(got, ref)
    if not bias:
        return
    exact = dy.double().sum(0)
    size = dy.double().abs().sum(0)
    for got in (layer.bias.grad, B.monarch_bwd_bias(dy, x, R, L)[3]):
        assert bool(((got.double() - exact).abs() <= 2.0 ** -8 * exact.abs() + 1e-6 * size).all())
    got = B.monarch_bwd_bias(dy, x, R, L, flags=B.MONARCH_FLAG_WGRAD_F32)[3]
    assert bool(((got.double() - exact).abs() <= 1e-6 * size).all())


# ... whose backward's workspace has no place for a vector that it does not recompute: nothing behind what is asked for is written, the
# bits are those of a longer workspace, and the layer's backward takes no more memory than that and its gradients.
@pytest.mark.gpu
@pytest.mark.parametrize("rows", [33, 2113])
def test_backward_of_a_kept_vector_needs_no_place_for_it(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import autograd
    from paper_2204_00595_amd import binding as B
    lib, dims, vector = B.lib(), (rows, 4096, 64, 64, 64, B.MONARCH_BF16), rows * 8192
    need, whole = lib.monarch_bwd_kept_workspace_bytes(*dims, 0), lib.monarch_bwd_workspace_bytes(*dims, 0)
    assert need == whole - vector
    gen = torch.Generator(device="cuda").manual_seed(70 + rows)
    x, dy, R, L = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
                   for shape in ((rows, 4096), (rows, 4096), (64, 64, 64), (64, 64, 64)))
    st = int(torch.cuda.current_stream().cuda_stream)
    kept = torch.empty(lib.monarch_kept_bytes(*dims, 0), dtype=torch.uint8, device="cuda")
    y = torch.empty_like(dy)
    assert lib.monarch_fwd_keep(*(t.data_ptr() for t in (x, R, L)), None, y.data_ptr(), kept.data_ptr(), kept.numel(), *dims, st, 0) == 0
    results = []
    for room in (need, whole):
        ws = torch.full((room + 65536,), 0xA5, dtype=torch.uint8, device="cuda")
        g = [torch.empty_like(t) for t in (x, R, L)] + [torch.empty(4096, dtype=torch.bfloat16, device="cuda")]
        assert lib.monarch_bwd_kept(*(t.data_ptr() for t in (dy, x, kept)), kept.numel(), R.data_ptr(), L.data_ptr(),
                                    *(t.data_ptr() for t in g), *dims, st, ws.data_ptr(), room, 0) == 0
        assert bool((ws[room:] == 0xA5).all())
        results.append(g)
    assert all(torch.equal(a, b) for a, b in zip(*results))
    layer = autograd.MonarchLinear(4096, 4096, nblocks=64, bias=True, q=64, device="cuda", dtype=torch.bfloat16)
    y = layer(x.clone().requires_grad_(True))
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    y.backward(dy)
    gradients = vector + 2 * 2 * 64 ** 3 + 2 * 4096
    assert torch.cuda.max_memory_allocated() - before <= need + gradients + 4 * 512   # a piece is a multiple of 512 bytes
