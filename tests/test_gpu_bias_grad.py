"""Bias and weight gradients of the bf16 four-block layers: column sums of dy taken from the fragments of the weight-gradient
products, and those products (every tile shape they have, rows at the edges of a 32-row step, of a chunk and of the choice of the
kernels)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

SHAPES = [(64, 64, 32), (64, 64, 64), (64, 64, 128), (128, 128, 64), (128, 128, 384), (192, 192, 192), (256, 256, 1024)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [1, 31, 33, 64, 65, 257, 1000, 2561, 4100])
def test_bias_gradient_is_the_exact_sum(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    for p, q, s in SHAPES:
        gen = torch.Generator(device="cuda").manual_seed(rows + s)
        # whole numbers up to 100: exact in bf16, and their sums over 4100 rows in 32 bits, so no order of adding shows
        dy = torch.randint(-100, 101, (rows, 4 * s), generator=gen, device="cuda").to(torch.bfloat16)
        x = torch.randn((rows, 4 * p), generator=gen, device="cuda").to(torch.bfloat16)
        R = torch.randn((4, q, p), generator=gen, device="cuda").to(torch.bfloat16)
        L = torch.randn((4, s, q), generator=gen, device="cuda").to(torch.bfloat16)
        got = B.monarch_bwd_bias(dy, x, R, L, flags=B.MONARCH_FLAG_WGRAD_F32)[3]
        want = dy.double().sum(0)
        assert got.dtype == torch.float32 and torch.equal(got.double(), want), (rows, p, q, s)
        rounded = B.monarch_bwd_bias(dy, x, R, L)[3]
        assert torch.equal(rounded, want.to(torch.bfloat16)), (rows, p, q, s)


@pytest.mark.gpu
@pytest.mark.parametrize("fp32", [False, True], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows", [1, 33, 257, 2561, 4100])
def test_weight_gradients_at_the_edges(rows, fp32):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2204_00595_amd import binding as B
    for p, q, s in SHAPES[:-1] + [(64, 128, 64), (96, 96, 96)]:
        gen = torch.Generator(device="cuda").manual_seed(rows * 1000 + s)
        x, dy, R, L = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
                       for shape in ((rows, 4 * p), (rows, 4 * s), (4, q, p), (4, s, q)))
        # whatever the buffers of the products held before must not show in the rows past the last one
        B.monarch_bwd_bias(torch.full_like(dy, float("nan")), torch.full_like(x, float("nan")), R, L)
        got = B.monarch_bwd_bias(dy, x, R, L, flags=B.MONARCH_FLAG_WGRAD_F32 if fp32 else 0)[1:3]
        want = oracle.bwd(*(a.float().cpu().numpy().astype(np.float64) for a in (dy, x, R, L)))[1:3]
        for name, g, w in zip(("dR", "dL"), got, want):
            # two bf16 roundings of 2^-9 at most: the vector between the factors, and the result or the chunks' sums
            err = np.linalg.norm(g.float().cpu().numpy() - w) / np.linalg.norm(w)
            assert err <= 2.0 ** -8, (name, rows, p, q, s, err)
