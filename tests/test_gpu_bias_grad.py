"""Bias gradients of the bf16 four-block layers: column sums of dy taken from the fragments of the weight-gradient products
(every tile shape they have, rows at the edges of a 32-row step, of a chunk and of the choice of the kernels)."""
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
