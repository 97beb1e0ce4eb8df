"""The projection at the edges of its 16-wide tiles, and on matrices whose squares leave the range of fp32."""
import numpy as np
import pytest

import oracle
from oracle import project
from paper_2204_00595_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1e-25, 1e25])
@pytest.mark.parametrize("m", [15, 17, 31, 32, 47, 48, 49])
def test_projection_at_tile_edges_and_scales(m, scale):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding
    A = synth.normal(7300 + m, (m * m, m * m))
    want = project.monarch_square(*project.project_square(A))
    L, R = binding.monarch_project(torch.from_numpy((A * np.float32(scale)).astype(np.float32)).cuda())
    got = project.monarch_square(L.cpu().numpy(), R.cpu().numpy()) / scale
    assert oracle.rel_fro(got, want) <= 1e-5


@pytest.mark.parametrize("seed", [0, 1])
@pytest.mark.parametrize("m", [12, 17, 33, 50, 64])
def test_every_slice_of_a_projection_is_as_exact_as_its_gap_allows(m, seed):
    """A perturbation of size eps * s1 of a slice moves its leading singular vectors by eps * s1 / (s1 - s2), so rounding in fp32
    leaves the leading rank-1 part eps * s1 * (1 + s1 / (s1 - s2)) off; the largest found over 54 matrices of these sizes is 1.01
    times that.  The bound holds slice by slice, so that the slices with a narrow gap (1e-4 at m = 64) cannot hide the others."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding
    n = m * m
    A = (synth.normal(9000 + 100 * m + seed, (n, n)) / m).astype(np.float32)
    L, R = (t.double().cpu() for t in binding.monarch_project(torch.from_numpy(A).cuda()))
    slices = torch.from_numpy(A).double().view(m, m, m, m).permute(1, 2, 0, 3).contiguous()   # [j][k][l][i]
    u, s, vt = torch.linalg.svd(slices)
    want = u[..., :, 0, None] * s[..., 0, None, None] * vt[..., 0, None, :]
    got = L.permute(0, 2, 1)[..., :, None] * R.permute(1, 0, 2)[..., None, :]
    err = (got - want).norm(dim=(-1, -2))
    bound = 4 * 2.0 ** -24 * s[..., 0] * (1 + s[..., 0] / (s[..., 0] - s[..., 1]))
    assert bool((err <= bound).all()), "slice %d: %.2f times the bound" % (int((err / bound).argmax()), float((err / bound).max()))
