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
