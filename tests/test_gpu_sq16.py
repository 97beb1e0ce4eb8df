"""The backward of the m = 16 fp32 transform on short batches, around its chunks of 64 rows and around the number of rows at which the
kernel with a workgroup per tile takes over."""
import numpy as np
import pytest

import oracle
import parity_util
from paper_2204_00595_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 15, 63, 64, 65, 128, 191, 192, 193])
def test_short_batch_backward(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    sh = synth.Shape("sq16_%d" % rows, "f32", rows, 16, 16, 16, 16, config=600 + rows)
    x, R, L, dy = synth.make_inputs(sh)
    args = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (dy, x, R, L)]
    guard = torch.full((rows + 1, 256), 7.0, device="cuda")
    dx, dR, dL = B.monarch_bwd(*args, dx=guard[:rows])
    for name, g, w in zip(("dx", "dR", "dL"), (dx, dR, dL), oracle.bwd(dy, x, R, L)):
        # fp32 sums of at most 192 products: 192 * 2^-24 of their size at the very most
        parity_util.check("%s.%s" % (sh.name, name), g.cpu().numpy(), w, 1e-5)
    assert bool((guard[rows] == 7.0).all())
    again = B.monarch_bwd(*args)
    for a, b in zip((dx, dR, dL), again):
        assert torch.equal(a, b)   # fixed summation order
