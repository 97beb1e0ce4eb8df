"""The forward of the four-block layers on short batches (one launch per factor, with or without a fused kernel) at the edges of its tiles: row counts around 32
and around the numbers at which the tile and the dealing of row tiles change, every width, with and without packed weights."""
import numpy as np
import pytest

import oracle
import parity_util
from oracle import activation
from paper_2204_00595_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# B, p, q, s
CASES = [(1, 64, 64, 64), (31, 64, 64, 128), (33, 128, 64, 64), (97, 128, 128, 512), (2817, 128, 128, 128), (513, 512, 128, 128), (65, 192, 192, 576),
         (250, 192, 192, 768), (700, 768, 192, 192), (45, 96, 96, 384), (1300, 384, 96, 96), (129, 48, 32, 96), (1, 256, 256, 1024), (545, 256, 256, 768), (290, 1024, 256, 256)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_short_batch_forward(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, p, q, s = case
    sh = synth.Shape("split_%s" % (case,), "bf16", rows, 4, p, q, s, config=500 + parity_util.stable_seed(str(case)))
    x, R, L, _ = synth.make_inputs(sh)
    bias = synth.quantize(synth.normal(78, (sh.n_out,)), "bf16")
    xd, Rd, Ld, bd = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L, bias))
    want = oracle.fwd(x, R, L)

    def check(name, got, want):
        parity_util.check("%s.%s" % (sh.name, name), got.float().cpu().numpy(), want, 2e-2)

    need = B.monarch_fwd_workspace_bytes(rows, sh.n_in, 4, q, s, 1)
    packed = B.monarch_fwd_workspace_bytes(0, sh.n_in, 4, q, s, 1)
    assert need > packed
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    y = B.monarch_fwd_ws(xd, Rd, Ld, workspace=ws)
    check("y", y, want)
    again = B.monarch_fwd_ws(xd, Rd, Ld, workspace=ws, flags=B.MONARCH_FLAG_WS_PACKED)
    assert torch.equal(y, again)
    check("y_long", B.monarch_fwd_ws(xd, Rd, Ld, workspace=ws[:packed], flags=B.MONARCH_FLAG_WS_PACKED), want)  # no room behind the packed weights
    check("y_bias", B.monarch_fwd_bias(xd, Rd, Ld, bd, workspace=ws), oracle.fwd_bias(x, R, L, bias))
    pre, act = B.monarch_fwd_bias_gelu(xd, Rd, Ld, bd, workspace=ws)
    check("pre", pre, oracle.fwd_bias(x, R, L, bias))
    check("gelu", act, activation.gelu(oracle.fwd_bias(x, R, L, bias)))
    _, act2 = B.monarch_fwd_bias_gelu(xd, Rd, Ld, bd, want_pre=False, workspace=ws)
    assert torch.equal(act, act2)


# the last rows of narrow, wide and square layers, and the first past them; batches in slices, with and without packed weights, with and
# without a fused kernel (four slices and an odd last one, two; one row more than seven can hold; two)
@pytest.mark.parametrize("case", [(4352, 128, 64, 64), (4353, 128, 64, 64), (2048, 192, 192, 768), (2049, 192, 192, 576), (3072, 64, 64, 128),
                                  (3073, 192, 192, 192), (2848, 1024, 256, 256), (4352, 1024, 256, 256), (8190, 384, 96, 96), (1001, 256, 224, 4096),
                                  (2047, 128, 160, 5120), (2241, 256, 224, 4096), (6235, 160, 160, 160)], ids=str)
def test_forward_at_the_limits_of_the_short_batch_kernels(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, p, q, s = case
    sh = synth.Shape("lfsplit_%s" % (case,), "bf16", rows, 4, p, q, s, config=550 + parity_util.stable_seed(str(case)))
    x, R, L, _ = synth.make_inputs(sh)
    xd, Rd, Ld = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L))
    y, ys = B.monarch_fwd_ws(xd, Rd, Ld), torch.empty((rows, sh.n_out), dtype=torch.bfloat16, device="cuda")
    B.monarch_fwd_static(xd, Rd, Ld, ys)
    assert torch.equal(y, ys)
    ws = torch.full((B.monarch_fwd_workspace_bytes(rows, sh.n_in, 4, q, s, 1),), 0xFF, dtype=torch.uint8, device="cuda")
    pre, act = B.monarch_fwd_bias_gelu(xd, Rd, Ld, None, workspace=ws)
    assert torch.equal(pre, y)
    pre2, act2 = B.monarch_fwd_bias_gelu(xd, Rd, Ld, None, workspace=ws, flags=B.MONARCH_FLAG_WS_PACKED)
    assert torch.equal(pre2, y) and torch.equal(act, act2)
    parity_util.check(sh.name, y.float().cpu().numpy(), oracle.fwd(x, R, L), 2e-2)


# B, p, q, s: short-batch backward at the edges of its tiles, of its step counts (s = 1024 .. 32) and of its row limits
BWD = [(1, 96, 96, 384), (33, 384, 96, 96), (4096, 32, 32, 64), (63, 64, 64, 64), (2559, 128, 128, 128), (97, 512, 128, 128), (545, 192, 192, 576),
       (65, 192, 192, 768), (31, 768, 192, 192), (130, 256, 256, 1024), (290, 1024, 256, 256)]


@pytest.mark.parametrize("case", BWD, ids=str)
def test_short_batch_backward(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, p, q, s = case
    sh = synth.Shape("bsplit_%s" % (case,), "bf16", rows, 4, p, q, s, config=600 + parity_util.stable_seed(str(case)))
    x, R, L, dy = synth.make_inputs(sh)
    pre = synth.quantize(synth.normal(79, (rows, sh.n_in)), "bf16")
    xd, Rd, Ld, dyd, pred = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L, dy, pre))
    want = oracle.bwd_bias(dy, x, R, L)

    def check(name, got, want):
        parity_util.check("%s.%s" % (sh.name, name), got.float().cpu().numpy(), want, 2e-2)

    need = B.monarch_bwd_workspace_bytes(rows, sh.n_in, 4, q, s, 1)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    got = B.monarch_bwd_bias(dyd, xd, Rd, Ld, workspace=ws)
    for name, g, w in zip(("dx", "dR", "dL", "dbias"), got, want):
        check(name, g, w)
    again = B.monarch_bwd_bias(dyd, xd, Rd, Ld, workspace=ws)
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    for name, g, w in zip(("dx32", "dR32", "dL32"), B.monarch_bwd(dyd, xd, Rd, Ld, workspace=ws, flags=B.MONARCH_FLAG_WGRAD_F32), want):
        check(name, g, w)
    act = B.monarch_bwd_bias_gelu_in(dyd, xd, pred, Rd, Ld, workspace=ws)
    check("dx_pre", act[0], want[0] * activation.gelu_grad(pre))
    assert all(torch.equal(a, b) for a, b in zip(got[1:], act[1:]))
    _, saved = B.monarch_fwd_save(xd, Rd, Ld)
    for name, g, w in zip(("dx_s", "dR_s", "dL_s"), B.monarch_bwd_saved(dyd, xd, saved, Rd, Ld), want):
        check(name, g, w)


# The last rows, and the first past them, of what the kernels of short batches take (square layers, others, without a fused kernel, with
# the nonlinearity's factor, which they take further) and of the wide kernel in tiles of 32 rows; each in the room that is asked for,
# and in that of a slightly longer batch.
LIMITS = [(1536, 192, 192, 192), (1537, 128, 128, 128), (1800, 256, 256, 1024), (1801, 256, 256, 768), (1805, 192, 192, 576), (16384, 32, 32, 64),
          (16385, 64, 32, 32), (2200, 768, 192, 192), (2201, 512, 128, 128), (2203, 1024, 256, 256), (2560, 128, 64, 64), (2561, 64, 64, 128),
          (4096, 192, 192, 768), (4097, 192, 192, 192), (47, 64, 64, 64), (33, 64, 64, 64), (3009, 256, 256, 256),
          (4096, 64, 160, 32), (4097, 32, 160, 64), (6144, 96, 96, 192), (6145, 160, 96, 32), (16384, 96, 96, 288), (16385, 288, 96, 96)]


@pytest.mark.parametrize("case", LIMITS, ids=str)
def test_backward_at_the_limits_of_the_short_batch_kernels(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, p, q, s = case
    sh = synth.Shape("lsplit_%s" % (case,), "bf16", rows, 4, p, q, s, config=650 + parity_util.stable_seed(str(case)))
    x, R, L, dy = synth.make_inputs(sh)
    pre = synth.quantize(synth.normal(79, (rows, sh.n_in)), "bf16")
    xd, Rd, Ld, dyd, pred = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L, dy, pre))
    want = oracle.bwd_bias(dy, x, R, L)
    act = (want[0] * activation.gelu_grad(pre),) + tuple(want[1:])
    need = B.monarch_bwd_workspace_bytes(rows, sh.n_in, 4, q, s, 1)
    longer = B.monarch_bwd_workspace_bytes(rows + 1, sh.n_in, 4, q, s, 1)
    for room in (need, longer):
        ws = torch.full((room + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        for got, wanted in ((B.monarch_bwd_bias(dyd, xd, Rd, Ld, workspace=ws[:room]), want),
                            (B.monarch_bwd_bias_gelu_in(dyd, xd, pred, Rd, Ld, workspace=ws[:room]), act)):
            for name, g, w in zip(("dx", "dR", "dL", "dbias"), got, wanted):
                parity_util.check("%s.%s" % (sh.name, name), g.float().cpu().numpy(), w, 2e-2)
            assert bool((ws[room:] == 0xFF).all())


# p, q, s without a fused kernel: what an earlier call left in the workspace depends on its batch and on the room it had
@pytest.mark.parametrize("dims", [(96, 96, 384), (128, 128, 384), (384, 96, 96)], ids=str)
def test_packed_flag_after_a_call_that_packed_nothing(dims):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    p, q, s = dims
    sh = synth.Shape("flag_%s" % (dims,), "bf16", 40, 4, p, q, s, config=800 + parity_util.stable_seed(str(dims)))
    x, R, L, _ = synth.make_inputs(sh)
    xd, Rd, Ld = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L))
    want = oracle.fwd(x, R, L)
    need = B.monarch_fwd_workspace_bytes(40, sh.n_in, 4, q, s, 1)
    long_x = torch.zeros((8193, sh.n_in), dtype=torch.bfloat16, device="cuda")
    for first in (lambda ws: B.monarch_fwd_ws(long_x, Rd, Ld, workspace=ws), lambda ws: B.monarch_fwd_ws(xd, Rd, Ld, workspace=ws[:256])):
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN in bf16
        first(ws)
        y = B.monarch_fwd_ws(xd, Rd, Ld, workspace=ws, flags=B.MONARCH_FLAG_WS_PACKED)
        parity_util.check(sh.name, y.float().cpu().numpy(), want, 2e-2)


# 8 and 3072 rows: the first and the last that the kernels of short batches take; 3073 and m = 64: the fused kernels
@pytest.mark.parametrize("dims", [(8, 4, 256, 256, 1024), (3072, 4, 64, 64, 64), (3073, 4, 64, 64, 64), (70, 64, 64, 64, 64)], ids=str)
def test_packed_weights_are_only_read(dims):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, k, p, q, s = dims
    sh = synth.Shape("shared_%s" % (dims,), "bf16", rows, k, p, q, s, config=820 + parity_util.stable_seed(str(dims)))
    x, R, L, _ = synth.make_inputs(sh)
    bias = synth.quantize(synth.normal(81, (sh.n_out,)), "bf16")
    xd, Rd, Ld, bd = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L, bias))
    want = oracle.fwd_bias(x, R, L, bias)
    ws = torch.zeros(B.monarch_fwd_workspace_bytes(rows, sh.n_in, k, q, s, 1), dtype=torch.uint8, device="cuda")
    first = B.monarch_fwd_ws(xd, Rd, Ld, workspace=ws)
    ws[2 * (R.size + L.size):] = 0x5A   # what lies behind the packed weights is not the packed calls' either
    kept = ws.clone()
    nan = torch.full_like(Rd, float("nan")), torch.full_like(Ld, float("nan"))

    def check(name, got, want):
        parity_util.check("%s.%s" % (sh.name, name), got.float().cpu().numpy(), want, 2e-2)
        assert torch.equal(ws, kept), name

    y = B.monarch_fwd_ws(xd, *nan, workspace=ws, flags=B.MONARCH_FLAG_WS_PACKED)
    check("y", y, oracle.fwd(x, R, L))
    assert torch.equal(y, first)
    check("bias", B.monarch_fwd_bias(xd, *nan, bd, workspace=ws, flags=B.MONARCH_FLAG_WS_PACKED), want)
    pre, act = B.monarch_fwd_bias_gelu(xd, *nan, bd, workspace=ws, flags=B.MONARCH_FLAG_WS_PACKED)
    check("pre", pre, want)
    check("gelu", act, activation.gelu(want))
    # through the C ABI, where nothing is allocated: the fused kernel
    y.fill_(float("nan"))
    st = int(torch.cuda.current_stream().cuda_stream)
    rc = B.lib().monarch_fwd_ws(xd.data_ptr(), nan[0].data_ptr(), nan[1].data_ptr(), y.data_ptr(), rows, sh.n_in, k, q, s, 1, st,
                                ws.data_ptr(), ws.numel(), B.MONARCH_FLAG_WS_PACKED)
    assert rc == B.MONARCH_OK
    check("y_abi", y, oracle.fwd(x, R, L))


# Up to 256 rows the chunks of the batch are summed in fp32: bf16 gradients are the fp32 ones, rounded once.
@pytest.mark.parametrize("case", [(64, 64, 64, 64), (65, 192, 192, 768), (256, 256, 256, 1024), (256, 96, 96, 384), (200, 512, 128, 128)], ids=str)
def test_short_batch_gradients_are_rounded_once(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, p, q, s = case
    sh = synth.Shape("once_%s" % (case,), "bf16", rows, 4, p, q, s, config=840 + parity_util.stable_seed(str(case)))
    x, R, L, dy = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in synth.make_inputs(sh))
    narrow, wide = B.monarch_bwd(dy, x, R, L), B.monarch_bwd(dy, x, R, L, flags=B.MONARCH_FLAG_WGRAD_F32)
    for name, a, b in zip(("dx", "dR", "dL"), narrow, wide):
        assert torch.equal(a, b.to(torch.bfloat16)), name


def test_calls_on_two_streams_share_packed_weights():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    sh = synth.Shape("streams", "bf16", 3000, 4, 256, 256, 1024, config=860)
    x, R, L, _ = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in synth.make_inputs(sh))
    ws = torch.empty(B.monarch_fwd_workspace_bytes(0, sh.n_in, 4, 256, 1024, 1), dtype=torch.uint8, device="cuda")
    B.monarch_fwd_ws(x[:8], R, L, workspace=ws)
    parts = [x[:8], x[8:520], x[520:]]   # of several batch sizes
    want = [B.monarch_fwd_ws(p, R, L) for p in parts]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = []
    for i in range(24):
        with torch.cuda.stream(streams[i % 2]):
            got.append(B.monarch_fwd_ws(parts[i % 3], R, L, workspace=ws, flags=B.MONARCH_FLAG_WS_PACKED))
    torch.cuda.synchronize()
    for i, y in enumerate(got):
        assert torch.equal(y, want[i % 3]), i


# the vector between the factors is kept in tiles of 32 rows, the last one no longer than it is: nothing past what the queries name
@pytest.mark.parametrize("case", [(1, 64, 64, 64), (33, 128, 64, 64), (545, 256, 256, 768), (2817, 128, 128, 128), (57, 128, 160, 6368), (58, 128, 160, 6368)], ids=str)
def test_tiles_stay_inside_the_workspace(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, p, q, s = case
    sh = synth.Shape("guard_%s" % (case,), "bf16", rows, 4, p, q, s, config=560 + parity_util.stable_seed(str(case)))
    x, R, L, _ = synth.make_inputs(sh)
    xd, Rd, Ld = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L))
    need = B.monarch_fwd_workspace_bytes(rows, sh.n_in, 4, q, s, 1)
    ws = torch.full((need + 65536,), 0xA5, dtype=torch.uint8, device="cuda")
    y = B.monarch_fwd_ws(xd, Rd, Ld, workspace=ws[:need])
    parity_util.check(sh.name, y.float().cpu().numpy(), oracle.fwd(x, R, L), 2e-2)
    assert bool((ws[need:] == 0xA5).all())


# The backward on either side of its row limits: short-batch kernels up to them (2048, 2560 rows; none for blocks of 64), and the
# recomputed vector from a product of its own beyond 8192 rows.
LINES = [(256, 256, 1024, 2048), (192, 192, 192, 2560), (128, 128, 512, 2560), (512, 128, 128, 2048), (1024, 256, 256, 2048), (64, 64, 64, 40),
         (1024, 256, 256, 8192), (768, 192, 192, 8192)]


@pytest.mark.parametrize("past", [0, 1])
@pytest.mark.parametrize("case", LINES, ids=str)
def test_backward_at_its_row_limits(case, past):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    p, q, s, rows = case
    rows += past
    gen = torch.Generator(device="cuda").manual_seed(rows + p)
    x, R, L, dy = (torch.randn(shp, generator=gen, device="cuda").mul_(std).to(torch.bfloat16) for shp, std in (
        ((rows, 4 * p), 1.0), ((4, q, p), p ** -0.5), ((4, s, q), q ** -0.5), ((rows, 4 * s), 1.0)))
    dx, dR, dL, db = B.monarch_bwd_bias(dy, x, R, L)
    xd, Rd, Ld, dyd = (t.double() for t in (x, R, L, dy))
    # y[b][l*4 + c] = sum_r L[c][l][r] U[b][c][r], and U[b][c][r] is Y1 at the flat position c*q + r of (j, kk)
    Y1 = torch.stack([xd[:, kk * p:(kk + 1) * p] @ Rd[kk].T for kk in range(4)], 2).reshape(rows, 4, q)
    dW = dyd.reshape(rows, s, 4)
    dU = torch.stack([dW[:, :, c] @ Ld[c] for c in range(4)], 1)
    dY1 = dU.reshape(rows, q, 4)
    want = (torch.cat([dY1[:, :, kk] @ Rd[kk] for kk in range(4)], 1),
            torch.stack([dY1[:, :, kk].T @ xd[:, kk * p:(kk + 1) * p] for kk in range(4)]),
            torch.stack([dW[:, :, c].T @ Y1[:, c] for c in range(4)]), dyd.sum(0))
    for name, g, w in zip(("dx", "dR", "dL", "dbias"), (dx, dR, dL, db), want):
        # bf16 roundings of 2^-9 / sqrt(3) root mean square each: the vector, a partial sum, the result; a third more for the largest
        err = float(torch.linalg.norm(g.double() - w) / torch.linalg.norm(w))
        assert err <= 4e-3, (name, err)
    rel = torch.linalg.norm(dx.double() - want[0], dim=1) / torch.linalg.norm(want[0], dim=1)
    assert float(rel.max()) <= 6e-3   # no row: twice the root mean square


# A few rows on packed weights: both factors in one launch.  Every quarter of R against its tiles (q = 96: 24 rows, 192: 48), a last
# pair of column tiles with one of them, rows at the edges of a tile and past the second one; the bits of the two launches that the same
# call makes where it packs, with bias and nonlinearity too.
@pytest.mark.parametrize("rows", (1, 7, 32, 33, 64, 65))
@pytest.mark.parametrize("dims", [(256, 256, 1024), (192, 192, 768), (192, 192, 576), (128, 128, 512), (64, 64, 64), (128, 64, 64), (64, 128, 128)], ids=str)
def test_few_rows_in_one_launch(dims, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    p, q, s = dims
    sh = synth.Shape("once_%s" % (dims,), "bf16", rows, 4, p, q, s, config=990 + rows)
    x, R, L, _ = synth.make_inputs(sh)
    bias = synth.quantize(synth.normal(78, (sh.n_out,)), "bf16")
    xd, Rd, Ld, bd = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L, bias))
    ws = torch.empty(B.monarch_fwd_workspace_bytes(rows, sh.n_in, 4, q, s, 1), dtype=torch.uint8, device="cuda")
    guard = torch.full((rows + 1, sh.n_out), 7.0, device="cuda", dtype=torch.bfloat16)
    want = (B.monarch_fwd_ws(xd, Rd, Ld, workspace=ws), B.monarch_fwd_bias(xd, Rd, Ld, bd, workspace=ws), *B.monarch_fwd_bias_gelu(xd, Rd, Ld, bd, workspace=ws))
    flag = B.MONARCH_FLAG_WS_PACKED
    got = (B.monarch_fwd_ws(xd, Rd, Ld, y=guard[:rows], workspace=ws, flags=flag), B.monarch_fwd_bias(xd, Rd, Ld, bd, workspace=ws, flags=flag),
           *B.monarch_fwd_bias_gelu(xd, Rd, Ld, bd, workspace=ws, flags=flag))
    assert bool((guard[rows] == 7.0).all())
    for name, g, w in zip(("y", "bias", "pre", "gelu"), got, want):
        assert torch.equal(g, w), name
    parity_util.check("once_%s.y" % (dims,), got[0].float().cpu().numpy(), oracle.fwd(x, R, L), 2e-2)


# The same where no call leaves packed weights: R and L as they are, in one launch of up to 64 rows, against the rows of a 65-row batch,
# which takes two launches: quarters of R inside a tile and across two, fewer K-steps than quarters of p, the longest p
# and one past it, blocks of L that end a pair of column tiles.
@pytest.mark.parametrize("dims", [(96, 96, 384), (256, 96, 96), (96, 96, 96), (16, 32, 32), (240, 128, 160), (144, 64, 96), (384, 96, 96)], ids=str)
def test_few_rows_in_one_launch_on_weights_as_they_are(dims):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    p, q, s = dims
    sh = synth.Shape("once_direct_%s" % (dims,), "bf16", 65, 4, p, q, s, config=996)
    x, R, L, _ = synth.make_inputs(sh)
    bias = synth.quantize(synth.normal(79, (sh.n_out,)), "bf16")
    xd, Rd, Ld, bd = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L, bias))
    ws = torch.empty(B.monarch_fwd_workspace_bytes(65, sh.n_in, 4, q, s, 1), dtype=torch.uint8, device="cuda")

    def run(n, y=None):
        return (B.monarch_fwd_ws(xd[:n], Rd, Ld, y=y, workspace=ws), B.monarch_fwd_bias(xd[:n], Rd, Ld, bd, workspace=ws),
                *B.monarch_fwd_bias_gelu(xd[:n], Rd, Ld, bd, workspace=ws))

    want = run(65)
    parity_util.check("once_direct_%s.y" % (dims,), want[0].float().cpu().numpy(), oracle.fwd(x, R, L), 2e-2)
    for rows in (1, 7, 32, 33, 64):
        guard = torch.full((rows + 1, sh.n_out), 7.0, device="cuda", dtype=torch.bfloat16)
        got = run(rows, guard[:rows])
        assert bool((guard[rows] == 7.0).all())
        for name, g, w in zip(("y", "bias", "pre", "gelu"), got, want):
            assert torch.equal(g, w[:rows]), (name, rows)


# Shapes without a fused kernel whose packed weights leave the vector between the factors little of the workspace, for every q above
# the 128 that the one-launch kernel takes on weights as they are: batches in slices whose later ones find the weights packed, and so
# short that they are a few rows (42: 32 and 10; 100: 32, 32, 32 and 4).  Through both calls that have a workspace, with bias and
# nonlinearity.
@pytest.mark.parametrize("rows", (42, 100))
@pytest.mark.parametrize("dims", [(256, 224, 4384), (224, 224, 4416), (256, 160, 6240), (128, 160, 6368), (256, 192, 5152), (256, 256, 3808)], ids=str)
def test_short_slices_without_a_fused_kernel(dims, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    p, q, s = dims
    room = B.MONARCH_STATIC_WORKSPACE_BYTES - 8 * q * (p + s)
    assert 32 <= room // (8 * q) < 64   # rows of the vector between the factors
    sh = synth.Shape("slices_%s" % (dims,), "bf16", rows, 4, p, q, s, config=1010)
    x, R, L, _ = synth.make_inputs(sh)
    bias = synth.quantize(synth.normal(82, (sh.n_out,)), "bf16")
    xd, Rd, Ld, bd = (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(torch.bfloat16) for a in (x, R, L, bias))
    want, want_bias = oracle.fwd(x, R, L), oracle.fwd_bias(x, R, L, bias)

    def check(name, got, want):
        parity_util.check("%s.%s" % (sh.name, name), got.float().cpu().numpy(), want, 2e-2)

    y, ys = B.monarch_fwd_ws(xd, Rd, Ld), torch.empty((rows, sh.n_out), dtype=torch.bfloat16, device="cuda")
    check("y", y, want)
    B.monarch_fwd_static(xd, Rd, Ld, ys)
    assert torch.equal(y, ys)
    check("bias", B.monarch_fwd_bias(xd, Rd, Ld, bd), want_bias)
    pre, act = B.monarch_fwd_bias_gelu(xd, Rd, Ld, bd)
    check("pre", pre, want_bias)
    check("gelu", act, activation.gelu(want_bias))
