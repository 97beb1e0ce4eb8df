"""The shape-generic matrix-core kernels (one launch per contraction) at the sizes where they can go wrong: block sizes
around the 32-wide tiles and the 32-deep chunks, aligned and unaligned pieces, row counts around the tiles and around
the number at which row tiles and batch chunks are dealt to the XCDs; with and without a workspace."""
import numpy as np
import pytest

import oracle
import parity_util
from paper_2204_00595_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}
# B, k, p, q, s
CASES = [(1, 4, 16, 16, 16), (65, 2, 17, 16, 250), (300, 4, 49, 49, 64), (129, 3, 33, 31, 97), (1100, 1, 64, 95, 128),
         (3000, 4, 96, 64, 160), (640, 8, 101, 37, 16), (900, 4, 192, 192, 36),
         (4200, 4, 17, 16, 33), (130, 5, 33, 17, 65), (260, 1, 41, 129, 23)]   # pieces that start anywhere and end at the limit; many chunks


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)


@pytest.mark.parametrize("reading", [0, 1], ids=["reading_a", "reading_b"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=str)
def test_every_call_on_the_shape_generic_kernels(case, dtype, reading):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    sh = synth.Shape("ops_%s" % (case,), dtype, *case, config=400 + parity_util.stable_seed(str(case)))
    flags = B.MONARCH_FLAG_PERM_B if reading else 0
    rd = oracle.READING_B if reading else oracle.READING_A
    x, R, L, dy = synth.make_inputs(sh)
    bias = synth.quantize(synth.normal(77, (sh.n_out,)), dtype)
    xd, Rd, Ld, dyd, bd = (_dev(a, dtype) for a in (x, R, L, dy, bias))
    want_y, want_g = oracle.fwd(x, R, L, rd), oracle.bwd_bias(dy, x, R, L, rd)

    def check(name, got, want):
        parity_util.check("%s.%s" % (sh.name, name), got.float().cpu().numpy(), want, TOL[dtype])

    check("y_ws", B.monarch_fwd_ws(xd, Rd, Ld, flags=flags), want_y)
    check("y", B.monarch_fwd(xd, Rd, Ld, flags=flags), want_y)   # no workspace: the kernels that need none
    check("y_bias", B.monarch_fwd_bias(xd, Rd, Ld, bd, flags=flags), oracle.fwd_bias(x, R, L, bias, rd))
    check("xM", B.monarch_fwd_t(dyd, Rd, Ld, flags=flags), oracle.fwd_t(dy, R, L, rd))
    y, saved = B.monarch_fwd_save(xd, Rd, Ld, flags=flags)
    check("y_save", y, want_y)
    plain = B.monarch_bwd_bias(dyd, xd, Rd, Ld, flags=flags)
    again = B.monarch_bwd_saved(dyd, xd, saved, Rd, Ld, flags=flags, want_dbias=True)
    for name, a, b, w in zip(("dx", "dR", "dL", "dbias"), plain, again, want_g):
        check(name, a, w)
        check(name + "_saved", b, w)
        assert torch.equal(a, b) or saved is None, name   # fixed summation order


# shape-generic fp32 and bf16, and the fused bf16 forward with and without full tiles of 64 rows and whole passes of l tiles
@pytest.mark.parametrize("case", [(65, 4, 49, 33, 64, "f32"), (300, 3, 49, 49, 50, "bf16"), (1, 4, 64, 64, 128, "bf16"), (2051, 4, 192, 192, 576, "bf16"),
                                  (2500, 4, 128, 64, 64, "bf16"), (97, 4, 1024, 256, 256, "bf16")], ids=str)
def test_forward_with_bias_that_keeps_the_vector(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import autograd
    from paper_2204_00595_amd import binding as B
    *dims, dtype = case
    sh = synth.Shape("keep_%s" % (case,), dtype, *dims, config=700 + parity_util.stable_seed(str(case)))
    x, R, L, dy = synth.make_inputs(sh)
    bias = synth.quantize(synth.normal(79, (sh.n_out,)), dtype)
    xd, Rd, Ld, dyd, bd = (_dev(a, dtype) for a in (x, R, L, dy, bias))
    want = (oracle.fwd_bias(x, R, L, bias), *oracle.bwd_bias(dy, x, R, L))
    y, saved = B.monarch_fwd_bias_save(xd, Rd, Ld, bd)
    assert saved is not None
    got = (y, *B.monarch_bwd_saved(dyd, xd, saved, Rd, Ld, want_dbias=True))
    layer = autograd.MonarchLinear(sh.n_in, sh.n_out, nblocks=sh.k, q=sh.q, device="cuda", dtype=xd.dtype)
    with torch.no_grad():
        for par, value in ((layer.R, Rd), (layer.L, Ld), (layer.bias, bd)):
            par.copy_(value)
    xg = xd.clone().requires_grad_(True)
    out = layer(xg)
    out.backward(dyd)
    for name, a, b, w in zip(("y", "dx", "dR", "dL", "dbias"), got, (out, xg.grad, layer.R.grad, layer.L.grad, layer.bias.grad), want):
        parity_util.check("%s.%s" % (sh.name, name), a.float().cpu().numpy(), w, TOL[dtype])
        parity_util.check("%s.layer.%s" % (sh.name, name), b.detach().float().cpu().numpy(), w, TOL[dtype])


# bf16 layers hold the vector between the factors in 32 bits: a result is rounded to 16 bits once, when it is stored, which puts
# every element within 2^-9 of its value (2e-5: sums of products in fp32).  With a 16-bit vector between them the whole is 2.3e-3 off.
ONE_ROUNDING = 2.0 ** -9 + 2e-5


@pytest.mark.parametrize("reading", [0, 1], ids=["reading_a", "reading_b"])
@pytest.mark.parametrize("case", [(2000, 4, 49, 49, 64), (300, 2, 17, 16, 250), (640, 8, 101, 37, 16), (1100, 1, 64, 95, 128), (129, 3, 250, 97, 131)], ids=str)
def test_vector_between_the_factors_keeps_32_bits(case, reading):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    sh = synth.Shape("bits_%s" % (case,), "bf16", *case, config=900 + parity_util.stable_seed(str(case)))
    flags = B.MONARCH_FLAG_PERM_B if reading else 0
    rd = oracle.READING_B if reading else oracle.READING_A
    x, R, L, dy = synth.make_inputs(sh)
    bias = synth.quantize(synth.normal(83, (sh.n_out,)), "bf16")
    xd, Rd, Ld, dyd, bd = (_dev(a, "bf16") for a in (x, R, L, dy, bias))
    want = oracle.bwd(dy, x, R, L, rd)
    y, saved = B.monarch_fwd_bias_save(xd, Rd, Ld, bd, flags=flags)
    got = [("y", B.monarch_fwd_ws(xd, Rd, Ld, flags=flags), oracle.fwd(x, R, L, rd)), ("y_bias", y, oracle.fwd_bias(x, R, L, bias, rd)),
           ("xM", B.monarch_fwd_t(dyd, Rd, Ld, flags=flags), oracle.fwd_t(dy, R, L, rd))]
    got += zip(("dx", "dR", "dL"), B.monarch_bwd(dyd, xd, Rd, Ld, flags=flags), want)
    got += zip(("dx_saved", "dR_saved", "dL_saved"), B.monarch_bwd_saved(dyd, xd, saved, Rd, Ld, flags=flags)[:3], want)
    for name, g, w in got:
        err = parity_util.rel_fro(g.float().cpu().numpy(), w)
        assert err <= ONE_ROUNDING, "%s.%s: %.3e" % (sh.name, name, err)
    for name, g, w in zip(("dR32", "dL32"), B.monarch_bwd(dyd, xd, Rd, Ld, flags=flags | B.MONARCH_FLAG_WGRAD_F32)[1:], want[1:]):
        err = parity_util.rel_fro(g.cpu().numpy(), w)
        assert err <= 1e-5, "%s.%s: %.3e" % (sh.name, name, err)


# four-block shapes with a bf16 forward whose backward has no bf16 kernel: fp32 between the factors for short batches too
@pytest.mark.parametrize("case", [(1, 4, 1024, 256, 1024), (200, 4, 32, 256, 1024), (2560, 4, 1024, 256, 32)], ids=str)
def test_backward_keeps_32_bits_on_short_batches(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    sh = synth.Shape("bits_%s" % (case,), "bf16", *case, config=920 + parity_util.stable_seed(str(case)))
    x, R, L, dy = synth.make_inputs(sh)
    want = oracle.bwd(dy, x, R, L)
    for name, g, w in zip(("dx", "dR", "dL"), B.monarch_bwd(*(_dev(a, "bf16") for a in (dy, x, R, L))), want):
        err = parity_util.rel_fro(g.float().cpu().numpy(), w)
        assert err <= ONE_ROUNDING, "%s.%s: %.3e" % (sh.name, name, err)


# A workspace of the largest batch serves a shorter last one, also where the shorter one asks for more: four-block layers on both
# sides of the limits of the short-batch kernels (wide: 2560 rows, shape-generic bf16: 4096), batches with one chunk more than a
# slightly longer one, and those with a workspace that only the SIMT kernels can use.
LAST = [((128, 128, 512), 4, 2561, 2560, "bf16"), ((192, 192, 192), 4, 2600, 1500, "bf16"), ((96, 96, 96), 4, 4097, 4096, "bf16"),
        ((192, 192, 768), 4, 2049, 2048, "f32"), ((101, 37, 16), 8, 6145, 6144, "bf16"), ((192, 192, 36), 4, 0, 3072, "bf16"),
        ((64, 64, 64), 64, 257, 256, "bf16"), ((256, 256, 1024), 4, 3073, 3072, "bf16"), ((192, 192, 192), 4, 8193, 8192, "bf16"),
        ((64, 96, 96), 2, 9217, 9216, "bf16"), ((32, 32, 32), 32, 4097, 4096, "bf16"), ((16, 16, 16), 16, 4097, 4096, "bf16")]


@pytest.mark.parametrize("case", LAST, ids=str)
def test_workspace_of_the_largest_batch_serves_a_shorter_one(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    (p, q, s), k, most, rows, dtype = case
    code = 0 if dtype == "f32" else 1
    sh = synth.Shape("last_%s" % (case,), dtype, rows, k, p, q, s, config=940 + parity_util.stable_seed(str(case)))
    size = B.monarch_bwd_workspace_bytes(rows, sh.n_in, k, q, s, code)
    if most:
        have = B.monarch_bwd_workspace_bytes(most, sh.n_in, k, q, s, code)
    else:  # what the SIMT kernels ask for
        have = B.monarch_bwd_workspace_bytes(rows, sh.n_in, k, q, s, code, B.MONARCH_FLAG_GENERIC)
    assert have < size
    x, R, L, dy = synth.make_inputs(sh)
    want = oracle.bwd_bias(dy, x, R, L)
    xd, Rd, Ld, dyd = (_dev(a, dtype) for a in (x, R, L, dy))
    guard = 4096
    ws = torch.full((have + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    got = B.monarch_bwd_bias(dyd, xd, Rd, Ld, workspace=ws[:have])
    for name, g, w in zip(("dx", "dR", "dL", "dbias"), got, want):
        parity_util.check("%s.%s" % (sh.name, name), g.float().cpu().numpy(), w, TOL[dtype])
    assert bool((ws[have:] == 0xA5).all())
    with pytest.raises(B.MonarchError) as e:  # not the partial rows of the bias gradient alone
        B.monarch_bwd_bias(dyd, xd, Rd, Ld, workspace=ws[:256])
    assert e.value.status == B.MONARCH_ERR_WORKSPACE


# 64 blocks of 64: fp32 gradients in the room that bf16 ones ask for, and in that of a batch half as long (fewer chunks, down to one)
@pytest.mark.parametrize("rows, room_of", [(2100, 2100), (700, 700), (300, 300), (300, 150), (257, 257)])
def test_workspace_of_bf16_gradients_serves_fp32_ones(rows, room_of):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    sh = synth.Shape("room_%d_%d" % (rows, room_of), "bf16", rows, 64, 64, 64, 64, config=950)
    activations = 2 * 2 * 4096
    have = B.monarch_bwd_workspace_bytes(room_of, 4096, 64, 64, 64, 1) + activations * (rows - room_of)
    assert have < B.monarch_bwd_workspace_bytes(rows, 4096, 64, 64, 64, 1, B.MONARCH_FLAG_WGRAD_F32)
    x, R, L, dy = synth.make_inputs(sh)
    want = oracle.bwd(dy, x, R, L)
    xd, Rd, Ld, dyd = (_dev(a, "bf16") for a in (x, R, L, dy))
    ws = torch.full((have + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    got = B.monarch_bwd(dyd, xd, Rd, Ld, workspace=ws[:have], flags=B.MONARCH_FLAG_WGRAD_F32)
    for name, g, w in zip(("dx", "dR", "dL"), got, want):
        parity_util.check("%s.%s" % (sh.name, name), g.float().cpu().numpy(), w, TOL["bf16"])
    assert bool((ws[have:] == 0xA5).all())


# batches of one chunk or a few, where a chunk's own sum is what errs; the SIMT kernels add 16 rows at a time
@pytest.mark.parametrize("case", [(302, 8, 43, 43, 66), (389, 3, 21, 21, 85), (363, 8, 154, 21, 21), (329, 4, 96, 96, 384)], ids=str)
def test_fp32_weight_gradients_are_as_exact_as_the_simt_kernels(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    sh = synth.Shape("exact_%s" % (case,), "f32", *case, config=960 + parity_util.stable_seed(str(case)))
    x, R, L, dy = synth.make_inputs(sh)
    want = oracle.bwd(dy, x, R, L)
    args = [_dev(a, "f32") for a in (dy, x, R, L)]
    for name, g, simt, w in zip(("dx", "dR", "dL"), B.monarch_bwd(*args), B.monarch_bwd(*args, flags=B.MONARCH_FLAG_GENERIC), want):
        ours, theirs = parity_util.rel_fro(g.cpu().numpy(), w), parity_util.rel_fro(simt.cpu().numpy(), w)
        assert ours <= 1.05 * theirs, "%s.%s: %.3e and %.3e" % (sh.name, name, ours, theirs)   # 5 %: the order of the SIMT atomics varies


# What the bf16 planes of an fp32 operand cannot hold: infinities and NaN (their other planes are NaN), numbers that round to a bf16
# infinity, and rows so small that planes fall below bf16's smallest number.  Those results are as in fp32, and the rest of the batch is too.
@pytest.mark.parametrize("case", [(70, 4, 49, 33, 64, "f32"), (300, 4, 192, 192, 192, "f32"), (130, 3, 40, 128, 257, "f32"), (300, 4, 49, 49, 64, "bf16")], ids=str)
def test_values_that_three_bf16_planes_cannot_hold(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    *dims, dtype = case
    sh = synth.Shape("planes_%s" % (case,), dtype, *dims, config=980 + parity_util.stable_seed(str(case)))
    x, R, L, dy = synth.make_inputs(sh)
    inf = np.float32(np.inf)
    for a in (x, dy):
        a[0, 3], a[1, 5], a[2, 7] = inf, -inf, np.nan
        a[5] *= np.float32(2.0 ** -100)
        a[6] = 0
        if dtype == "f32":
            a[3, 2] = np.float32(3.4e38)   # rounds to infinity in bf16; the sums stay below it
            a[4] *= np.float32(2.0 ** -115)
    R[:, :, 2] *= np.float32(2.0 ** -6)
    L[:, 2 // sh.k, :] *= np.float32(2.0 ** -6)
    xd, Rd, Ld, dyd = (_dev(a, dtype) for a in (x, R, L, dy))
    with np.errstate(all="ignore"):
        want = dict(zip(("dx", "dR", "dL"), oracle.bwd(dy, x, R, L)), y=oracle.fwd(x, R, L))
    got = dict(zip(("dx", "dR", "dL"), B.monarch_bwd(dyd, xd, Rd, Ld)), y=B.monarch_fwd_ws(xd, Rd, Ld))
    limit = TOL[dtype]
    for name in ("y", "dx"):
        for row in range(sh.B):
            g, w = got[name][row].float().cpu().numpy().astype(np.float64), want[name][row]
            fine = np.isfinite(w)
            assert np.array_equal(np.isnan(g), np.isnan(w)) and np.array_equal(g[~fine & ~np.isnan(w)], w[~fine & ~np.isnan(w)]), (sh.name, name, row)
            size = np.linalg.norm(w[fine])
            assert np.linalg.norm(g[fine] - w[fine]) <= limit * size, (sh.name, name, row)
    for name in ("dR", "dL"):   # sums over rows with infinities, NaN and both: nothing finite may come of what is not
        assert not np.isfinite(got[name].float().cpu().numpy()[~np.isfinite(want[name])]).any(), (sh.name, name)
