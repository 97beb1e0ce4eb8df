"""The complex calls with a workspace at block sizes that are no multiple of the 16 outputs of a wave's tile, with block counts that
are multiples of eight (the eight-blocks-per-workgroup stages) and not, and ragged batches."""
import numpy as np
import pytest

from oracle import complex_ref
from paper_2204_00595_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _normal(seed, shape, std):
    return (synth.normal(seed, shape, std) + 1j * synth.normal(seed + 1, shape, std)).astype(np.complex64)


@pytest.mark.parametrize("reading", [0, 1], ids=["reading_a", "reading_b"])
@pytest.mark.parametrize("case", [(1, 24, 24), (700, 24, 24), (33, 40, 8), (257, 40, 5), (31, 48, 48), (515, 48, 3), (64, 56, 16), (2049, 56, 2)], ids=str)
def test_blocks_between_the_tiles(case, reading):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, m, k = case
    x, R, L, dy = (_normal(8800 + 10 * i, shp, std) for i, (shp, std) in enumerate(
        (((rows, k * m), 1.0), ((k, m, m), m ** -0.5), ((k, m, m), m ** -0.5), ((rows, k * m), 1.0))))
    xd, Rd, Ld, dyd = (torch.from_numpy(a).cuda() for a in (x, R, L, dy))
    flags = B.MONARCH_FLAG_PERM_B if reading else 0
    got = [B.monarch_fwd_c64_ws(xd, Rd, Ld, flags=flags), B.monarch_fwd_h_c64_ws(dyd, Rd, Ld, flags=flags)]
    got += list(B.monarch_bwd_c64_ws(dyd, xd, Rd, Ld, flags=flags))
    want = [complex_ref.fwd(x, R, L, reading), complex_ref.fwd_h(dy, R, L, reading)] + list(complex_ref.bwd(dy, x, R, L, reading))
    for name, g, w in zip(("y", "xMh", "dx", "dR", "dL"), got, want):
        g = g.cpu().numpy().astype(np.complex128)
        rel = np.linalg.norm((g - w).reshape(g.shape[0], -1), axis=1) / np.linalg.norm(w.reshape(g.shape[0], -1), axis=1)
        assert float(rel.max()) <= 4e-5, (name, int(rel.argmax()), float(rel.max()))   # no row, no block of a gradient
        assert np.linalg.norm(g - w) / np.linalg.norm(w) <= 1e-5, name


# Infinities, NaN and numbers that the scale of the planes makes infinite (5.3e36 2^24) do not fit them: what comes of them is what
# the SIMT kernels give, element by element, and the rest of the batch is not touched.  A row of tiny numbers fits.
@pytest.mark.parametrize("case", [(70, 16, 16), (40, 24, 8), (65, 64, 8), (33, 40, 5), (100, 64, 64)], ids=str)
def test_values_that_three_bf16_planes_cannot_hold(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, m, k = case
    x, R, L, dy = (_normal(8900 + 10 * i, shp, std) for i, (shp, std) in enumerate(
        (((rows, k * m), 1.0), ((k, m, m), m ** -0.5), ((k, m, m), m ** -0.5), ((rows, k * m), 1.0))))
    for a in (x, dy):
        a[0, 3], a[1, 5], a[2, 7] = np.inf, complex(0, -np.inf), np.nan
        a[3, 9] = 3.4e38 / 64 * 1j
        a[4] *= np.float32(2.0 ** -110)
        a[6] = 0
    xd, Rd, Ld, dyd = (torch.from_numpy(a).cuda() for a in (x, R, L, dy))
    got = [B.monarch_fwd_c64_ws(xd, Rd, Ld), B.monarch_fwd_h_c64_ws(dyd, Rd, Ld), *B.monarch_bwd_c64_ws(dyd, xd, Rd, Ld)]
    want = [B.monarch_fwd_c64(xd, Rd, Ld), B.monarch_fwd_h_c64(dyd, Rd, Ld), *B.monarch_bwd_c64(dyd, xd, Rd, Ld)]
    for name, g, w in zip(("y", "xMh", "dx", "dR", "dL"), got, want):
        g, w = (torch.view_as_real(t).cpu().double().numpy() for t in (g, w))
        fine = np.isfinite(w)
        assert np.array_equal(fine, np.isfinite(g)), name
        for row in range(len(w)):
            a, b = g[row][fine[row]], w[row][fine[row]]
            assert np.linalg.norm(a - b) <= 4e-5 * np.linalg.norm(b), (name, row)


@pytest.mark.parametrize("case", [(70, 32, 32), (100, 64, 64), (40, 64, 5)], ids=str)
def test_real_layers_with_values_that_three_bf16_planes_cannot_hold(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, m, k = case
    x, R, L, dy = (synth.normal(8950 + i, shp, std).astype(np.float32) for i, (shp, std) in enumerate(
        (((rows, k * m), 1.0), ((k, m, m), m ** -0.5), ((k, m, m), m ** -0.5), ((rows, k * m), 1.0))))
    for a in (x, dy):
        a[0, 3], a[1, 5], a[2, 7], a[3, 9], a[6] = np.inf, -np.inf, np.nan, 3.4e38 / 64, 0
        a[4] *= np.float32(2.0 ** -110)
    xd, Rd, Ld, dyd = (torch.from_numpy(a).cuda() for a in (x, R, L, dy))
    generic = B.MONARCH_FLAG_GENERIC
    got = [B.monarch_fwd_ws(xd, Rd, Ld), B.monarch_fwd_t(dyd, Rd, Ld), *B.monarch_bwd(dyd, xd, Rd, Ld)]
    want = [B.monarch_fwd(xd, Rd, Ld, flags=generic), B.monarch_fwd_t(dyd, Rd, Ld, flags=generic), *B.monarch_bwd(dyd, xd, Rd, Ld, flags=generic)]
    for name, g, w in zip(("y", "xM", "dx", "dR", "dL"), got, want):
        g, w = (t.cpu().double().numpy() for t in (g, w))
        fine = np.isfinite(w)
        assert np.array_equal(fine, np.isfinite(g)), name
        for row in range(len(w)):
            a, b = g[row][fine[row]], w[row][fine[row]]
            assert np.linalg.norm(a - b) <= 4e-5 * np.linalg.norm(b), (name, row)


# Real layers of blocks of 32 and 64 read dy in the order of the outer permutation, in pieces of four where the block count allows: for every
# remainder by four, dy as the last bytes of a mapping, and with NaN behind it.
@pytest.mark.parametrize("case", [(33, 32, 3), (64, 32, 5), (5, 32, 66), (33, 64, 1), (32, 64, 2), (65, 64, 67), (40, 64, 4), (31, 32, 12),
                                  (1801, 32, 19), (1001, 64, 18)], ids=str)
def test_real_layers_read_nothing_behind_dy(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, m, k = case
    x, R, L, dy = (synth.normal(8970 + i, shp, std).astype(np.float32) for i, (shp, std) in enumerate(
        (((rows, k * m), 1.0), ((k, m, m), m ** -0.5), ((k, m, m), m ** -0.5), ((rows, k * m), 1.0))))
    xd, Rd, Ld = (torch.from_numpy(a).cuda() for a in (x, R, L))
    flat = torch.from_numpy(dy).cuda().reshape(-1)
    room = torch.full((8 << 20,), float("nan"), device="cuda")   # 32 MiB: a mapping of its own
    lead = (room.numel() - flat.numel()) % 4                     # a tensor starts at a multiple of 16 bytes
    results = []
    for start in (0, room.numel() - flat.numel() - lead):
        view = room[start:start + flat.numel()]
        view.copy_(flat)
        results.append(B.monarch_bwd(view.view(rows, k * m), xd, Rd, Ld))
        view.fill_(float("nan"))
    plain = B.monarch_bwd(flat.view(rows, k * m), xd, Rd, Ld)
    simt = B.monarch_bwd(flat.view(rows, k * m), xd, Rd, Ld, flags=B.MONARCH_FLAG_GENERIC)
    for name, first, last, g, w in zip(("dx", "dR", "dL"), *results, plain, simt):
        assert torch.equal(first, g) and torch.equal(last, g), name
        assert float((g - w).double().norm()) <= 1e-5 * float(w.double().norm()), name


# The backward lays dy out in tiles in one of three ways (by block count and size of dy): (rows, block, blocks, real layer?) on either
# side of the rules, ragged rows.
LAYOUTS = [(77, 32, 11, True), (2501, 64, 7, True), (1801, 32, 19, True), (1001, 64, 18, True), (33, 64, 64, True), (300, 16, 9, False),
           (1501, 24, 12, False), (901, 32, 7, False), (40, 64, 16, False)]


@pytest.mark.parametrize("reading", [0, 1], ids=["reading_a", "reading_b"])
@pytest.mark.parametrize("case", LAYOUTS, ids=str)
def test_layouts_of_dy(case, reading):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, m, k, real = case
    draw = (lambda *a: synth.normal(*a).astype(np.float32)) if real else _normal
    x, R, L, dy = (torch.from_numpy(draw(8990 + 10 * i, shp, std)).cuda() for i, (shp, std) in enumerate(
        (((rows, k * m), 1.0), ((k, m, m), m ** -0.5), ((k, m, m), m ** -0.5), ((rows, k * m), 1.0))))
    flags = B.MONARCH_FLAG_PERM_B if reading else 0
    if real:
        got, want = B.monarch_bwd(dy, x, R, L, flags=flags), B.monarch_bwd(dy, x, R, L, flags=flags | B.MONARCH_FLAG_GENERIC)
    else:
        got, want = B.monarch_bwd_c64_ws(dy, x, R, L, flags=flags), B.monarch_bwd_c64(dy, x, R, L, flags=flags)
    for name, g, w in zip(("dx", "dR", "dL"), got, want):
        # two sums of at most `rows` fp32 products in different orders; per row of dx and per block of a gradient
        g, w = (t.reshape(t.shape[0], -1).to(torch.complex128) for t in (g, w))
        rel = torch.linalg.norm(g - w, dim=1) / torch.linalg.norm(w, dim=1)
        assert float(rel.max()) <= 1e-5, (name, float(rel.max()))


# The same on either side of the lines between gathering dy and laying it out first, and with either number of batch chunks.
BOTH = [(1181, 32, 33, True), (1301, 32, 35, True), (10001, 64, 8, True), (2305, 32, 32, True), (4001, 32, 32, True), (1, 64, 3, True),
        (1250, 64, 12, False), (2049, 64, 4, False), (8301, 24, 12, False), (1501, 16, 56, False), (65, 56, 49, False)]


@pytest.mark.parametrize("case", BOTH, ids=str)
def test_gradients_of_a_factor_in_one_launch(case):
    test_layouts_of_dy(case, 0)


@pytest.mark.parametrize("case", [(160, 64, 64), (161, 56, 56)], ids=str)
def test_values_that_three_bf16_planes_cannot_hold_in_tiles(case):
    test_values_that_three_bf16_planes_cannot_hold(case)


def test_real_layers_with_such_values_in_tiles():
    test_real_layers_with_values_that_three_bf16_planes_cannot_hold((330, 64, 64))


# A workspace with room for half of the chunks of 32 blocks of 32 is taken as before.
def test_fewer_chunks_in_a_shorter_workspace():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_00595_amd import binding as B
    rows, m, k = 4001, 32, 32
    x, R, L, dy = (torch.from_numpy(synth.normal(9100 + i, shp, std).astype(np.float32)).cuda() for i, (shp, std) in enumerate(
        (((rows, k * m), 1.0), ((k, m, m), m ** -0.5), ((k, m, m), m ** -0.5), ((rows, k * m), 1.0))))
    need = B.monarch_bwd_workspace_bytes(rows, k * m, k, m, m, B.MONARCH_F32)
    least = need - 16 * k * m * m * 4   # sixteen chunks of thirty-two
    want = B.monarch_bwd(dy, x, R, L, flags=B.MONARCH_FLAG_GENERIC)
    for room in (need, need - 256, least):
        ws = torch.full((room + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        got = B.monarch_bwd(dy, x, R, L, workspace=ws[:room])
        assert bool((ws[room:] == 0xA5).all())
        for name, g, w in zip(("dx", "dR", "dL"), got, want):
            assert float((g - w).double().norm()) <= 1e-5 * float(w.double().norm()), (room, name)
    with pytest.raises(Exception):
        B.monarch_bwd(dy, x, R, L, workspace=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))
