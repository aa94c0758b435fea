"""The tile configurations of the bf16 GEMM core through the public FFN calls, forced one by one and as the size rule
picks them, with rows, columns and contractions that end inside a tile, inside a 16-byte chunk of K (with NaN
behind it), or just past an edge."""
import pytest
import torch

from paper_2510_16415_amd import binding as B

pytestmark = pytest.mark.gpu


def padded(rows, cols, std, gen):
    """[rows x cols] bf16 values in rows of a multiple of eight elements, NaN behind the columns."""
    t = torch.full((rows, (cols + 7) // 8 * 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    t[:, :cols] = (torch.randn(rows, cols, generator=gen, device="cuda") * std).to(torch.bfloat16)
    return t


def relerr(got, want):
    return float((got.double() - want.double()).norm() / want.double().norm())


# (tokens, d, f): edges of the 64, 128 and 256 tiles and one past them; long ragged contractions with few output
# tiles; larger sizes, whose launches the rule spreads over all configurations
SIZES = [(1, 8, 1), (63, 64, 65), (64, 72, 7), (129, 128, 63), (255, 136, 257), (257, 264, 129),
         (129, 512, 2741), (2048, 512, 1999),
         (700, 1000, 1111), (3000, 2504, 1107), (2048, 1536, 2741), (4100, 4096, 1037)]
# what every configuration is forced onto: a single stage, stages that the wave groups of "T2" share out unevenly, and
# several workgroups per dimension of the largest tile
FORCED = [(t, *s) for t in ("S", "S4", "T", "T2", "L8") for s in
          ((1, 8, 1), (63, 64, 65), (129, 128, 63), (257, 264, 129), (129, 512, 2741), (600, 520, 1111))]


@pytest.mark.parametrize("b,d,f", SIZES)
def test_forward_products_with_a_ragged_contraction(b, d, f):
    check_forward_products(b, d, f)


@pytest.mark.parametrize("tile,b,d,f", FORCED)
def test_forward_products_on_every_tile(tile, b, d, f, mecefo_option):
    mecefo_option("tile", tile)
    check_forward_products(b, d, f)


def check_forward_products(b, d, f):
    """A = silu(U Wg^T) * (U Wu^T) and Y = A Wd^T: both operands K-contiguous, K = f ends anywhere.  Error: one
    bf16 rounding of A, one of Y (2^-9 each) and the fp32 sums: the gate of 1e-2 leaves a factor of two."""
    gen = torch.Generator(device="cuda").manual_seed(b * 7 + f)
    U = padded(b, d, 1.0, gen)
    Wg, Wu, Wd = padded(f, d, d ** -0.5, gen), padded(f, d, d ** -0.5, gen), padded(d, f, f ** -0.5, gen)
    ldf = Wd.shape[1]
    desc = B.make_desc(b, d, f, B.BF16, B.F32, d, ldf, d, ldf, 1e-6)
    A = torch.full((b, ldf), float("nan"), dtype=torch.bfloat16, device="cuda")
    Y = torch.full((b, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.mecefo_ffn_fwd_recompute(desc, U, Wg, Wu, Wd, None, None, A, Y)
    torch.cuda.synchronize()
    g, z = U.float() @ Wg.float().T, U.float() @ Wu.float().T
    want = torch.nn.functional.silu(g) * z
    assert relerr(A[:, :f].float(), want) <= 1e-2
    assert bool((A[:, f:] == 0).all())
    assert relerr(Y.float(), A[:, :f].float() @ Wd[:, :f].float().T) <= 1e-2


@pytest.mark.parametrize("b,d,f", SIZES)
def test_exact_backward_products(b, d, f):
    check_exact_backward(b, d, f)


@pytest.mark.parametrize("tile,b,d,f", FORCED)
def test_exact_backward_products_on_every_tile(tile, b, d, f, mecefo_option):
    mecefo_option("tile", tile)
    check_exact_backward(b, d, f)


def check_exact_backward(b, d, f):
    """dA (K-strided B), the fused SwiGLU backward, dU (two K segments) and the three weight gradients (both
    operands K-strided) against the same steps in fp32 torch.  The library keeps dA, dG, dZ and A in bf16: 2^-9
    per rounding, at most three in a row, below 1e-2 in the norm."""
    gen = torch.Generator(device="cuda").manual_seed(b + 13 * f)
    U, dY = padded(b, d, 1.0, gen), padded(b, d, 1.0, gen)
    Wg, Wu, Wd = padded(f, d, d ** -0.5, gen), padded(f, d, d ** -0.5, gen), padded(d, f, f ** -0.5, gen)
    ldf = Wd.shape[1]
    desc = B.make_desc(b, d, f, B.BF16, B.F32, d, ldf, d, ldf, 1e-6)
    ws = torch.full((B.mecefo_workspace_bytes(desc, 0, 0, 0),), 255, dtype=torch.uint8, device="cuda")
    dU = torch.full((b, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dWg, dWu = (torch.full((f, d), float("nan"), device="cuda") for _ in range(2))
    dWd = torch.full((d, ldf), float("nan"), device="cuda")
    B.mecefo_ffn_bwd_exact(desc, U, dY, Wg, Wu, Wd, None, None, dU, dWg, dWu, dWd, 0, ws)
    torch.cuda.synchronize()
    u, dy, wg, wu, wd = U.float(), dY.float(), Wg.float(), Wu.float(), Wd[:, :f].float()
    g, z, da = u @ wg.T, u @ wu.T, dy @ wd
    sg = torch.sigmoid(g)
    dg, dz, a = da * z * sg * (1 + g * (1 - sg)), da * g * sg, g * sg * z
    assert relerr(dU.float(), dg @ wg + dz @ wu) <= 1e-2
    assert relerr(dWg, dg.T @ u) <= 1e-2
    assert relerr(dWu, dz.T @ u) <= 1e-2
    assert relerr(dWd[:, :f], dy.T @ a) <= 1e-2


@pytest.mark.parametrize("b,d,f", [(1, 1, 1), (33, 31, 65), (64, 64, 32), (257, 130, 67), (1100, 522, 2051)])
def test_exact_backward_products_f32(b, d, f):
    """The fp32 core (32 x 32 tiles, and 64 x 64 for the largest size) with odd row strides, NaN behind every row
    and K ends inside a four-element load, against fp64: 1e-5 in the norm, the fp32 gate of the other tests."""
    gen = torch.Generator(device="cuda").manual_seed(b + 17 * f)

    def rows(n, cols, pad, std):
        t = torch.full((n, cols + pad), float("nan"), device="cuda")
        t[:, :cols] = torch.randn(n, cols, generator=gen, device="cuda") * std
        return t

    U, dY = rows(b, d, 3, 1.0), rows(b, d, 3, 1.0)
    Wg, Wu, Wd = rows(f, d, 1, d ** -0.5), rows(f, d, 1, d ** -0.5), rows(d, f, 5, f ** -0.5)
    desc = B.make_desc(b, d, f, B.F32, B.F32, d + 3, f, d + 1, f + 5, 1e-6)
    ws = torch.full((B.mecefo_workspace_bytes(desc, 0, 0, 0),), 255, dtype=torch.uint8, device="cuda")
    dU, dWg, dWu, dWd = rows(b, d, 3, 1.0), rows(f, d, 1, 1.0), rows(f, d, 1, 1.0), rows(d, f, 5, 1.0)
    B.mecefo_ffn_bwd_exact(desc, U, dY, Wg, Wu, Wd, None, None, dU, dWg, dWu, dWd, 0, ws)
    torch.cuda.synchronize()
    u, dy, wg, wu, wd = (t[:, :n].double() for t, n in ((U, d), (dY, d), (Wg, d), (Wu, d), (Wd, f)))
    g, z, da = u @ wg.T, u @ wu.T, dy @ wd
    sg = torch.sigmoid(g)
    dg, dz, a = da * z * sg * (1 + g * (1 - sg)), da * g * sg, g * sg * z
    for got, n, want in ((dU, d, dg @ wg + dz @ wu), (dWg, d, dg.T @ u), (dWu, d, dz.T @ u), (dWd, f, dy.T @ a)):
        assert relerr(got[:, :n], want) <= 1e-5
        assert bool(got[:, n:].isnan().all())


def test_f32_projection_with_a_row_stride_beyond_the_buffer_range():
    """A projection whose rows lie so far apart that the matrix spans more than 2 GiB is read like a dense one."""
    b, d, f, r = 70, 96, 130, 8
    gen = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")   # noqa: E731
    U, dY, Wg, Wu, Wd = rnd(b, d), rnd(b, d), rnd(f, d) * 0.1, rnd(f, d) * 0.1, rnd(d, f) * 0.1
    dense = [rnd(n, r) for n in (d, d, f)]
    far = torch.empty(f, 4400000, device="cuda")          # 130 rows of 17.6 MB: 2.29 GB
    far[:, :r] = dense[2]
    desc = B.make_desc(b, d, f, B.F32, B.F32, d, f, d, f, 1e-6)
    ws = torch.empty(B.mecefo_workspace_bytes(desc, r, r, r), dtype=torch.uint8, device="cuda")
    out = []
    for last in (dense[2], far):
        g = [torch.zeros(*s, device="cuda") for s in ((b, d), (f, d), (f, d), (d, f))]
        B.mecefo_ffn_bwd_lowrank(desc, U, dY, Wg, Wu, Wd, B.proj(dense[0], r), B.proj(dense[1], r), B.proj(last, r),
                                 B.SIDE_INPUT, g[0], g[1], g[2], g[3], 0, ws)
        torch.cuda.synchronize()
        out.append(g)
    for x, y in zip(*out):
        assert torch.equal(x, y)


@pytest.mark.parametrize("side", [B.SIDE_INPUT, B.SIDE_OUTPUT])
@pytest.mark.parametrize("ld", [8_388_607, 9_000_001, 18_000_000])
def test_f32_projection_whose_tile_rows_span_more_than_32_bits(ld, side):
    """Rows 36 MB apart put the last of a stage's 64 K rows (project) behind 2 GiB, rows of 72 MB those of a
    32-row tile (expand) as well, and the 64 K rows behind 4 GiB.  8388607 is the last stride in reach of 32-bit
    offsets.  Both sides read a projection in both products; the results are those of the dense matrix."""
    b, d, f, r = 70, 96, 130, 8
    gen = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")   # noqa: E731
    U, dY, Wg, Wu, Wd = rnd(b, d), rnd(b, d), rnd(f, d) * 0.1, rnd(f, d) * 0.1, rnd(d, f) * 0.1
    rows = (d, d, f) if side == B.SIDE_INPUT else (f, f, d)
    dense = [rnd(n, r) for n in rows]
    which = rows.index(f)
    far = torch.empty(f, ld, device="cuda")
    far[:, :r] = dense[which]
    desc = B.make_desc(b, d, f, B.F32, B.F32, d, f, d, f, 1e-6)
    ws = torch.empty(B.mecefo_workspace_bytes(desc, r, r, r), dtype=torch.uint8, device="cuda")
    out = []
    for last in (dense[which], far):
        P = [last if i == which else t for i, t in enumerate(dense)]
        g = [torch.zeros(*s, device="cuda") for s in ((b, d), (f, d), (f, d), (d, f))]
        B.mecefo_ffn_bwd_lowrank(desc, U, dY, Wg, Wu, Wd, *(B.proj(p, r) for p in P), side, *g, 0, ws)
        torch.cuda.synchronize()
        out.append(g)
    for x, y in zip(*out):
        assert torch.equal(x, y)


# dA and the recompute in one launch: 64 x 64 tiles with two groups of waves and with one, 128 x 128 tiles on four waves
# and on eight, with rows, columns and contractions that end inside a tile
@pytest.mark.parametrize("b,d,f", [(16, 256, 128), (65, 520, 201), (37, 72, 15), (306, 552, 1899), (534, 24, 4481),
                                   (2047, 520, 1371), (2078, 1016, 594), (3835, 712, 369)])
def test_backward_products_with_the_recompute_in_one_launch(b, d, f):
    check_exact_backward(b, d, f)
