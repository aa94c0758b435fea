"""The 32 x 32 and the 192 x 256 tile, and launches whose last round of 256 x 256 tiles is shared out in halves, quarters or sixteenths:
sizes at which each of them is taken, with edges of the matrices inside the cut-up tiles."""
import pytest
import torch

from paper_2510_16415_amd import binding as B
from test_gpu_gemm_tiles import check_exact_backward, check_forward_products, padded, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,d,f", [(1, 8, 8), (191, 136, 264), (193, 128, 256), (385, 72, 520), (600, 520, 1112)])
def test_products_on_192_row_tiles(b, d, f, mecefo_option):
    mecefo_option("tile", "K")
    check_forward_products(b, d, f)
    check_exact_backward(b, d, f)


@pytest.mark.parametrize("b,d,f", [(1, 8, 1), (31, 32, 33), (33, 72, 31), (63, 64, 65), (97, 520, 264), (129, 512, 2741)])
def test_products_on_32_row_tiles(b, d, f, mecefo_option):
    """One stage (seven of eight waves have nothing to do), stages that do not divide by eight, a ragged K."""
    mecefo_option("tile", "X")
    check_forward_products(b, d, f)
    check_exact_backward(b, d, f)


# 256 CUs take a tile each, so a launch of T tiles has T % 256 in its last round.  Tiles of the SwiGLU products:
# ceil(b / 256) * ceil(f / 128), of dA: ceil(b / 256) * ceil(f / 256), of the weight gradients: 3 * ceil(f / 256) * ceil(d / 256)
@pytest.mark.parametrize("b,d,f", [
    (4100, 72, 4104),      # SwiGLU 561: 49 in quarters; dA 289: 33 in quarters
    (4090, 136, 4104),     # SwiGLU 528: 16 in sixteenths; dA 272: 16 in sixteenths
    (2800, 72, 4104),      # SwiGLU 363: 107 in halves
    (130, 1304, 4104),     # weight gradients 306: 50 in quarters
    (130, 2040, 2810),     # 264: 8 in sixteenths
    (70, 1784, 4104)])     # 357: 101 in halves
def test_last_round_of_the_backward_products(b, d, f, mecefo_option):
    mecefo_option("tile", "LT")
    check_exact_backward(b, d, f)


@pytest.mark.parametrize("b,d,f", [(4100, 72, 4104), (2800, 136, 4104), (4100, 4104, 64), (4090, 4104, 64), (4100, 5400, 64)])
def test_last_round_of_the_forward_products(b, d, f, mecefo_option):
    mecefo_option("tile", "LT")
    check_forward_products(b, d, f)      # the last three: Y 289, 272 and 374 tiles


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("grad", [B.F32, B.BF16])
@pytest.mark.parametrize("f", [22000, 24600, 27600])      # 258, 291 and 324 tiles: sixteenths, quarters, halves
def test_last_round_of_the_expansion(f, grad, accumulate, mecefo_option):
    """K = r is one stage, so every tile adds up in the same order: the gradients equal those of whole tiles, and those on
    tiles of 192 rows."""
    b, d, r = 16, 64, 16
    gen = torch.Generator(device="cuda").manual_seed(f)
    U, dY = padded(b, d, 1.0, gen), padded(b, d, 1.0, gen)
    Wg, Wu, Wd = padded(f, d, d ** -0.5, gen), padded(f, d, d ** -0.5, gen), padded(d, f, f ** -0.5, gen)
    P = [padded(n, r, 1.0, gen) for n in (d, d, f)]
    desc = B.make_desc(b, d, f, B.BF16, grad, d, f, d, f, 1e-6)
    gt = torch.float32 if grad == B.F32 else torch.bfloat16
    old = [torch.randn(*s, generator=gen, device="cuda").to(gt) for s in ((f, d), (f, d), (d, f))]
    out = []
    for tile in ("L8", "LT", "K"):
        mecefo_option("tile", tile)
        ws = torch.full((B.mecefo_workspace_bytes(desc, r, r, r),), 255, dtype=torch.uint8, device="cuda")
        dU = torch.empty(b, d, dtype=torch.bfloat16, device="cuda")
        g = [t.clone() if accumulate else torch.full_like(t, float("nan")) for t in old]
        B.mecefo_ffn_bwd_lowrank(desc, U, dY, Wg, Wu, Wd, *(B.proj(p, r) for p in P), B.SIDE_INPUT, dU, *g, accumulate, ws)
        torch.cuda.synchronize()
        out.append([dU, *g])
    for x, *others in zip(*out):
        assert bool(x.isfinite().all())
        for y in others:
            assert torch.equal(x, y)


def test_last_round_of_the_residual_products(mecefo_option):
    """H = X + O Wo^T and Out = H + A Wd^T with 272 tiles against whole tiles.  The sums run in another order: a bf16
    result differs by single roundings, 2^-9 of it, here its own and those of Q, K and V before it."""
    batch, seq, d, f, heads = 4, 1024, 4104, 64, 27
    b = batch * seq
    gen = torch.Generator(device="cuda").manual_seed(11)
    w = {k: padded(d, d, d ** -0.5, gen) for k in ("Wq", "Wk", "Wv", "Wo")}
    w.update(Wg=padded(f, d, d ** -0.5, gen), Wu=padded(f, d, d ** -0.5, gen), Wd=padded(d, f, f ** -0.5, gen))
    inp = dict(X=padded(b, d, 1.0, gen), g_attn=padded(1, d, 1.0, gen).view(d), g_ffn=padded(1, d, 1.0, gen).view(d), **w)
    desc, attn = B.make_desc(b, d, f, B.BF16, B.F32, d, f, d, f, 1e-6), B.make_attn_desc(batch, seq, heads, d)
    out = []
    for tile in ("L8", "LT"):
        mecefo_option("tile", tile)
        ws = torch.full((B.mecefo_block_fwd_workspace_bytes(desc, attn),), 255, dtype=torch.uint8, device="cuda")
        o = {k: torch.full((b, d), float("nan"), dtype=torch.bfloat16, device="cuda") for k in ("Out", "H")}
        B.mecefo_block_fwd(desc, attn, inp, o, ws)
        torch.cuda.synchronize()
        out.append(o)
    for k in ("H", "Out"):
        assert relerr(out[1][k].float(), out[0][k].float()) <= 2 ** -8
