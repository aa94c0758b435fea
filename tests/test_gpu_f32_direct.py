"""fp32 products whose operands go straight to LDS (rows on 16 bytes, K in whole pieces of four) and the same ones with
odd row strides, which are staged through registers: equal bit for bit, and close to fp64."""
import pytest
import torch

from paper_2510_16415_amd import binding as B

pytestmark = pytest.mark.gpu


def rows(n, cols, ld, gen, std=1.0):
    t = torch.full((n, ld), float("nan"), device="cuda")
    t[:, :cols] = torch.randn(n, cols, generator=gen, device="cuda") * std
    return t


def relerr(got, want):
    return float((got.double() - want).norm() / want.norm())


# stages of 64 K: one, fewer than the ring holds, one more than it holds (dual 5, other 6), many; ragged rows and tokens
@pytest.mark.parametrize("b,d,f,r", [(1, 4, 4, 1), (33, 36, 68, 5), (64, 64, 32, 32), (130, 324, 388, 12), (257, 388, 452, 31),
                                     (70, 1000, 1364, 44), (700, 96, 100, 8),
                                     # 512 tiles of dA and of the recompute go straight to LDS, 544 do not
                                     (512, 64, 1024, 8), (513, 64, 1024, 8)])
@pytest.mark.parametrize("side", [B.SIDE_INPUT, B.SIDE_OUTPUT])
def test_both_stagings_give_the_same_sums(b, d, f, r, side):
    up = lambda x: (x + 3) // 4 * 4   # noqa: E731
    out = []
    for pad in (0, 1):                 # pad 1: odd strides
        gen = torch.Generator(device="cuda").manual_seed(b + 3 * f)
        ldd, ldf, ldr = up(d) + pad, up(f) + pad, up(r) + 4 * (1 - pad) + pad
        U, dY = rows(b, d, ldd, gen), rows(b, d, ldd, gen)
        W = [rows(f, d, ldd, gen, d ** -0.5), rows(f, d, ldd, gen, d ** -0.5), rows(d, f, ldf, gen, f ** -0.5)]
        dims = (d, d, f) if side == B.SIDE_INPUT else (f, f, d)
        P = [rows(n, r, ldr, gen, n ** -0.5) for n in dims]
        desc = B.make_desc(b, d, f, B.F32, B.F32, ldd, ldf, ldd, ldf, 1e-6)
        ws = torch.full((B.mecefo_workspace_bytes(desc, r, r, r),), 255, dtype=torch.uint8, device="cuda")
        dU = rows(b, d, ldd, gen)
        g = [torch.full_like(w, float("nan")) for w in W]
        B.mecefo_ffn_bwd_lowrank(desc, U, dY, *W, *(B.proj(p, r) for p in P), side, dU, *g, 0, ws)
        torch.cuda.synchronize()
        out.append([dU[:, :d].clone(), g[0][:, :d].clone(), g[1][:, :d].clone(), g[2][:, :f].clone()])
    u, dy, wg, wu, wd = (t[:, :n].double() for t, n in ((U, d), (dY, d), (W[0], d), (W[1], d), (W[2], f)))
    pg, pu, pd = (p[:, :r].double() for p in P)
    G, Z, da = u @ wg.T, u @ wu.T, dy @ wd
    sg = torch.sigmoid(G)
    dg, dz, a = da * Z * sg * (1 + G * (1 - sg)), da * G * sg, G * sg * Z
    if side == B.SIDE_INPUT:
        want = [dg @ wg + dz @ wu, dg.T @ (u @ pg) @ pg.T, dz.T @ (u @ pu) @ pu.T, dy.T @ (a @ pd) @ pd.T]
    else:
        want = [dg @ wg + dz @ wu, pg @ ((dg @ pg).T @ u), pu @ ((dz @ pu).T @ u), pd @ ((dy @ pd).T @ a)]
    for x, y, w in zip(*out, want):
        assert torch.equal(x, y)
        assert relerr(x, w) <= 1e-5      # the fp32 gate of the other tests


@pytest.mark.parametrize("b,d,f", [(65, 68, 132), (300, 256, 688)])
def test_forward_products(b, d, f):
    gen = torch.Generator(device="cuda").manual_seed(b)
    U, Wg, Wu, Wd = rows(b, d, d, gen), rows(f, d, d, gen, d ** -0.5), rows(f, d, d, gen, d ** -0.5), rows(d, f, f, gen, f ** -0.5)
    desc = B.make_desc(b, d, f, B.F32, B.F32, d, f, d, f, 1e-6)
    A, Y = torch.full((b, f), float("nan"), device="cuda"), torch.full((b, d), float("nan"), device="cuda")
    B.mecefo_ffn_fwd_recompute(desc, U, Wg, Wu, Wd, None, None, A, Y)
    torch.cuda.synchronize()
    g, z = U.double() @ Wg.double().T, U.double() @ Wu.double().T
    assert relerr(A, torch.nn.functional.silu(g) * z) <= 1e-5
    assert relerr(Y, A.double() @ Wd.double().T) <= 1e-5
