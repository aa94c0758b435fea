"""The skip and the full backward where the norm backward adds up the parts of dU itself (two to four of them, in bf16 and
fp32, over column remainders and ragged rows), where the sum of the gain gradient and the norm recompute ride on products'
launches or go out by themselves, and in a workspace that has no room for the parts."""
import pytest
import torch

from paper_2510_16415_amd import binding as B

pytestmark = pytest.mark.gpu
EPS = 1e-6


def relerr(got, want):
    return float((got.double() - want.double()).norm() / want.double().norm())


def skip(b, d, f, dtype, short=0, inplace=False, want_dgamma=True, accumulate=0):
    gen = torch.Generator(device="cuda").manual_seed(b * 31 + d + f)
    tt, dt = (torch.bfloat16, B.BF16) if dtype == "bf16" else (torch.float32, B.F32)
    ldf, r = (f + 7) // 8 * 8, 8

    def rnd(rows, cols, std, ld=None):
        t = torch.full((rows, ld or cols), float("nan"), dtype=tt, device="cuda")
        t[:, :cols] = (torch.randn(rows, cols, generator=gen, device="cuda") * std).to(tt)
        return t
    H, dOut, gamma = rnd(b, d, 1.0), rnd(b, d, 1.0), (1 + 0.1 * torch.randn(d, generator=gen, device="cuda")).to(tt)
    Wg, Wu, Wd = rnd(f, d, d ** -0.5), rnd(f, d, d ** -0.5), rnd(d, f, f ** -0.5, ldf)
    P = [B.proj(rnd(n, r, n ** -0.5), r) for n in (d, d, f)]
    desc = B.make_desc(b, d, f, dt, B.F32, d, ldf, d, ldf, EPS)
    ws = torch.full((B.mecefo_workspace_bytes(desc, r, r, r) - short,), 255, dtype=torch.uint8, device="cuda")
    go = dOut.double()
    dX = dOut if inplace else torch.full_like(dOut, float("nan"))
    dg = torch.ones(d, device="cuda")
    dW = [torch.zeros(*s, device="cuda") for s in ((f, d), (f, d), (d, ldf))]
    B.mecefo_block_bwd_skip(desc, H, dOut, gamma, Wg, Wu, Wd, *P, B.SIDE_INPUT, dX, dg if want_dgamma else None, *dW,
                            accumulate, ws)
    torch.cuda.synchronize()
    x, ga, Wg, Wu, Wd = H.double(), gamma.double(), Wg.double(), Wu.double(), Wd[:, :f].double()
    rs = torch.rsqrt(x.square().mean(1, keepdim=True) + EPS)
    n = x * rs
    u = (n * ga).to(tt).double()
    g, z, da = u @ Wg.T, u @ Wu.T, go @ Wd
    sg = torch.sigmoid(g)
    du = (da * z * sg * (1 + g * (1 - sg))) @ Wg + (da * g * sg) @ Wu
    dn = du * ga
    want = go + rs * (dn - n * (dn * n).mean(1, keepdim=True))
    # bf16: three roundings in a row behind dX (dA, dG, dX: 2^-9 each), dgamma sums such values; fp32: sums of up to 2 f terms
    tol = 1e-2 if dtype == "bf16" else 1e-5
    assert relerr(dX, want) <= tol
    if want_dgamma:
        assert relerr(dg - accumulate, (du * n).sum(0)) <= 2 * tol
    return dX, dg, dW


SIZES = [(1, 512, 3001), (37, 520, 4000), (129, 512, 2741), (130, 1032, 1500), (257, 2056, 1111), (300, 264, 2000), (67, 4104, 520)]


@pytest.mark.parametrize("b,d,f", SIZES)
def test_norm_backward_behind_a_cut_contraction(b, d, f):
    dX, dg, dW = skip(b, d, f, "bf16")
    again = skip(b, d, f, "bf16", inplace=True, want_dgamma=False)
    assert torch.equal(dX, again[0]) and all(torch.equal(p, q) for p, q in zip(dW, again[2]))
    skip(b, d, f, "bf16", accumulate=1)


@pytest.mark.parametrize("b,d,f", SIZES[:4])
def test_workspace_without_room_for_the_parts(b, d, f):
    """Of the size that calls took before the parts had a region of their own: dU goes out whole."""
    skip(b, d, f, "bf16", short=512)


@pytest.mark.parametrize("b,d,f", [(1, 64, 200), (33, 72, 1000), (65, 256, 688), (256, 128, 2000)])
def test_norm_backward_behind_a_cut_contraction_fp32(b, d, f):
    dX, _, _ = skip(b, d, f, "f32")
    assert torch.equal(dX, skip(b, d, f, "f32", inplace=True)[0])


@pytest.mark.parametrize("tile", ["L4", "L8R", "L8", "S", "X"])
def test_side_jobs_on_every_kind_of_kernel(tile, mecefo_option):
    """The register-staged kernels carry none: their launches leave the job to its own."""
    mecefo_option("tile", tile)
    skip(129, 520, 333, "bf16")


@pytest.mark.parametrize("b", [2047, 2048, 2049])
def test_norm_recompute_up_to_4_mib(b):
    skip(b, 1024, 264, "bf16")


@pytest.mark.parametrize("alias", ["none", "dOut", "O"])
def test_full_backward_whose_dx_lies_over_an_input(alias):
    """The weight gradients follow the norm backward, unless dX lies over O, which they read: dX and every gradient are the same."""
    b, d, f, heads = 256, 128, 264, 2
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda").to(torch.bfloat16)
    t = {k: rnd(b, d) for k in ("X", "H", "dOut", "Q", "K", "V", "O")}
    w = {k: rnd(d, d) * d ** -0.5 for k in ("Wq", "Wk", "Wv", "Wo")}
    w |= {"Wg": rnd(f, d) * d ** -0.5, "Wu": rnd(f, d) * d ** -0.5, "Wd": rnd(d, f) * f ** -0.5, "g_attn": rnd(d), "g_ffn": rnd(d)}
    L = torch.full((2 * heads, b // 2), 6.0, device="cuda")
    desc = B.make_desc(b, d, f, B.BF16, B.F32, d, f, d, f, EPS)
    attn = B.make_attn_desc(2, b // 2, heads, d)

    def run(over):
        i = {k: v.clone() for k, v in t.items()}
        dX = torch.empty_like(i["X"]) if over == "none" else i[over]
        g = {k: torch.empty_like(v, dtype=torch.float32) for k, v in w.items()}
        ws = torch.full((B.mecefo_block_full_workspace_bytes(desc, attn),), 255, dtype=torch.uint8, device="cuda")
        B.mecefo_block_bwd_full(desc, attn, dict(**i, **w, L=L), dict(dX=dX, **{f"d{k}": v for k, v in g.items()}), 0, ws)
        torch.cuda.synchronize()
        return [dX, *g.values()]
    for got, want in zip(run(alias), run("none")):
        assert torch.equal(got, want) and bool(torch.isfinite(want).all())
