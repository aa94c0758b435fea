"""Edges of the norm backward (rows per wave and per workgroup, column remainders of every register variant) and of
the rotary and residual epilogues of the block forward (each tile that carries them), against fp32 torch."""
import math

import pytest
import torch

from paper_2510_16415_amd import binding as B

pytestmark = pytest.mark.gpu
EPS = 1e-6


def rnd(rows, cols, std, gen, ld=None):
    t = torch.full((rows, ld or cols), float("nan"), dtype=torch.bfloat16, device="cuda")
    t[:, :cols] = (torch.randn(rows, cols, generator=gen, device="cuda") * std).to(torch.bfloat16)
    return t


def relerr(got, want):
    return float((got.double() - want.double()).norm() / want.double().norm())


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("b", [1, 15, 17, 37])
@pytest.mark.parametrize("d", [8, 512, 520, 1024, 1032, 2048, 2056, 4096, 4104, 8200])
def test_norm_backward_rows_and_columns(b, d, inplace):
    """dX = dOut + normbwd(dU) and dgamma of the skip backward.  dU is a bf16 tensor behind three bf16 roundings
    (dA, dG, dU: 2^-9 each), dgamma sums it: 1e-2 and 2e-2 in the norm."""
    f, r = 24, 8
    gen = torch.Generator(device="cuda").manual_seed(b * 10007 + d)
    H, dOut = rnd(b, d, 1.0, gen), rnd(b, d, 1.0, gen)
    gamma = (1 + 0.1 * torch.randn(d, generator=gen, device="cuda")).to(torch.bfloat16)
    Wg, Wu, Wd = rnd(f, d, d ** -0.5, gen), rnd(f, d, d ** -0.5, gen), rnd(d, f, 1.0, gen)
    P = [B.proj(rnd(n, r, n ** -0.5, gen), r) for n in (d, d, f)]
    desc = B.make_desc(b, d, f, B.BF16, B.F32, d, f, d, f, EPS)
    ws = torch.full((B.mecefo_workspace_bytes(desc, r, r, r),), 255, dtype=torch.uint8, device="cuda")
    go = dOut.float()
    dX = dOut if inplace else torch.full_like(dOut, float("nan"))
    dg = torch.full((d,), float("nan"), device="cuda")
    dWg, dWu, dWd = (torch.zeros(*s, device="cuda") for s in ((f, d), (f, d), (d, f)))
    B.mecefo_block_bwd_skip(desc, H, dOut, gamma, Wg, Wu, Wd, *P, B.SIDE_INPUT, dX, dg, dWg, dWu, dWd, 0, ws)
    torch.cuda.synchronize()
    x, ga = H.float(), gamma.float()
    rs = torch.rsqrt(x.square().mean(1, keepdim=True) + EPS)
    n = x * rs
    u = (n * ga).to(torch.bfloat16).float()
    g, z, da = u @ Wg.float().T, u @ Wu.float().T, go @ Wd.float()
    sg = torch.sigmoid(g)
    du = (da * z * sg * (1 + g * (1 - sg))) @ Wg.float() + (da * g * sg) @ Wu.float()
    dn = du * ga
    want = go + rs * (dn - n * (dn * n).mean(1, keepdim=True))
    assert relerr(dX.float(), want) <= 1e-2
    assert relerr(dg, (du * n).sum(0)) <= 2e-2


def rotate(x, seq, heads, dh):
    half = dh // 2
    ang = torch.arange(seq, device="cuda", dtype=torch.float64)[:, None] * 10000.0 ** (
        -torch.arange(half, device="cuda", dtype=torch.float64) / half)
    c, s = (t.float()[None, :, None, :] for t in (ang.cos(), ang.sin()))
    v = x.view(-1, seq, heads, 2, half)
    a, b = v[:, :, :, 0], v[:, :, :, 1]
    return torch.stack((a * c - b * s, b * c + a * s), 3).reshape(x.shape)


@pytest.mark.parametrize("batch,seq,heads,dh,pad", [
    (1, 5, 1, 64, 0), (2, 33, 2, 128, 8), (3, 131, 13, 64, 16), (4, 1000, 10, 64, 0), (8, 256, 8, 64, 0),
    (3, 700, 16, 128, 8), (2, 1100, 30, 64, 0)])
def test_forward_with_rotation_and_residual_epilogues(batch, seq, heads, dh, pad):
    """The tile, and whether the rotation is an epilogue, as the size rule has it."""
    check_forward(batch, seq, heads, dh, pad)


@pytest.mark.parametrize("tile,dh", [
    ("S", 64), ("S4", 64), ("L8", 64), ("L8", 128),                      # rotation in the epilogue
    ("S", 128), ("S4", 128), ("T", 64), ("T", 128), ("T2", 64)])         # rotation as a launch
@pytest.mark.parametrize("batch,seq,heads,pad", [(1, 5, 1, 0), (3, 131, 5, 16)])
def test_forward_with_rotation_on_every_tile(batch, seq, heads, pad, tile, dh, mecefo_option):
    """One head in one corner of a tile; rows and heads that end inside a tile, positions that wrap inside one."""
    mecefo_option("tile", tile)
    check_forward(batch, seq, heads, dh, pad)


def check_forward(batch, seq, heads, dh, pad):
    """Q, K (rotated), V and the residual sums H, Out.  bf16 products of a bf16 norm output, one rounding on
    storing: 2^-9 each, below 1e-2; H and Out add a bf16 attention output and FFN of the library's own."""
    b, d, f = batch * seq, heads * dh, 72
    gen = torch.Generator(device="cuda").manual_seed(b + d)
    ld = d + pad
    X = rnd(b, d, 1.0, gen, ld)
    W = {k: rnd(d, d, d ** -0.5, gen) for k in ("Wq", "Wk", "Wv", "Wo")}
    W.update(Wg=rnd(f, d, d ** -0.5, gen), Wu=rnd(f, d, d ** -0.5, gen), Wd=rnd(d, f, f ** -0.5, gen))
    g1, g2 = ((1 + 0.1 * torch.randn(d, generator=gen, device="cuda")).to(torch.bfloat16) for _ in range(2))
    desc, attn = B.make_desc(b, d, f, B.BF16, B.F32, ld, f, d, f, EPS), B.make_attn_desc(batch, seq, heads, d)
    ws = torch.full((B.mecefo_block_fwd_workspace_bytes(desc, attn),), 255, dtype=torch.uint8, device="cuda")
    out = {k: torch.full((b, ld), float("nan"), dtype=torch.bfloat16, device="cuda") for k in ("Out", "H", "Q", "K", "V", "O")}
    out["L"] = torch.full((b * heads,), float("nan"), device="cuda")
    B.mecefo_block_fwd(desc, attn, dict(X=X, g_attn=g1, g_ffn=g2, **W), out, ws)
    torch.cuda.synchronize()
    got = {k: out[k][:, :d].float() for k in ("Out", "H", "Q", "K", "V", "O")}
    for k in ("Out", "H", "Q", "K", "V", "O"):
        assert bool(out[k][:, d:].isnan().all()), k
    x = X[:, :d].float()
    norm = lambda t, g: (t * torch.rsqrt(t.square().mean(1, keepdim=True) + EPS) * g.float()).to(torch.bfloat16).float()
    xn = norm(x, g1)
    assert relerr(got["Q"], rotate(xn @ W["Wq"].float().T, seq, heads, dh)) <= 1e-2
    assert relerr(got["K"], rotate(xn @ W["Wk"].float().T, seq, heads, dh)) <= 1e-2
    assert relerr(got["V"], xn @ W["Wv"].float().T) <= 1e-2
    # attention and FFN on the library's own Q, K, V and H
    mask = torch.triu(torch.ones(seq, seq, dtype=torch.bool, device="cuda"), 1)
    for i in range(batch):
        q, k, v = (got[n][i * seq:(i + 1) * seq].view(seq, heads, dh).transpose(0, 1).contiguous() for n in ("Q", "K", "V"))
        s = torch.matmul(q, k.transpose(1, 2).contiguous()).mul_(dh ** -0.5).masked_fill_(mask, -math.inf)
        o = torch.matmul(torch.softmax(s, -1), v).transpose(0, 1).reshape(seq, d)
        assert relerr(got["O"][i * seq:(i + 1) * seq], o) <= 1e-2
        lse = out["L"].view(batch, heads, seq)[i]
        assert float((lse - torch.logsumexp(s, -1)).abs().max()) <= 1e-2
    assert relerr(got["H"], x + got["O"] @ W["Wo"].float().T) <= 1e-2
    u = norm(got["H"], g2)
    a = (torch.nn.functional.silu(u @ W["Wg"].float().T) * (u @ W["Wu"].float().T)).to(torch.bfloat16).float()
    assert relerr(got["Out"], got["H"] + a @ W["Wd"].float().T) <= 1e-2
