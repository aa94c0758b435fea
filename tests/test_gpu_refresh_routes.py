"""The ways in and out of the projection refresh: a start basis read where it lies or converted first, results written by
the last step or converted last, in place, with and without conditioning and polishing steps."""
import pytest
import torch

from paper_2510_16415_amd import binding as B

pytestmark = pytest.mark.gpu
M, N, R = 700, 384, 40


def refresh(V0, ldv, ldp, r, left=0, iters=2, cond=8, polish=3, in_place=False, scale=1.0, wscale=1.0):
    gen = torch.Generator(device="cuda").manual_seed(5)
    W = (torch.randn(M, N, generator=gen, device="cuda") * 0.02).to(torch.bfloat16) * wscale
    dim = M if left else N
    V = torch.full((dim, ldv), float("nan"), dtype=torch.bfloat16, device="cuda")
    V[:, :r] = (V0[:dim, :r].float() * scale).to(torch.bfloat16)
    P = V if in_place else torch.full((dim, ldp), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((B.mecefo_projection_workspace_bytes(B.BF16, M, N, r, left),), 255, dtype=torch.uint8, device="cuda")
    B.mecefo_projection_refresh(B.BF16, W, M, N, N, left, V, ldv, r, iters, cond, polish, P, ldp, ws)
    torch.cuda.synchronize()
    assert bool(P[:, :r].isfinite().all()) and bool(P[:, r:].isnan().all())      # columns behind r stay as they were
    return P[:, :r].float()


def start(r):
    gen = torch.Generator(device="cuda").manual_seed(7)
    return (torch.randn(M, r, generator=gen, device="cuda") * N ** -0.5).to(torch.bfloat16)


@pytest.mark.parametrize("left", [0, 1])
@pytest.mark.parametrize("cond,polish", [(8, 3), (8, 0), (0, 0), (0, 3), (1, 1)])
@pytest.mark.parametrize("r", [40, 33])
def test_where_the_result_goes_does_not_change_it(r, cond, polish, left):
    V0, up = start(r), (r + 7) // 8 * 8
    want = refresh(V0, up, up, r, left, cond=cond, polish=polish)
    assert torch.equal(refresh(V0, up, up + 16, r, left, cond=cond, polish=polish), want)
    assert torch.equal(refresh(V0, up, up, r, left, cond=cond, polish=polish, in_place=True), want)


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** 60])
def test_the_scale_of_the_start_basis_does_not_matter(scale):
    V0 = start(R)
    assert torch.equal(refresh(V0, 40, 40, R, scale=scale), refresh(V0, 40, 40, R))


@pytest.mark.parametrize("left", [0, 1])
@pytest.mark.parametrize("cond,polish", [(8, 3), (8, 0), (0, 3)])
@pytest.mark.parametrize("wscale", [2.0 ** -40, 2.0 ** -20, 2.0 ** 20, 2.0 ** 40])
def test_the_scale_of_the_weights_does_not_matter(wscale, cond, polish, left):
    """A power of two in W is one in W^T W X, which its norm takes out again: the same bits, for weights near 1e-14 (a
    down projection that started at zero) as for weights near 1e10."""
    V0 = start(R)
    assert torch.equal(refresh(V0, 40, 40, R, left, cond=cond, polish=polish, wscale=wscale),
                       refresh(V0, 40, 40, R, left, cond=cond, polish=polish))


@pytest.mark.parametrize("left", [0, 1])
@pytest.mark.parametrize("cond,polish", [(8, 3), (8, 0), (0, 3)])
def test_a_start_basis_that_has_to_be_converted(cond, polish, left):
    """Rows of 43 elements are converted and normalised first: the same iteration from the start basis rounded to hi + lo
    (2^-16 of it) instead of exactly.  The span is compared (a conditioning step multiplies a change of the singular values
    by up to 3.4, so without polishing steps the bases differ): bf16 rounding of the halves and of P, 2^-9 of entries of
    equal size, a few times that in the worst direction."""
    V0 = start(R)
    a, b = (torch.linalg.qr(refresh(V0, ld, ld, R, left, cond=cond, polish=polish).double())[0] for ld in (40, 43))
    assert float((b - a @ (a.T @ b)).norm(2)) <= 2e-2


@pytest.mark.parametrize("cond,polish", [(8, 3), (8, 0), (0, 3), (0, 0)])
def test_without_power_rounds(cond, polish):
    """Only conditions and polishes the start basis; its span stays: with V0 = Q diag, against torch's QR in 64 bits."""
    V0 = start(R)
    P = refresh(V0, 40, 40, R, iters=0, cond=cond, polish=polish).double()
    q1, q0 = torch.linalg.qr(P)[0], torch.linalg.qr(V0[:N].double())[0]
    # one bf16 rounding of P: 2^-9 of entries of equal size, a few times that in the worst direction of a conditioned basis
    assert float((q1 - q0 @ (q0.T @ q1)).norm(2)) <= 2e-2


def test_a_zero_matrix_gives_finite_results():
    V0 = torch.zeros(M, R, dtype=torch.bfloat16, device="cuda")
    assert bool((refresh(V0, 40, 40, R) == 0).all())


def test_a_start_basis_whose_rows_lie_far_apart():
    """48 rows that span 2 GiB, further than a product's 32-bit offsets reach: converted first, like rows of 41 elements."""
    dim, r, ldv = 48, 40, 22900000
    rows = start(r)[:dim]
    flat = torch.empty((dim - 1) * ldv + r, dtype=torch.bfloat16, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(11)
    W = torch.randn(200, dim, generator=gen, device="cuda").to(torch.bfloat16)
    out = []
    for V0, ld in ((flat.as_strided((dim, r), (ldv, 1)), ldv), (torch.empty(dim, r + 1, dtype=torch.bfloat16, device="cuda")[:, :r], r + 1)):
        V0.copy_(rows)
        ws = torch.full((B.mecefo_projection_workspace_bytes(B.BF16, 200, dim, r, 0),), 255, dtype=torch.uint8, device="cuda")
        P = torch.empty(dim, r, dtype=torch.bfloat16, device="cuda")
        B.mecefo_projection_refresh(B.BF16, W, 200, dim, dim, 0, V0, ld, r, 2, 8, 3, P, r, ws)
        torch.cuda.synchronize()
        out.append(P)
    assert torch.equal(*out)
