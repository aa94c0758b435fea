"""GPU parity of the block forward (Alg. 2: the same forward in both modes; the modes differ in
what is kept) against the oracle's block_fwd_full, and the forward -> backward chains of both
modes running entirely on the library's kernels."""
import numpy as np
import pytest
import torch

from oracle import mecefo_oracle as O
from paper_2510_16415_amd import binding as B
from paper_2510_16415_amd import inputs as I
from gpu_util import TOL, assert_close, dev, host, relerr, tdtype, poisoned_ws
from test_gpu_full_block import FullBlock, GRADS, make_case, token_major

pytestmark = pytest.mark.gpu
EPS = 1e-6


class Forward:
    def __init__(self, blk: FullBlock, heads, batch, seq):
        self.blk = blk
        b, ld = blk.b, blk.ld_d
        t = tdtype(blk.dtype)
        nan = float("nan")
        self.out = {k: torch.full((b, ld), nan, dtype=t, device="cuda") for k in ("Out", "H", "Q", "K", "V", "O")}
        self.out["L"] = torch.full((batch * heads * seq,), nan, dtype=torch.float32, device="cuda")
        self.inp = {k: blk.inp[k] for k in ("X", "g_attn", "g_ffn", "Wq", "Wk", "Wv", "Wo", "Wg", "Wu", "Wd")}
        self.ws = poisoned_ws(B.mecefo_block_fwd_workspace_bytes(blk.desc, blk.attn))

    def run(self, neighbor=False):
        out = {k: v for k, v in self.out.items() if not neighbor or k in ("Out", "H")}
        B.mecefo_block_fwd(self.blk.desc, self.blk.attn, self.inp, out, self.ws)
        torch.cuda.synchronize()
        return {k: (host(v, self.blk.d) if v.ndim == 2 else host(v)) for k, v in out.items()}


def oracle_forward(p, X, heads, batch, seq):
    out, H, c = O.block_fwd_full(X, p, heads, batch, seq, EPS)
    b, d = X.shape
    return dict(Out=out, H=H, Q=token_major(c["Q"], b, d), K=token_major(c["K"], b, d), V=token_major(c["V"], b, d),
                O=c["O"], L=c["L"].reshape(-1))


def run_fwd(seed, batch, seq, d, f, heads, dtype, pad=0):
    p, X, dOut = make_case(seed, batch, seq, d, f, heads, dtype)
    blk = FullBlock(p, X, dOut, heads, batch, seq, dtype, pad=pad)
    fwd = Forward(blk, heads, batch, seq)
    got = fwd.run()
    want = oracle_forward(p, X, heads, batch, seq)
    errs = assert_close(got, want, TOL[dtype], label=f"fwd {dtype} B{batch} S{seq} d{d} h{heads}: ")
    return p, X, dOut, blk, fwd, got, want, errs


@pytest.mark.parametrize("batch,seq,d,f,heads", [(2, 37, 48, 100, 4), (1, 130, 64, 72, 2), (3, 9, 32, 40, 8)])
def test_block_fwd_f32_ragged(batch, seq, d, f, heads):
    print(run_fwd(21, batch, seq, d, f, heads, "f32")[-1])


@pytest.mark.parametrize("batch,seq,d,f,heads,pad", [(3, 150, 128, 344, 4, 0), (2, 77, 64, 200, 8, 8), (1, 300, 256, 512, 2, 0)])
def test_block_fwd_bf16_ragged(batch, seq, d, f, heads, pad):
    print(run_fwd(22, batch, seq, d, f, heads, "bf16", pad=pad)[-1])


@pytest.mark.parametrize("tile", ["S", "S4", "T", "T2", "X", "K", "LT", "L8R", "L8"])
def test_block_fwd_bf16_forced_tiles_cross_the_diagonal(tile, mecefo_option):
    mecefo_option("tile", tile)
    print(tile, run_fwd(23, 2, 523, 256, 344, 2, "bf16")[-1])
    print(tile, run_fwd(24, 1, 768, 256, 344, 4, "bf16")[-1])


@pytest.mark.parametrize("batch,seq,d,heads,pad", [(2, 523, 256, 2, 0), (1, 768, 256, 4, 8), (3, 1, 128, 2, 0),
                                                   (2, 63, 128, 1, 0), (1, 129, 64, 1, 8), (2, 257, 512, 4, 0)])
def test_block_fwd_bf16_fused_attention_shapes(batch, seq, d, heads, pad):
    """Head dimensions 64 and 128 take the fused attention forward: single tokens, sequences shorter
    than one key block, one past a block boundary, padded row strides."""
    print(run_fwd(29, batch, seq, d, 200, heads, "bf16", pad=pad)[-1])


@pytest.mark.parametrize("tile", ["S", "S4", "T", "T2", "X", "K", "LT", "L8"])
def test_block_fwd_bf16_materialised_scores_on_every_tile(tile, mecefo_option):
    mecefo_option("attention", "gemm")
    mecefo_option("tile", tile)
    print(tile, run_fwd(31, 2, 523, 256, 344, 2, "bf16")[-1])
    print(tile, run_fwd(33, 1, 520, 256, 344, 2, "bf16")[-1])      # a contraction that the 192-row tile takes


@pytest.mark.parametrize("batch,seq,d,heads", [(2, 523, 256, 2), (1, 768, 256, 4)])
def test_block_fwd_bf16_materialised_scores_path(batch, seq, d, heads, mecefo_option):
    """the "attention" = "gemm" switch keeps the chunked fp32-score form (the one other head dimensions use) covered
    at head dimensions 128 and 64."""
    mecefo_option("attention", "gemm")
    print(run_fwd(30, batch, seq, d, 344, heads, "bf16")[-1])


@pytest.mark.parametrize("heads", [8, 16])
def test_block_fwd_bf16_last_round_of_the_qkv_products(heads):
    """264 tiles of 256 x 256 for Q, K and V, 8 more than the CUs: cut up with the rotation behind, or on tiles that rotate."""
    print(run_fwd(34, 22, 256, 1024, 64, heads, "bf16")[-1])


@pytest.mark.parametrize("b,heads,dh", [(1024, 46, 64), (768, 29, 128), (2816, 30, 64)])
def test_block_fwd_bf16_rotates_before_it_rounds(b, heads, dh):
    """Sizes whose plain launch for Q, K and V would be shorter on tiles that cannot rotate: Q and K are rounded to bf16 once
    all the same.  One rounding leaves 2^-7 / sqrt 12 = 2.26e-3 of the power of two below each value, 1.66e-3 of the norm for
    values spread over the binades; two leave sqrt 2 times that, 2.35e-3."""
    d, seq = heads * dh, 256
    gen = torch.Generator(device="cuda").manual_seed(b)
    rnd = lambda n, k, s=1.0: (torch.randn(n, k, generator=gen, device="cuda") * s).to(torch.bfloat16)   # noqa: E731
    inp = dict(X=rnd(b, d), g_attn=torch.ones(d, dtype=torch.bfloat16, device="cuda"),
               g_ffn=torch.ones(d, dtype=torch.bfloat16, device="cuda"), **{k: rnd(d, d, d ** -0.5) for k in ("Wq", "Wk", "Wv", "Wo")},
               Wg=rnd(64, d), Wu=rnd(64, d), Wd=rnd(d, 64))
    desc, attn = B.make_desc(b, d, 64, B.BF16), B.make_attn_desc(b // seq, seq, heads, d)
    out = {k: torch.empty(b, d, dtype=torch.bfloat16, device="cuda") for k in ("Out", "H", "Q", "K", "V", "O")}
    out["L"] = torch.empty(b * heads, device="cuda")
    B.mecefo_block_fwd(desc, attn, inp, out, poisoned_ws(B.mecefo_block_fwd_workspace_bytes(desc, attn)))
    torch.cuda.synchronize()
    x = inp["X"].double()
    xn = (x * torch.rsqrt(x.square().mean(1, keepdim=True) + 1e-6)).to(torch.bfloat16).double()      # the operand of the products
    inv = 10000.0 ** (-torch.arange(dh // 2, device="cuda", dtype=torch.float64) / (dh // 2))
    ang = torch.arange(seq, device="cuda", dtype=torch.float64)[:, None] * inv
    c, s = (t.repeat(b // seq, 1)[:, None, :] for t in (ang.cos(), ang.sin()))
    for k in ("Q", "K"):
        v = (xn @ inp["W" + k.lower()].double().T).view(b, heads, 2, dh // 2)
        want = torch.stack((v[:, :, 0] * c - v[:, :, 1] * s, v[:, :, 1] * c + v[:, :, 0] * s), 2).reshape(b, d)
        err = float((out[k].double() - want).norm() / want.norm())
        print(k, err)
        assert err <= 1.2 * 1.66e-3


def test_fused_attention_random_shapes_forward_then_backward():
    """Seeded sweep over sequence lengths, batch sizes, head counts and both fused head dimensions: the
    forward on the GPU, then the standard-mode backward fed with the tensors that forward kept, each
    against the oracle."""
    rng = np.random.default_rng(20251017)
    for i in range(8):
        dh = int(rng.choice([64, 128]))
        heads = int(rng.integers(1, 4))
        batch = int(rng.integers(1, 4))
        seq = int(rng.integers(1, 600))
        f = int(rng.integers(1, 40)) * 8
        pad = int(rng.integers(0, 2)) * 8
        d = dh * heads
        label = f"case {i}: B{batch} S{seq} heads {heads} dh {dh} f {f} pad {pad}"
        p, X, dOut, blk, fwd, got, want, errs = run_fwd(6000 + i, batch, seq, d, f, heads, "bf16", pad=pad)
        for k in ("H", "Q", "K", "V", "O", "L"):
            blk.inp[k] = fwd.out[k]
        res = blk.run()
        ref = O.block_bwd_full(X, dOut, p, heads, batch, seq, EPS)
        berrs = assert_close(res, ref, TOL["bf16"], keys=["dX"] + GRADS, label=label + " bwd: ")
        print(label, max(errs.values()), max(berrs.values()))


@pytest.mark.parametrize("dh", [64, 128])
def test_fused_attention_with_rising_maxima_and_infinite_scores(dh):
    """The fused forward rescales only when a query's maximum rises by more than 8 (log2 units) above its reference:
    scores whose maximum rises from key block to key block by 6 to 10, by little, by a lot and not at all.  Then keys
    whose scores overflow: -inf is no probability at all, +inf makes the query (and no other) not a number.
    One head; rotary base 1e30 leaves head dimensions from dh/4 on unrotated, where the scores are made:
    rows (a, c, e, 0 ...) of rms 1, q = c in two dimensions, k = 14 a in one and 1e38 e in the other."""
    rng = np.random.default_rng([37, dh])
    steps = [0, 7.5, 8.5, 6, 10, 0.5, -20, 16.5, 7.8, 8.2, 30, -3, 9]
    seq, d, f = 64 * len(steps) + 5, dh, 72
    top = np.cumsum(steps)[np.minimum(np.arange(seq) // 64, len(steps) - 1)]
    a = (top - 10 * rng.random(seq)) / (1.4427 * 14)                 # scores below the block's maximum ...
    a[::64] = top[::64] / (1.4427 * 14)                              # ... which its first key has
    X = np.zeros((seq, d), dtype=np.float32)
    X[:, 0], X[:, 1] = a, np.sqrt(d - a * a)
    eye = lambda: np.zeros((d, d), dtype=np.float32)                 # noqa: E731
    Wq, Wk, Wv, Wo = eye(), eye(), rng.standard_normal((d, d)).astype(np.float32) * d ** -0.5, eye()
    i, j = dh // 4, dh // 4 + 1
    Wq[i, 1] = Wq[j, 1] = 1
    Wk[i, 0], Wk[j, 2] = 14, 1e38
    g = np.ones(d, dtype=np.float32)
    W = dict(Wq=Wq, Wk=Wk, Wv=Wv, Wo=Wo, Wg=np.zeros((f, d), np.float32), Wu=np.zeros((f, d), np.float32),
             Wd=np.zeros((d, f), np.float32), g_attn=g, g_ffn=g)
    desc, attn = B.make_desc(seq, d, f, B.BF16), B.make_attn_desc(1, seq, 1, d, rope_theta=1e30)
    for special in ({}, {70: -4.0, 300: -3.0, seq - 20: 4.0}):       # key -> e
        Xs = X.copy()
        for key, e in special.items():
            Xs[key, 2], Xs[key, 1] = e, np.sqrt(d - a[key] ** 2 - e * e)
        inp = {k: dev(v, "bf16") for k, v in dict(W, X=Xs).items()}
        out = {k: torch.full((seq, d), float("nan"), dtype=torch.bfloat16, device="cuda") for k in ("Out", "H", "Q", "K", "V", "O")}
        out["L"] = torch.full((seq,), float("nan"), device="cuda")
        B.mecefo_block_fwd(desc, attn, inp, out, poisoned_ws(B.mecefo_block_fwd_workspace_bytes(desc, attn)))
        torch.cuda.synchronize()
        q, k, v, o = (out[n].float().cpu() for n in ("Q", "K", "V", "O"))
        # fp32 products, which overflow where the kernel's do
        s = (q @ k.T * dh ** -0.5).masked_fill(torch.triu(torch.ones(seq, seq, dtype=torch.bool), 1), -float("inf"))
        assert int(torch.isinf(torch.tril(s)).sum()) == sum(seq - key for key in special)
        bad = (s == float("inf")).any(1)
        assert int(bad.sum()) == (20 if special else 0)
        assert bool(o[bad].isnan().all()) and not bool(out["L"].cpu()[bad].isfinite().any())
        want = torch.softmax(s.double(), 1)[~bad] @ v.double()
        err = (o[~bad].double() - want).norm(dim=1) / want.norm(dim=1)
        assert float(err.max()) <= 1e-2, int(err.argmax())           # bf16 probabilities and output: 2^-9 each
        # scores up to 90 in fp32 with an FMA on top: 90 x 2^-22 and the rounding of exp2 and log2
        assert float((out["L"].cpu()[~bad].double() - torch.logsumexp(s[~bad].double(), 1)).abs().max()) <= 1e-3


def test_neighbor_mode_forward_keeps_only_h_and_matches_standard_mode():
    p, X, dOut, blk, fwd, std, want, _ = run_fwd(25, 2, 200, 128, 344, 4, "bf16")
    nb = fwd.run(neighbor=True)
    assert set(nb) == {"Out", "H"}
    assert np.array_equal(nb["Out"], std["Out"]) and np.array_equal(nb["H"], std["H"])


@pytest.mark.parametrize("dtype,batch,seq,d,f,heads", [("f32", 2, 64, 64, 172, 4), ("bf16", 2, 300, 256, 688, 4)])
def test_forward_then_backward_both_modes_on_gpu(dtype, batch, seq, d, f, heads):
    """Standard mode: the saved tensors written by the GPU forward feed mecefo_block_bwd_full.
    Neighbor mode: only H is kept and feeds mecefo_block_bwd_skip.  Both against the oracle."""
    p, X, dOut, blk, fwd, got, want, _ = run_fwd(26, batch, seq, d, f, heads, dtype)
    for k in ("H", "Q", "K", "V", "O", "L"):
        blk.inp[k] = fwd.out[k]
    res = blk.run()
    ref = O.block_bwd_full(X, dOut, p, heads, batch, seq, EPS)
    errs = assert_close(res, ref, TOL[dtype], keys=["dX"] + GRADS, label="fwd->full bwd: ")
    print("standard mode chain", errs)
    # neighbor mode
    from gpu_util import Layer
    r = d // 4
    rng = np.random.default_rng(5)
    Pg, Pu = I.random_orthonormal(rng, d, r, dtype), I.random_orthonormal(rng, d, r, dtype)
    Pd = I.random_orthonormal(rng, f, r, dtype)
    lay = Layer(blk.b, d, f, dtype, p["Wg"], p["Wu"], p["Wd"], p["g_ffn"], Pg, Pu, Pd, EPS)
    Hgpu = fwd.run(neighbor=True)["H"]
    res2 = lay.block_bwd_skip(Hgpu, dOut)
    ref2 = O.block_bwd_skip(want["H"], dOut, p["g_ffn"], p["Wg"], p["Wu"], p["Wd"], Pg, Pu, Pd, EPS)
    errs2 = assert_close(res2, ref2, TOL[dtype], label="fwd->skip bwd: ")
    print("neighbor mode chain", errs2)


def test_config_c2_block_fwd():
    cfg = I.CONFIGS["C2"]
    print("C2 fwd", run_fwd(27, cfg.batch, cfg.seq, cfg.d_model, cfg.d_ff, cfg.heads, cfg.dtype)[-1])


def test_config_c5_block_fwd_whole_batch():
    """The 7B-shaped layer at its full batch (4 x 2048 tokens); the oracle walks it one sequence at a time."""
    cfg = I.CONFIGS["C5"]
    heads, batch, seq, d = cfg.heads, cfg.batch, cfg.seq, cfg.d_model
    p, X, dOut = make_case(28, batch, seq, d, cfg.d_ff, heads, cfg.dtype)
    parts = [oracle_forward(p, X[i * seq:(i + 1) * seq], heads, 1, seq) for i in range(batch)]
    want = {k: np.concatenate([q[k] for q in parts]) for k in parts[0]}
    blk = FullBlock.__new__(FullBlock)
    blk.init_from_saved(p, X, dOut, want, heads, batch, seq, cfg.dtype)
    fwd = Forward(blk, heads, batch, seq)
    got = fwd.run()
    print("C5 fwd, whole batch", assert_close(got, want, TOL["bf16"], label="C5 fwd: "))


def test_tile_option_changed_by_another_thread_during_a_forward():
    """The switch may change between any two launches of a call: whether Q and K are rotated in the product's
    epilogue is one decision, whatever the switch says when the product is launched (one head of dimension 128:
    "auto" rotates in the epilogue, "S" in a launch of its own).  Every call succeeds with the usual error."""
    import threading
    b, S, heads, d, f = 1, 64, 1, 128, 344
    gen = torch.Generator(device="cuda").manual_seed(9)
    rnd = lambda n, k, s=1.0: (torch.randn(n, k, generator=gen, device="cuda") * s).to(torch.bfloat16)   # noqa: E731
    inp = dict(X=rnd(S, d), g_attn=torch.ones(d, dtype=torch.bfloat16, device="cuda"),
               g_ffn=torch.ones(d, dtype=torch.bfloat16, device="cuda"),
               **{k: rnd(d, d, d ** -0.5) for k in ("Wq", "Wk", "Wv", "Wo")},
               Wg=rnd(f, d, d ** -0.5), Wu=rnd(f, d, d ** -0.5), Wd=rnd(d, f, f ** -0.5))
    desc, attn = B.make_desc(b * S, d, f, B.BF16), B.make_attn_desc(b, S, heads, d)
    ws = torch.empty(B.mecefo_block_fwd_workspace_bytes(desc, attn), dtype=torch.uint8, device="cuda")
    mk = lambda: dict(Out=torch.empty(S, d, dtype=torch.bfloat16, device="cuda"),   # noqa: E731
                      H=torch.empty(S, d, dtype=torch.bfloat16, device="cuda"))
    ref = mk()
    B.mecefo_block_fwd(desc, attn, inp, ref, ws)
    stop = threading.Event()

    def toggle():
        while not stop.is_set():
            B.mecefo_set_option("tile", "S")
            B.mecefo_set_option("tile", "auto")
    thread = threading.Thread(target=toggle)
    thread.start()
    try:
        for i in range(20):
            out = mk()
            for _ in range(200):
                B.mecefo_block_fwd(desc, attn, inp, out, ws)
            torch.cuda.synchronize()
            for k in ("Out", "H"):
                err = (out[k].double() - ref[k].double()).norm() / ref[k].double().norm()
                assert float(err) <= TOL["bf16"], (i, k, float(err))
    finally:
        stop.set()
        thread.join()
        B.mecefo_set_option("tile", "auto")
