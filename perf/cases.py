"""The work that a user of this library has it do, as cases that can be timed and compared.

A case names a path through the public entry points of ``paper_2510_16415_amd.binding`` and its sizes:

  skip     the neighbor-mode backward of one block (mecefo_block_bwd_skip), the library's main call;
           two micro-batches: the node's own one overwrites the gradients, the absorbed one accumulates
  ffn      the same without norm and residual (mecefo_ffn_bwd_lowrank): an expert on its token group
  full     the standard-mode backward of one block (mecefo_block_bwd_full)
  fwd      the forward of one block (mecefo_block_fwd), keeping H only or everything
  stack    forward and backward of a whole neighbor-mode stack (mecefo_stack_fwd_neighbor, _bwd_skip)
  refresh  the projections of one layer's three FFN matrices recomputed (mecefo_projection_refresh),
           warm-started from the previous ones: two rounds, eight conditioning and three polishing steps
  update   what follows a backward pass: gradient average over the ranks (mecefo_grad_average) and
           AdamW (mecefo_adamw_step) on one parameter group

Sizes are those of the library's workload configurations (inputs.CONFIGS); `draw` spreads over the ranges
between and around them.  Inputs are made on the GPU from the seed alone: weights N(0, 0.02^2), gains
around 1, block inputs and upstream gradients N(0, 1), projections with columns of about unit norm.
"""
import math

import torch

from paper_2510_16415_amd import binding as B
from paper_2510_16415_amd import inputs as I

EPS = 1e-6


def _config(path, name, index, **more):
    c = I.CONFIGS[index]
    case = dict(name=name, path=path, dtype=c.dtype, batch=c.batch, seq=c.seq, d=c.d_model, f=c.d_ff)
    case.update(more)
    return case


def listed():
    c2, c3, c4, c5 = (I.CONFIGS[k] for k in ("C2", "C3", "C4", "C5"))
    return [
        # smallest bf16 call: one expert of a mixture on a ragged group of tokens; launches and latency count
        dict(name="ffn_expert", path="ffn", dtype="bf16", batch=1, seq=129, d=512, f=200, rank=32, grad="f32",
             side="input"),
        # the reference-precision block: everything fp32, 256 tokens
        _config("skip", "skip_tiny_f32", "C1", rank=I.CONFIGS["C1"].rank, micro=1, grad="f32", side="input"),
        # a training pass over a small stack in neighbor mode: 8 layers forward and backward
        _config("stack", "stack_60m", "C2", heads=c2.heads, rank=c2.rank, layers=c2.layers),
        # a neighbor's step on one layer of the 350M shape: own micro-batch, then the absorbed one
        _config("skip", "skip_350m_two", "C3", rank=c3.rank, micro=2, grad="f32", side="input"),
        # one layer of the 1B shape, odd d_ff
        _config("skip", "skip_1b", "C4", rank=c4.rank, micro=1, grad="f32", side="input"),
        # the 7B-shaped layer: the headline workload
        _config("skip", "skip_7b", "C5", rank=c5.rank, micro=1, grad="f32", side="input"),
        # a healthy node's backward of the same layers, head dimension 64 at 256 tokens and 128 at 2048
        _config("full", "full_1b", "C4", heads=c4.heads, grad="f32"),
        _config("full", "full_7b", "C5", heads=c5.heads, grad="f32"),
        # forward of a layer: neighbor mode (H only) and standard mode (H, Q, K, V, O, L)
        _config("fwd", "fwd_350m_neighbor", "C3", heads=c3.heads, keep=False),
        _config("fwd", "fwd_7b_standard", "C5", heads=c5.heads, keep=True),
        # Alg. 3's refresh of a layer's three projections, every tau steps
        dict(name="refresh_1b", path="refresh", dtype="bf16", d=c4.d_model, f=c4.d_ff, rank=c4.rank),
        # average over four ranks and AdamW on the FFN weights of one 1B layer
        dict(name="update_1b", path="update", dtype="bf16", n=3 * c4.d_model * c4.d_ff, ranks=4, grad="f32"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _tokens(rng, most, seq_lo=64, seq_hi=2048):
    """(batch, seq) with a log-uniform number of tokens up to `most`; the sequence length need not be round."""
    seq = int(_log(rng, seq_lo, seq_hi))
    if rng.random() < 0.6:
        seq = max(64, seq // 64 * 64)
    return max(1, int(_log(rng, 256, most)) // seq), seq


def draw(rng):
    path = rng.choice(["skip", "skip", "skip", "ffn", "full", "fwd", "stack", "refresh", "update"])
    grad = "f32" if rng.random() < 0.75 else "bf16"
    side = "input" if rng.random() < 0.85 else "output"
    if path == "skip" and rng.random() < 0.2:
        d = 8 * int(_log(rng, 16, 64))
        return dict(path=path, dtype="f32", batch=rng.randint(1, 4), seq=int(_log(rng, 32, 256)), d=d,
                    f=int(d * rng.uniform(2.4, 3.0)), rank=max(8, d // 8 + rng.randint(-3, 3)), micro=1, grad="f32", side=side)
    if path == "ffn":
        return dict(path=path, dtype="bf16", batch=1, seq=int(_log(rng, 16, 1024)), d=64 * rng.randint(4, 16),
                    f=int(_log(rng, 128, 1024)), rank=8 * rng.randint(2, 8), grad=grad, side=side)
    if path == "update":
        return dict(path=path, dtype=rng.choice(["bf16", "bf16", "f32"]), n=int(_log(rng, 3e5, 1.2e8)),
                    ranks=rng.randint(2, 8), grad="f32")
    if path == "stack":
        heads, dh = rng.randint(4, 12), 64
        batch, seq = _tokens(rng, 4096, 64, 512)
        return dict(path=path, dtype="bf16", batch=batch, seq=seq, d=heads * dh, f=int(heads * dh * rng.uniform(2.5, 2.8)),
                    heads=heads, rank=16 * rng.randint(4, 12), layers=rng.randint(4, 10))
    dh = rng.choice([64, 128])
    heads = max(1, round(_log(rng, 512, 4096) / dh))
    d = heads * dh
    f = int(d * rng.uniform(2.5, 2.8))
    if path == "refresh":
        d = min(d, 3072)
        return dict(path=path, dtype="bf16", d=d, f=int(d * rng.uniform(2.5, 2.8)), rank=max(32, d // rng.randint(3, 8)))
    batch, seq = _tokens(rng, 8192)
    if path == "skip":
        micro = 2 if rng.random() < 0.25 and batch * seq * d <= 4096 * 4096 else 1
        return dict(path=path, dtype="bf16", batch=batch, seq=seq, d=d, f=f, rank=max(16, d // rng.randint(3, 8)),
                    micro=micro, grad=grad, side=side)
    if path == "full":
        return dict(path=path, dtype="bf16", batch=batch, seq=seq, d=d, f=f, heads=heads, grad=grad)
    return dict(path="fwd", dtype="bf16", batch=batch, seq=seq, d=d, f=f, heads=heads, keep=rng.random() < 0.5)


# ---- inputs ---------------------------------------------------------------------------------------
class _Maker:
    """Tensors of one case, drawn in a fixed order from one generator."""

    def __init__(self, case, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(I.BASE_SEED + int(seed))
        self.dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        self.code = B.BF16 if case["dtype"] == "bf16" else B.F32

    def normal(self, rows, cols, std=1.0, ld=None, dtype=None):
        t = torch.zeros(rows, ld or cols, dtype=dtype or self.dtype, device="cuda")
        t[:, :cols] = torch.randn(rows, cols, generator=self.gen, device="cuda") * std
        return t

    def gain(self, d):
        return (1 + 0.1 * torch.randn(d, generator=self.gen, device="cuda")).to(self.dtype)

    def like(self, *shape, dtype=None):
        return torch.zeros(*shape, dtype=dtype or self.dtype, device="cuda")


def _up8(x):
    return (x + 7) // 8 * 8


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device="cuda")


def _grad_type(case, m):
    return (torch.float32, B.F32) if case.get("grad", "f32") == "f32" else (m.dtype, m.code)


def _desc(case, m, tokens):
    d, f = case["d"], case["f"]
    return B.make_desc(tokens, d, f, m.code, _grad_type(case, m)[1], d, _up8(f), d, _up8(f), EPS)


def _ffn_weights(m, d, f):
    return dict(Wg=m.normal(f, d, 0.02), Wu=m.normal(f, d, 0.02), Wd=m.normal(d, f, 0.02, _up8(f)))


def _projections(m, d, f, r, side):
    dims = (d, d, f) if side == "input" else (f, f, d)
    return [B.proj(m.normal(n, r, n ** -0.5, _up8(r)), r) for n in dims]


def _ffn_grads(m, d, f, gt):
    return dict(dWg=m.like(f, d, dtype=gt), dWu=m.like(f, d, dtype=gt), dWd=m.like(d, _up8(f), dtype=gt))


def _mha_weights(m, d):
    return {k: m.normal(d, d, 0.02) for k in ("Wq", "Wk", "Wv", "Wo")}


def _rotate(x, batch, seq, heads, dh):
    """Rotary embedding of a token-major [batch * seq, heads * dh] tensor, pairs (j, j + dh / 2)."""
    half = dh // 2
    inv = 10000.0 ** (-torch.arange(half, device="cuda", dtype=torch.float64) / half)
    ang = torch.arange(seq, device="cuda", dtype=torch.float64)[:, None] * inv
    c, s = (t.float()[None, :, None, :] for t in (ang.cos(), ang.sin()))
    v = x.float().view(batch, seq, heads, 2, half)
    a, b = v[:, :, :, 0], v[:, :, :, 1]
    return torch.stack((a * c - b * s, b * c + a * s), 3).reshape(batch * seq, heads * dh).to(x.dtype)


def _saved_by_forward(case, w, g_attn, X):
    """What a forward pass keeps of its attention: rotated Q and K, V, O, the row log-sum-exp, and H."""
    batch, seq, heads, d = case["batch"], case["seq"], case["heads"], case["d"]
    dh = d // heads
    x = X.float()
    xn = (x * torch.rsqrt(x.square().mean(1, keepdim=True) + EPS) * g_attn.float()).to(X.dtype)
    Q, K, V = (torch.nn.functional.linear(xn, w[k]) for k in ("Wq", "Wk", "Wv"))
    Q, K = _rotate(Q, batch, seq, heads, dh), _rotate(K, batch, seq, heads, dh)
    O = torch.empty_like(Q)
    L = torch.empty(batch, heads, seq, dtype=torch.float32, device="cuda")
    mask = torch.triu(torch.ones(seq, seq, dtype=torch.bool, device="cuda"), 1)
    for i in range(batch):
        rows = slice(i * seq, (i + 1) * seq)
        q, k, v = (t[rows].view(seq, heads, dh).transpose(0, 1).float().contiguous() for t in (Q, K, V))
        s = torch.matmul(q, k.transpose(1, 2).contiguous()).mul_(dh ** -0.5).masked_fill_(mask, -math.inf)
        L[i] = torch.logsumexp(s, dim=-1)
        O[rows] = torch.matmul(torch.softmax(s, dim=-1), v).transpose(0, 1).reshape(seq, d).to(O.dtype)
    H = (x + torch.nn.functional.linear(O, w["Wo"]).float()).to(X.dtype)
    return dict(Q=Q, K=K, V=V, O=O, L=L.reshape(-1), H=H)


def prepare(case, seed):
    B.mecefo_init()
    return _PREPARE[case["path"]](case, _Maker(case, seed))


def _prepare_skip(case, m):
    d, f, r, b = case["d"], case["f"], case["rank"], case["batch"] * case["seq"]
    gt, _ = _grad_type(case, m)
    s = dict(case=case, desc=_desc(case, m, b), side=B.SIDE_INPUT if case["side"] == "input" else B.SIDE_OUTPUT,
             **_ffn_weights(m, d, f))
    s["P"] = _projections(m, d, f, r, case["side"])
    s["ws"] = _bytes(B.mecefo_workspace_bytes(s["desc"], r, r, r))
    s["grads"] = _ffn_grads(m, d, f, gt)
    if case["path"] == "ffn":
        s["U"], s["dY"], s["dU"] = m.normal(b, d), m.normal(b, d), m.like(b, d)
        s["out"] = dict(s["grads"], dU=s["dU"])
        return s
    s["gamma"], s["dgamma"] = m.gain(d), m.like(d, dtype=gt)
    s["batches"] = [(m.normal(b, d), m.normal(b, d), m.like(b, d)) for _ in range(case["micro"])]
    s["out"] = dict(s["grads"], dgamma=s["dgamma"], dX=[dX for _, _, dX in s["batches"]])
    return s


def _prepare_full(case, m):
    d, f, b = case["d"], case["f"], case["batch"] * case["seq"]
    gt, _ = _grad_type(case, m)
    mha = _mha_weights(m, d)
    inp = dict(X=m.normal(b, d), dOut=m.normal(b, d), g_attn=m.gain(d), g_ffn=m.gain(d), **mha, **_ffn_weights(m, d, f))
    inp.update(_saved_by_forward(case, mha, inp["g_attn"], inp["X"]))
    out = dict(dX=m.like(b, d), dg_attn=m.like(d, dtype=gt), dg_ffn=m.like(d, dtype=gt), **_ffn_grads(m, d, f, gt),
               **{k: m.like(d, d, dtype=gt) for k in ("dWq", "dWk", "dWv", "dWo")})
    desc, attn = _desc(case, m, b), B.make_attn_desc(case["batch"], case["seq"], case["heads"], d)
    return dict(case=case, desc=desc, attn=attn, inp=inp, out=out,
                ws=_bytes(B.mecefo_block_full_workspace_bytes(desc, attn)))


def _prepare_fwd(case, m):
    d, f, b = case["d"], case["f"], case["batch"] * case["seq"]
    inp = dict(X=m.normal(b, d), g_attn=m.gain(d), g_ffn=m.gain(d), **_mha_weights(m, d), **_ffn_weights(m, d, f))
    out = {k: m.like(b, d) for k in (("Out", "H", "Q", "K", "V", "O") if case["keep"] else ("Out", "H"))}
    if case["keep"]:
        out["L"] = m.like(b * case["heads"], dtype=torch.float32)
    desc, attn = _desc(case, m, b), B.make_attn_desc(case["batch"], case["seq"], case["heads"], d)
    return dict(case=case, desc=desc, attn=attn, inp=inp, out=out,
                ws=_bytes(B.mecefo_block_fwd_workspace_bytes(desc, attn)))


def _prepare_stack(case, m):
    d, f, r, b = case["d"], case["f"], case["rank"], case["batch"] * case["seq"]
    layers, low = [], []
    for _ in range(case["layers"]):
        layers.append(dict(g_attn=m.gain(d), g_ffn=m.gain(d), **_mha_weights(m, d), **_ffn_weights(m, d, f)))
        P = _projections(m, d, f, r, "input")
        low.append(dict(Pg=P[0], Pu=P[1], Pd=P[2], dg_ffn=m.like(d, dtype=torch.float32),
                        **_ffn_grads(m, d, f, torch.float32)))
    ids = torch.randint(0, I.VOCAB, (b,), generator=m.gen, device="cuda")
    X0 = m.normal(I.VOCAB, d, 0.02)[ids].contiguous()
    desc, attn = _desc(case, m, b), B.make_attn_desc(case["batch"], case["seq"], case["heads"], d)
    s = dict(case=case, desc=desc, attn=attn, layers=layers, low=low, X0=X0, dOut=m.normal(b, d), X_out=m.like(b, d),
             dX=m.like(b, d), H=[m.like(b, d) for _ in layers], lw=B.layer_weights(layers), lr=B.layer_lowrank(low),
             ws=_bytes(B.mecefo_stack_workspace_bytes(desc, attn, r, r, r)))
    s["out"] = dict(X_out=s["X_out"], dX=s["dX"], H=s["H"],
                    grads=[{k: q[k] for k in ("dg_ffn", "dWg", "dWu", "dWd")} for q in low])
    return s


def _prepare_refresh(case, m):
    d, f, r = case["d"], case["f"], case["rank"]
    w = _ffn_weights(m, d, f)
    jobs = []
    for W, rows, cols in ((w["Wg"], f, d), (w["Wu"], f, d), (w["Wd"], d, f)):
        V0 = m.normal(cols, r, cols ** -0.5, _up8(r))
        jobs.append((W, rows, cols, V0, m.like(cols, _up8(r))))
    most = max(B.mecefo_projection_workspace_bytes(m.code, rows, cols, r) for _, rows, cols, _, _ in jobs)
    return dict(case=case, code=m.code, jobs=jobs, ws=_bytes(most), out=[j[4] for j in jobs])


def _prepare_update(case, m):
    n = case["n"]
    flat = lambda std, dtype=torch.float32: m.normal(1, n, std, dtype=dtype).view(n)   # noqa: E731
    s = dict(case=case, code=m.code, W=flat(0.02, m.dtype), M=flat(1e-3), V=flat(1e-3).square_(),
             G=[flat(1e-3) for _ in range(case["ranks"])], mean=m.like(n, dtype=torch.float32))
    s["out"] = dict(W=s["W"], M=s["M"], V=s["V"], mean=s["mean"])
    return s


_PREPARE = dict(skip=_prepare_skip, ffn=_prepare_skip, full=_prepare_full, fwd=_prepare_fwd, stack=_prepare_stack,
                refresh=_prepare_refresh, update=_prepare_update)


# ---- one pass -------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    path = case["path"]
    if path == "skip":
        g = s["grads"]
        for i, (H, dOut, dX) in enumerate(s["batches"]):
            B.mecefo_block_bwd_skip(s["desc"], H, dOut, s["gamma"], s["Wg"], s["Wu"], s["Wd"], *s["P"], s["side"], dX,
                                    s["dgamma"], g["dWg"], g["dWu"], g["dWd"], int(i > 0), s["ws"])
    elif path == "ffn":
        g = s["grads"]
        B.mecefo_ffn_bwd_lowrank(s["desc"], s["U"], s["dY"], s["Wg"], s["Wu"], s["Wd"], *s["P"], s["side"], s["dU"],
                                 g["dWg"], g["dWu"], g["dWd"], 0, s["ws"])
    elif path == "full":
        B.mecefo_block_bwd_full(s["desc"], s["attn"], s["inp"], s["out"], 0, s["ws"])
    elif path == "fwd":
        B.mecefo_block_fwd(s["desc"], s["attn"], s["inp"], s["out"], s["ws"])
    elif path == "stack":
        B.mecefo_stack_fwd_neighbor(s["desc"], s["attn"], s["lw"], s["X0"], s["H"], s["X_out"], s["ws"])
        B.mecefo_stack_bwd_skip(s["desc"], s["lw"], s["H"], s["lr"], B.SIDE_INPUT, s["dOut"], s["dX"], 0, s["ws"])
    elif path == "refresh":
        for W, rows, cols, V0, P in s["jobs"]:
            B.mecefo_projection_refresh(s["code"], W, rows, cols, W.stride(0), 0, V0, V0.stride(0), case["rank"],
                                        2, 8, 3, P, P.stride(0), s["ws"])
    else:
        n = case["n"]
        B.mecefo_grad_average(B.F32, s["G"], [1] * case["ranks"], s["mean"], n)
        B.mecefo_adamw_step(s["code"], B.F32, s["W"], s["mean"], s["M"], s["V"], n, 100, 1e-3)
    return s["out"]


# ---- what a pass cannot do without ------------------------------------------------------------------
def _skip_work(case, micro):
    b, d, f, r = case["batch"] * case["seq"], case["d"], case["f"], case["rank"]
    e, g = (2 if case["dtype"] == "bf16" else 4), (4 if case.get("grad", "f32") == "f32" else 2)
    flops = micro * (b * (10 * d * f + 6 * r * (d + f)) + 6 * r * d * f)
    dims = 2 * d + f if case.get("side", "input") == "input" else 2 * f + d
    return flops, micro * 3 * b * d * e + (3 * d * f + r * dims) * e + 3 * d * f * g


def _fwd_work(case, keep):
    b, d, f = case["batch"] * case["seq"], case["d"], case["f"]
    flops = 6 * b * d * f + 8 * b * d * d + 2 * b * case["seq"] * d
    return flops, (b * d * (7 if keep else 3) + 3 * d * f + 4 * d * d) * 2 + (4 * b * case["heads"] if keep else 0)


def work(case):
    path = case["path"]
    if path in ("skip", "ffn"):
        flops, nbytes = _skip_work(case, case.get("micro", 1))
    elif path == "full":
        b, d, f, g = case["batch"] * case["seq"], case["d"], case["f"], (4 if case["grad"] == "f32" else 2)
        flops = 16 * b * d * f + 16 * b * d * d + 5 * b * case["seq"] * d
        nbytes = 8 * b * d * 2 + 4 * b * case["heads"] + (3 * d * f + 4 * d * d) * (2 + g)
    elif path == "fwd":
        flops, nbytes = _fwd_work(case, case["keep"])
    elif path == "stack":
        (f1, n1), (f2, n2) = _fwd_work(case, False), _skip_work(case, 1)
        flops, nbytes = case["layers"] * (f1 + f2), case["layers"] * (n1 + n2)
    elif path == "refresh":
        d, f, r = case["d"], case["f"], case["rank"]
        flops = sum(2 * (4 * d * f * r + 8 * (4 * n * r * r + 2 * r ** 3)) + 3 * 4 * n * r * r for n in (d, d, f))
        nbytes = 2 * (3 * d * f + 2 * r * (2 * d + f))
    else:
        n, w = case["n"], (2 if case["dtype"] == "bf16" else 4)
        flops, nbytes = n * (case["ranks"] + 16), n * (4 * case["ranks"] + 4 + 2 * w + 16)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Seen between two summation orders of a path (another tile size; attention as batched products): bf16
    skip 0.9e-3, fwd 3.7e-3, full 4.0e-3, refresh 4.9e-3, the stack of eight layers 1.2e-2; against the same
    path in 64 bits skip 4.4e-3 and, all fp32, 0.7e-6.  The update is elementwise: single roundings differ."""
    path = case["path"]
    if path == "update":
        return {"rel": 1e-4, "max": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-6, "max": 2e-5}
    if case["dtype"] == "f32":
        return {"rel": 4e-6}
    return {"rel": {"skip": 1e-2, "ffn": 1e-2, "fwd": 1.5e-2, "full": 1.6e-2, "refresh": 2e-2, "stack": 2.5e-2}[path]}
