"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol
the header declares, sizes workspaces, and rejects bad arguments before touching a device."""
import ctypes as C
import os
import re

import pytest

from paper_2510_16415_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "mecefo.h")).read()
    names = sorted(set(re.findall(r"\b(mecefo_[a-z_0-9]+)\s*\(", hdr)))
    assert {"mecefo_ffn_fwd_recompute", "mecefo_ffn_bwd_exact", "mecefo_ffn_bwd_lowrank",
            "mecefo_block_bwd_skip", "mecefo_workspace_bytes", "mecefo_last_error"} <= set(names)
    lib = B.lib()
    for n in names:
        assert hasattr(lib, n), n
    assert B.mecefo_version().startswith("mecefo")


def test_workspace_bytes_grows_with_the_problem():
    small = B.mecefo_workspace_bytes(B.make_desc(256, 256, 688, B.F32), 32, 32, 32)
    big = B.mecefo_workspace_bytes(B.make_desc(8192, 4096, 11008, B.BF16), 1024, 1024, 1024)
    assert 0 < small < big
    # three [b x f] activations dominate at the 7B shape
    assert big >= 3 * 8192 * 11008 * 2


@pytest.mark.parametrize("dtype,b,f,taken,wider", [(B.BF16, 512, 11008, 2048, 2056), (B.F32, 32, 688, 2048, 2052),
                                                  (B.F32, 64, 688, 512, 513)])
def test_workspace_keeps_parts_of_du_only_where_the_norm_backward_takes_them(dtype, b, f, taken, wider):
    """Four fp32 parts of dU, 16 bytes per token and column, up to d = 2048 (and for fp32 whole vectors of four): a wider
    layer needs less."""
    small, large = (B.mecefo_workspace_bytes(B.make_desc(b, d, f, dtype), 32, 32, 32) for d in (taken, wider))
    assert 0 < small - large < 16 * b * taken


def _err(fn, *a):
    with pytest.raises(B.MecefoError) as e:
        fn(*a)
    return e.value


def test_descriptor_validation():
    e = _err(B.mecefo_workspace_bytes, B.make_desc(16, 64, 100, B.BF16), 8, 8, 8)   # ld_act_f=100 not %8
    assert e.status == B.ERR_INVALID_ARG and "multiple of 8" in str(e)
    e = _err(B.mecefo_workspace_bytes, B.make_desc(16, 60, 104, B.BF16), 8, 8, 8)   # d % 8 != 0
    assert e.status in (B.ERR_UNSUPPORTED, B.ERR_INVALID_ARG)
    e = _err(B.mecefo_workspace_bytes, B.make_desc(16, 64, 104, B.BF16, ld_act_d=32), 8, 8, 8)
    assert e.status == B.ERR_INVALID_ARG
    e = _err(B.mecefo_workspace_bytes, B.make_desc(-1, 64, 104, B.F32), 8, 8, 8)
    assert e.status == B.ERR_INVALID_ARG
    e = _err(B.mecefo_workspace_bytes, B.make_desc(16, 64, 104, B.F32, grad_dtype=B.BF16), 8, 8, 8)
    assert e.status == B.ERR_UNSUPPORTED
    e = _err(B.mecefo_workspace_bytes, B.make_desc(1 << 20, 4096, 11008, B.BF16), 8, 8, 8)   # > 2 GiB tensor
    assert e.status == B.ERR_UNSUPPORTED


def test_null_and_rank_validation_happens_before_any_launch():
    lib = B.lib()
    d = B.make_desc(16, 64, 104, B.BF16)
    P = B.Proj(0x1000, 8, 8)
    fake = C.c_void_p(0x10000)
    st = lib.mecefo_block_bwd_skip(C.byref(d), None, fake, fake, fake, fake, fake, P, P, P, 0,
                                   fake, fake, fake, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "H is NULL" in B.mecefo_last_error()
    bad = B.Proj(0x1000, 65, 72)   # rank above the projected dimension d = 64
    st = lib.mecefo_block_bwd_skip(C.byref(d), fake, fake, fake, fake, fake, fake, bad, P, P, 0,
                                   fake, fake, fake, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "rank" in B.mecefo_last_error()
    st = lib.mecefo_block_bwd_skip(C.byref(d), fake, fake, fake, fake, fake, fake, P, P, P, 0,
                                   fake, fake, fake, fake, fake, 0, fake, 16, None)
    assert st == B.ERR_WORKSPACE_TOO_SMALL
    mis = C.c_void_p(0x10002)
    st = lib.mecefo_ffn_bwd_lowrank(C.byref(d), mis, fake, fake, fake, fake, P, P, P, 0,
                                    fake, fake, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "aligned" in B.mecefo_last_error()
    st = lib.mecefo_ffn_bwd_exact(C.byref(d), fake, fake, fake, fake, fake, fake, None,
                                  fake, fake, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "both" in B.mecefo_last_error()
    st = lib.mecefo_block_bwd_skip(C.byref(d), fake, fake, fake, fake, fake, fake, P, P, P, 7,
                                   fake, fake, fake, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "side" in B.mecefo_last_error()


@pytest.mark.parametrize("side", [B.SIDE_INPUT, B.SIDE_OUTPUT])
def test_bf16_projection_beyond_the_buffer_range_is_rejected(side):
    """bf16 operands are addressed with 32-bit offsets: the projection with the most rows (f = 104) may end at the
    last byte below 2 GiB, not behind it.  fp32 ones are not bounded."""
    lib = B.lib()
    f = 104
    fake = C.c_void_p(0x10000)
    last = ((2**31 - 1) // 2 - 8) // (f - 1) // 8 * 8          # (f - 1) ld + r elements of two bytes below 2 GiB
    for dtype, ld, want in ((B.BF16, last, B.ERR_WORKSPACE_TOO_SMALL), (B.BF16, last + 8, B.ERR_UNSUPPORTED),
                            (B.BF16, 1 << 40, B.ERR_UNSUPPORTED), (B.F32, 1 << 40, B.ERR_WORKSPACE_TOO_SMALL)):
        d = B.make_desc(16, 64, f, dtype)
        P = [B.Proj(0x1000, 8, 8) for _ in range(3)]
        P[2 if side == B.SIDE_INPUT else 1] = B.Proj(0x1000, 8, ld)
        st = lib.mecefo_block_bwd_skip(C.byref(d), fake, fake, fake, fake, fake, fake, *P, side,
                                       fake, fake, fake, fake, fake, 0, fake, 16, None)
        assert st == want, (dtype, ld, B.mecefo_last_error())
        assert st != B.ERR_UNSUPPORTED or "reach 2 GiB" in B.mecefo_last_error()


def test_partially_overlapping_dx_is_rejected():
    """dX may be dOut or H themselves (in-place) or lie apart from them; a partial overlap would let the
    Eq. (2) launches read rows of dOut that the norm backward has already overwritten."""
    lib = B.lib()
    d = B.make_desc(16, 64, 104, B.BF16)            # [16 x 64] bf16 = 2048 bytes
    P = B.Proj(0x1000, 8, 8)
    fake = C.c_void_p(0x100000)
    dOut, H = C.c_void_p(0x200000), C.c_void_p(0x300000)
    for dX, other in ((0x200000 + 1024, "dOut"), (0x200000 - 2032, "dOut"), (0x300000 + 16, "H")):
        st = lib.mecefo_block_bwd_skip(C.byref(d), H, dOut, fake, fake, fake, fake, P, P, P, 0,
                                       C.c_void_p(dX), fake, fake, fake, fake, 0, fake, 16, None)
        assert st == B.ERR_INVALID_ARG and "overlaps " + other in B.mecefo_last_error(), B.mecefo_last_error()
    # equal pointers and disjoint ranges pass the alias check (and then fail on the 16-byte workspace)
    for dX in (0x200000, 0x300000, 0x200000 + 2048, 0x200000 - 2048):
        st = lib.mecefo_block_bwd_skip(C.byref(d), H, dOut, fake, fake, fake, fake, P, P, P, 0,
                                       C.c_void_p(dX), fake, fake, fake, fake, 0, fake, 16, None)
        assert st == B.ERR_WORKSPACE_TOO_SMALL, B.mecefo_last_error()


def test_localised_gate_sees_one_wrong_column_of_a_large_matrix():
    """The Frobenius ratio of a 2048 x 5461 matrix moves by 1/sqrt(5461) when one column is wrong, which is
    below the 2e-2 gate; the per-row / per-column measure of the GPU parity tests reads order one."""
    import numpy as np
    from gpu_util import assert_close, local_relerr, relerr
    rng = np.random.default_rng(5)
    want = rng.standard_normal((2048, 5461))
    good = want * (1 + 3e-3 * rng.standard_normal(want.shape))
    assert_close({"dWd": good}, {"dWd": want}, 2e-2)
    wrong_col = good.copy(); wrong_col[:, 5460] = 0.0                       # ragged last column lost
    wrong_row = good.copy(); wrong_row[2047, :] *= 1.1                      # last row scaled
    wrong_tile = good.copy(); wrong_tile[2016:, 5376:] = 0.0                # one wave's last 32 x 85 piece not written
    for name, m in (("col", wrong_col), ("row", wrong_row), ("tile", wrong_tile)):
        assert relerr(m, want) < 2e-2, name                                 # the global gate alone would pass
        loc = local_relerr(m, want)
        assert max(loc.values()) > 5e-2, (name, loc)
        with pytest.raises(AssertionError):
            assert_close({"dWd": m}, {"dWd": want}, 2e-2)
    v = rng.standard_normal(4096)
    assert local_relerr(v * (1 + 1e-3), v)["block"] < 2e-3
    lost = v.copy(); lost[4032:] = 0.0                                      # the last 64 columns of a gain gradient
    assert relerr(lost, v) > 2e-2 or local_relerr(lost, v)["block"] > 0.5
    assert local_relerr(lost, v)["block"] > 0.5


def test_refresh_schedule_of_alg3_and_counter_reset_of_alg1():
    """Alg. 3: the projection of a layer is recomputed when its local step counter is a multiple of tau
    (steps 0, tau, 2 tau, ... of the node's time as a neighbor); Alg. 1: a failure sets the counters of
    the layers taken over to zero, so the next neighbor step refreshes again."""
    tau = 100                                   # the paper's setting (App. E)
    t = (C.c_int64 * 3)(0, 0, 0)
    refreshed = []
    for step in range(250):
        if step == 130:                         # a second failure: layers taken over anew
            B.mecefo_counters_reset(t)
        if B.mecefo_refresh_due(t[0], tau):
            refreshed.append(step)
        for l in range(3):
            t[l] += 1                           # what mecefo_stack_bwd_mixed does per neighbor-mode backward
    assert refreshed == [0, 100, 130, 230]
    assert [B.mecefo_refresh_due(x, 1) for x in (0, 1, 2)] == [True, True, True]
    assert not B.mecefo_refresh_due(5, 0) and not B.mecefo_refresh_due(-1, 100)
    # argument checks of the driver that consumes the schedule (before anything is enqueued)
    lib = B.lib()
    d = B.make_desc(32, 64, 104, B.BF16)
    a = B.make_attn_desc(2, 16, 4, 64)
    fake = C.c_void_p(0x10000)
    modes = (C.c_int * 2)(B.MODE_NEIGHBOR, 7)
    tin, tout = (B.BlockInputs * 2)(), (B.BlockGrads * 2)()
    low = (B.LayerLowrank * 2)()
    st = lib.mecefo_stack_bwd_mixed(C.byref(d), C.byref(a), 2, modes, tin, tout, low, 0, None, None, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "mode" in B.mecefo_last_error()
    modes[1] = B.MODE_STANDARD
    st = lib.mecefo_stack_bwd_mixed(C.byref(d), C.byref(a), 2, modes, tin, tout, None, 0, None, None, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "lowrank" in B.mecefo_last_error()
    pol = B.RefreshPolicy(100, 2, 8, 3)
    st = lib.mecefo_stack_bwd_mixed(C.byref(d), C.byref(a), 2, modes, tin, tout, low, 0, C.byref(pol), None, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "both" in B.mecefo_last_error()
    bad = B.RefreshPolicy(0, 2, 8, 3)
    st = lib.mecefo_stack_bwd_mixed(C.byref(d), C.byref(a), 2, modes, tin, tout, low, 0, C.byref(bad), t, fake, fake, 0, fake, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "tau" in B.mecefo_last_error()
    assert B.mecefo_stack_mixed_workspace_bytes(d, a, 8, 8, 8) >= B.mecefo_workspace_bytes(d, 8, 8, 8)


def test_set_option_validates_names_and_values():
    for tile in ("S", "S4", "T", "T2", "L4", "L8R", "L8", "auto"):
        B.mecefo_set_option("tile", tile)
    B.mecefo_set_option("attention", "gemm")
    B.mecefo_set_option("attention", "auto")
    for name, value in (("tile", "L"), ("tile", "L9"), ("attention", "fast"), ("speed", "max")):
        e = _err(B.mecefo_set_option, name, value)
        assert e.status == B.ERR_INVALID_ARG


def test_full_block_descriptor_and_pointer_validation():
    lib = B.lib()
    d = B.make_desc(32, 64, 104, B.BF16)
    ok = B.make_attn_desc(2, 16, 4, 64)
    n = B.mecefo_block_full_workspace_bytes(d, ok)
    # at least the probabilities: batch * heads * seq * seq bf16 elements
    assert n >= 2 * 4 * 16 * 16 * 2
    big = B.mecefo_block_full_workspace_bytes(B.make_desc(8192, 4096, 11008, B.BF16), B.make_attn_desc(4, 2048, 32, 4096))
    assert big >= 4 * 32 * 2048 * 2048 * 2
    for bad, word in [(B.make_attn_desc(2, 15, 4, 64), "tokens"), (B.make_attn_desc(2, 16, 5, 64), "multiple of heads"),
                      (B.make_attn_desc(2, 16, 32, 64), "multiple of 8"), (B.make_attn_desc(2, 16, 4, 60), "ld_w_dd"),
                      (B.make_attn_desc(2, 16, 4, 64, rope_theta=0.0), "rope_theta")]:
        with pytest.raises(B.MecefoError) as e:
            B.mecefo_block_full_workspace_bytes(d, bad)
        assert word in str(e.value), (word, str(e.value))
    with pytest.raises(B.MecefoError) as e:   # odd head dimension
        B.mecefo_block_full_workspace_bytes(B.make_desc(32, 12, 16, B.F32), B.make_attn_desc(2, 16, 4, 12))
    assert "even" in str(e.value)
    fake = 0x10000
    tin = B.BlockInputs(*([fake] * 17))
    tout = B.BlockGrads(*([fake] * 10))
    ws = C.c_void_p(fake)
    st = lib.mecefo_block_bwd_full(C.byref(d), C.byref(ok), C.byref(tin), C.byref(tout), 0, ws, 16, None)
    assert st == B.ERR_WORKSPACE_TOO_SMALL
    tin.L = None
    st = lib.mecefo_block_bwd_full(C.byref(d), C.byref(ok), C.byref(tin), C.byref(tout), 0, ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "L is NULL" in B.mecefo_last_error()
    tin.L = fake
    tout.dWo = None
    st = lib.mecefo_block_bwd_full(C.byref(d), C.byref(ok), C.byref(tin), C.byref(tout), 0, ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "gradient buffer" in B.mecefo_last_error()
    st = lib.mecefo_block_bwd_full(C.byref(d), C.byref(ok), None, C.byref(tout), 0, ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG


def test_projection_refresh_validation():
    lib = B.lib()
    n = B.mecefo_projection_workspace_bytes(B.BF16, 11008, 4096, 1024)
    # fp32 master copies of the basis (twice) and of W X dominate
    assert n >= (2 * 4096 + 11008) * 1024 * 4
    assert B.mecefo_projection_workspace_bytes(B.BF16, 11008, 4096, 1024, left=1) > n
    for args, word in [((B.BF16, 64, 32, 33), "rank"), ((B.BF16, 0, 32, 4), "m >= 1"), ((7, 64, 32, 4), "dtype")]:
        with pytest.raises(B.MecefoError) as e:
            B.mecefo_projection_workspace_bytes(*args)
        assert word in str(e.value)
    fake, ws = C.c_void_p(0x10000), C.c_void_p(0x20000)
    call = lambda *a: lib.mecefo_projection_refresh(*a)
    st = call(B.BF16, fake, 64, 32, 36, 0, fake, 8, 8, 1, 1, 1, fake, 8, ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "ldw" in B.mecefo_last_error()
    st = call(B.BF16, fake, 64, 32, 32, 0, fake, 4, 8, 1, 1, 1, fake, 8, ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "ldv" in B.mecefo_last_error()
    st = call(B.BF16, fake, 64, 32, 32, 0, None, 8, 8, 1, 1, 1, fake, 8, ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "required" in B.mecefo_last_error()
    st = call(B.BF16, fake, 64, 32, 32, 0, fake, 8, 8, -1, 1, 1, fake, 8, ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "iteration" in B.mecefo_last_error()
    st = call(B.BF16, fake, 64, 32, 32, 0, fake, 8, 8, 1, 1, 1, fake, 8, ws, 64, None)
    assert st == B.ERR_WORKSPACE_TOO_SMALL
    st = call(B.BF16, C.c_void_p(0x10004), 64, 32, 32, 0, fake, 8, 8, 1, 1, 1, fake, 8, ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "aligned" in B.mecefo_last_error()


def test_block_fwd_validation():
    lib = B.lib()
    d = B.make_desc(32, 64, 104, B.BF16)
    a = B.make_attn_desc(2, 16, 4, 64)
    n = B.mecefo_block_fwd_workspace_bytes(d, a)
    assert n >= 4 * 16 * 16 * 4          # fp32 scores of the heads of one sequence
    fake = 0x10000
    tin = B.BlockFwdInputs(*([fake] * 10))
    tout = B.BlockFwdOutputs(fake + 0x100000, fake, fake, fake, None, fake, fake)
    ws = C.c_void_p(fake)
    st = lib.mecefo_block_fwd(C.byref(d), C.byref(a), C.byref(tin), C.byref(tout), ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "all be given" in B.mecefo_last_error()
    tout = B.BlockFwdOutputs(fake, fake, None, None, None, None, None)
    st = lib.mecefo_block_fwd(C.byref(d), C.byref(a), C.byref(tin), C.byref(tout), ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "alias" in B.mecefo_last_error()
    tout = B.BlockFwdOutputs(fake + 0x100000, fake, None, None, None, None, None)
    st = lib.mecefo_block_fwd(C.byref(d), C.byref(a), C.byref(tin), C.byref(tout), ws, 16, None)
    assert st == B.ERR_WORKSPACE_TOO_SMALL
    tin.Wo = None
    st = lib.mecefo_block_fwd(C.byref(d), C.byref(a), C.byref(tin), C.byref(tout), ws, 1 << 30, None)
    assert st == B.ERR_INVALID_ARG and "Wo is NULL" in B.mecefo_last_error()


def test_stage_names_follow_the_header_enum():
    hdr = open(os.path.join(ROOT, "include", "mecefo.h")).read()
    enum = re.findall(r"MECEFO_STAGE_([A-Z_]+)\s*=\s*(\d+)", hdr)
    count = dict(enum).pop("COUNT")
    names = [n.lower() for n, v in sorted(((n, int(v)) for n, v in enum if n != "COUNT"), key=lambda x: x[1])]
    assert names == B.STAGES and int(count) == len(B.STAGES)


def test_forward_workspace_has_no_score_buffer_when_the_attention_is_fused(mecefo_option):
    """bf16 with head dimension 64 or 128 runs the fused attention forward: the workspace is a handful
    of activations.  the "attention" = "gemm" switch (or another head dimension) adds fp32 scores and probabilities."""
    b, d, f, seq, batch = 8192, 4096, 11008, 2048, 4
    desc = B.make_desc(b, d, f, B.BF16)
    fused = B.mecefo_block_fwd_workspace_bytes(desc, B.make_attn_desc(batch, seq, 32, d))       # dh = 128
    other = B.mecefo_block_fwd_workspace_bytes(desc, B.make_attn_desc(batch, seq, 16, d))       # dh = 256
    mecefo_option("attention", "gemm")
    forced = B.mecefo_block_fwd_workspace_bytes(desc, B.make_attn_desc(batch, seq, 32, d))
    act = b * d * 2
    assert 6 * act <= fused <= 6 * act + b * f * 2 + (16 << 20)
    assert forced >= fused + (256 << 20) and other >= fused + (128 << 20)


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""
