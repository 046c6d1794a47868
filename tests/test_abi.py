"""C ABI contract, checked without a GPU: the library loads, exports what
include/swr.h declares, and validates every argument before any HIP call."""
import ctypes
import os
import re

import pytest

import paper_2512_13921_amd as swr

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "swr.h")

BF16, F32 = swr.SWR_DTYPE_BF16, swr.SWR_DTYPE_F32
OK, E_NULL, E_SHAPE, E_DTYPE, E_BLOCK, E_ALIGN, E_ALIAS, E_UNSUP, E_HIP, E_VER, E_SCRATCH = (
    0, -1, -2, -3, -4, -5, -6, -7, -8, -9, -10)

# Where a GPU is visible, a call that passes validation with the fake
# addresses below would launch kernels on them: such calls are skipped there.
NO_GPU = not os.path.exists("/dev/kfd")
reaches_launch = pytest.mark.skipif(not NO_GPU, reason="fake device addresses would reach a kernel launch")

# Fake, well-aligned "device" addresses far apart: validation never dereferences them.
GB = 1 << 30
X, A, B_, C, Y, DY, DX, DA, DB, DC, V = (GB * (i + 1) for i in range(11))


def problem(B=2, T=256, H=4, D=64, block=64, dtype=BF16, residual=False, run_len=0,
            x_strides=None, a_strides=None, per_channel=False):
    xs = x_strides or (T * H * D, H * D, D)
    as_ = a_strides or (T * H, H, 1)
    return swr.make_problem(B, T, H, D, block, dtype, xs, as_, residual, run_len, per_channel)


def fwd(p, x=X, a=A, b=B_, c=C, y=Y, v_=0):
    v = ctypes.c_void_p
    return swr.load().swr_forward(ctypes.byref(p) if p is not None else None,
                                  v(x), v(a), v(b), v(c), v(y), v(v_), None)


def bwd(p, x=X, a=A, b=B_, c=C, dy=DY, v_=V, dx=DX, da=DA, db=DB, dc=DC):
    v = ctypes.c_void_p
    return swr.load().swr_backward(ctypes.byref(p), v(x), v(a), v(b), v(c), v(dy), v(v_), v(dx),
                                   v(da), v(db), v(dc), None)


def car(p, x=X, a=A, b=B_, v_=V):
    v = ctypes.c_void_p
    return swr.load().swr_carriers(ctypes.byref(p), v(x), v(a), v(b), v(v_), None)


def test_library_exports_every_declared_symbol():
    text = open(HEADER).read()
    names = set(re.findall(r"^\s*(?:const\s+)?\w+\*?\s+\*?(swr_\w+)\s*\(", text, re.M))
    assert {"swr_forward", "swr_backward", "swr_carriers", "swr_error_string", "swr_abi_version",
            "swr_launch_info", "swr_carrier_elems"} <= names
    lib = swr.load()
    for name in names:
        assert hasattr(lib, name), name


def test_abi_version_and_struct_layout():
    assert swr.swr_abi_version() == swr.SWR_ABI_VERSION == 1
    text = open(HEADER).read()
    assert "#define SWR_ABI_VERSION 1" in text
    # the ctypes mirror must match the C struct: 2 int32, 5 int64, uint32 + int32, 7 int64
    assert ctypes.sizeof(swr.SwrProblem) == 4 + 4 + 5 * 8 + 4 + 4 + 7 * 8


@pytest.mark.parametrize("code", [OK, E_NULL, E_SHAPE, E_DTYPE, E_BLOCK, E_ALIGN, E_ALIAS,
                                  E_UNSUP, E_HIP, E_VER, E_SCRATCH, 17])
def test_error_strings(code):
    s = swr.swr_error_string(code)
    assert isinstance(s, str) and s


def test_null_problem():
    assert fwd(None) == E_NULL


def test_version_mismatch():
    p = problem()
    p.abi_version = 2
    assert fwd(p) == E_VER and bwd(p) == E_VER


@pytest.mark.parametrize("kw,code", [
    (dict(dtype=7), E_DTYPE),
    (dict(T=-1), E_SHAPE), (dict(B=-3), E_SHAPE), (dict(D=0), E_SHAPE),
    (dict(block=48), E_BLOCK), (dict(block=256), E_BLOCK), (dict(block=0), E_BLOCK),
    (dict(D=24), E_UNSUP), (dict(D=8), E_UNSUP), (dict(D=272), E_UNSUP), (dict(D=4096), E_UNSUP),
    (dict(run_len=100), E_UNSUP), (dict(run_len=-64), E_UNSUP),
    (dict(block=128, run_len=64), E_UNSUP),
    (dict(x_strides=(256 * 4 * 64, 4 * 64, 1)), E_SHAPE),           # heads overlap channels
    (dict(a_strides=(256 * 4, 1, 1)), E_SHAPE),                       # a overlaps itself
    # sizes whose product passes 2^63 (the sanitized build of these tests sees an overflow)
    (dict(B=1 << 31, T=1 << 31, H=(1 << 31) + 1, D=16, x_strides=(1, 1, 16), a_strides=(1, 1, 1)), E_SHAPE),
    (dict(T=2 ** 63 - 1, D=64, x_strides=(1, 1, 64), a_strides=(1, 1, 1)), E_SHAPE),
    (dict(B=1 << 40, H=1 << 40, D=256, x_strides=(1, 1, 256), a_strides=(1, 1, 1)), E_SHAPE),
])
def test_shape_validation(kw, code):
    p = problem(**kw)
    assert fwd(p) == code and bwd(p) == code and car(p) == code


@reaches_launch
@pytest.mark.parametrize("D", [48, 80, 96, 112, 144, 160, 192, 208, 240, 256])
@pytest.mark.parametrize("per_channel", [False, True])
def test_any_multiple_of_16_up_to_256(D, per_channel):
    # the jagged window's forward, carriers and backward take any D % 16 == 0 up
    # to 256 (past validation only the launch is left, which fails without a GPU)
    for dtype in (BF16, F32):
        p = problem(D=D, dtype=dtype, per_channel=per_channel)
        assert fwd(p) in (OK, E_HIP) and bwd(p) in (OK, E_HIP) and car(p) in (OK, E_HIP)
        assert bwd(p, v_=0) in (OK, E_HIP)
        assert swr.swr_carrier_elems(p) == 2 * 4 * (256 // 64) * D
    # the other entry points keep the kernels' own widths
    p = problem(D=D)
    assert swr.load().swr_exact_workspace_bytes(ctypes.byref(p)) == E_UNSUP


@pytest.mark.parametrize("D,per_channel,heads_x", [
    (48, False, 1), (112, False, 1), (144, False, 2), (256, False, 2),
    (48, True, 1), (96, True, 2), (144, True, 4), (256, True, 4)])
def test_wide_and_odd_heads_launch_plan(D, per_channel, heads_x):
    # heads wider than a kernel head (128 channels, 64 with a per-channel
    # decay) run as 2 or 4 virtual heads: the backward's grid grows with them
    base = swr.swr_launch_info(problem(B=2, T=4096, H=4, D=64, block=64, per_channel=per_channel))
    info = swr.swr_launch_info(problem(B=2, T=4096, H=4, D=D, block=64, per_channel=per_channel))
    seqs = 2 * 4 * heads_x
    assert info["bwd_workgroups"] == seqs * -(-4096 // info["bwd_run_len"])
    assert info["bwd_workgroups"] >= base["bwd_workgroups"] * heads_x // 2


def test_unknown_flags_and_reserved():
    for bit in (16, 32, 1 << 31):
        p = problem()
        p.flags = bit
        assert fwd(p) == E_UNSUP and bwd(p) == E_UNSUP and car(p) == E_UNSUP
    p = problem()
    p.reserved = 1
    assert bwd(p) == E_UNSUP


def test_empty_problems_are_noops_even_with_null_pointers():
    for kw in (dict(T=0), dict(B=0), dict(H=0)):
        p = problem(**kw)
        assert fwd(p, 0, 0, 0, 0, 0) == OK
        assert bwd(p, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0) == OK
        assert car(p, 0, 0, 0, 0) == OK


@pytest.mark.parametrize("which", range(5))
def test_null_pointers_forward(which):
    ptrs = [X, A, B_, C, Y]
    ptrs[which] = 0
    assert fwd(problem(), *ptrs) == E_NULL


@pytest.mark.parametrize("which", [0, 1, 2, 3, 4, 6, 7, 8, 9])
def test_null_pointers_backward(which):
    ptrs = [X, A, B_, C, DY, V, DX, DA, DB, DC]
    ptrs[which] = 0
    assert bwd(problem(), *ptrs) == E_NULL


@reaches_launch
@pytest.mark.parametrize("kw", [dict(), dict(D=128, block=128), dict(dtype=F32, per_channel=True),
                                dict(D=16, block=16, T=1000)])
def test_backward_without_carriers_passes_validation(kw):
    # the problem statement's call shape (inputs and coefficients only): NULL
    # carriers pass validation (the kernels recompute them) and reach the launch,
    # which without a GPU is the only failure left
    p = problem(**kw)
    assert bwd(p, v_=0) == bwd(p) != E_NULL
    assert bwd(p, v_=0) in (OK, E_HIP)
    # everything else is still validated with NULL carriers
    assert bwd(p, v_=0, x=0) == E_NULL and bwd(p, v_=0, dx=DB) == E_ALIAS
    assert bwd(p, v_=0, da=DA + 2) == E_ALIGN


@pytest.mark.parametrize("which", range(4))
def test_null_pointers_carriers(which):
    ptrs = [X, A, B_, V]
    ptrs[which] = 0
    assert car(problem(), *ptrs) == E_NULL


def test_alignment():
    # bf16, D = 64: each lane reads 4 channels = 8 bytes.
    assert fwd(problem(), x=X + 4) == E_ALIGN
    assert fwd(problem(), y=Y + 2) == E_ALIGN
    assert bwd(problem(), da=DA + 2) == E_ALIGN
    assert fwd(problem(D=128), c=C + 8) == E_ALIGN     # 16-byte vectors at D = 128
    assert fwd(problem(dtype=F32), a=A + 2) == E_ALIGN
    # row stride of 65 elements breaks the 8-byte vectors
    assert fwd(problem(H=1, x_strides=(256 * 65, 65, 65))) == E_ALIGN
    assert fwd(problem(), v_=V + 8) == E_ALIGN          # carriers: 16-byte aligned
    assert bwd(problem(), v_=V + 4) == E_ALIGN
    assert car(problem(), v_=V + 8) == E_ALIGN


def test_aliasing():
    assert fwd(problem(), y=X) == E_ALIAS
    assert fwd(problem(), y=A) == E_ALIAS
    assert fwd(problem(), y=X + 64) == E_ALIAS
    assert bwd(problem(), dx=DB) == E_ALIAS
    assert bwd(problem(), dc=DY) == E_ALIAS
    assert bwd(problem(), da=A) == E_ALIAS
    assert bwd(problem(), db=B_) == E_ALIAS
    assert fwd(problem(), v_=X) == E_ALIAS              # carriers written by the forward
    assert fwd(problem(), v_=Y) == E_ALIAS
    assert car(problem(), v_=A) == E_ALIAS
    assert bwd(problem(), dx=V) == E_ALIAS              # carriers read by the backward
    # (inputs may alias each other: exercised with real tensors in the GPU tests,
    # since a call that passes validation launches a kernel)


def test_per_channel_validation():
    # a and da take the [B, T, H, D] layout of x; every call below fails before any launch
    pc = dict(per_channel=True)
    assert fwd(problem(D=40, **pc)) == E_UNSUP and bwd(problem(block=48, **pc)) == E_BLOCK
    assert fwd(problem(**pc), a=A + 2) == E_ALIGN          # a needs x's 8-byte lane vectors
    assert fwd(problem(dtype=F32, **pc), a=A + 8) == E_ALIGN
    assert bwd(problem(**pc), da=DA + 8) == E_ALIGN        # 4 fp32 channels per lane: 16 bytes
    assert bwd(problem(D=32, **pc), da=DA + 4) == E_ALIGN  # 2 fp32 channels per lane: 8 bytes
    # D = 128 runs as two 64-channel halves: x needs only the 8-byte (bf16) lane vectors
    assert fwd(problem(D=128, **pc), x=X + 4) == E_ALIGN
    assert fwd(problem(D=128, **pc), y=Y + 8, x=X + 4) == E_ALIGN
    # a's span is x's span: an output inside it aliases
    span_x = 2 * 256 * 4 * 64 * 2
    assert fwd(problem(**pc), y=A + span_x - 64) == E_ALIAS
    assert bwd(problem(**pc), dx=A + span_x - 64) == E_ALIAS
    assert bwd(problem(**pc), da=X + span_x - 64) == E_ALIAS
    # sa_* are ignored with per-channel decay: even overlapping ones are accepted
    # (checked through launch_info, which never launches)
    p = problem(a_strides=(1, 1, 1), **pc)
    assert swr.swr_launch_info(p)["fwd_workgroups"] > 0
    p = problem(a_strides=(1, 1, 1))
    assert swr.load().swr_launch_info(ctypes.byref(p), None, None, None, None) == E_SHAPE


def test_per_channel_launch_shape():
    # B=8, T=16384, H=16, D=128 with per-channel decay: 32 virtual heads of 64 channels
    p = problem(B=8, T=16384, H=16, D=128, block=128, per_channel=True)
    info = swr.swr_launch_info(p)
    assert info["fwd_workgroups"] == 8 * 16 * (-(-16384 // info["fwd_run_len"]))
    assert info["bwd_workgroups"] == 8 * 32 * (-(-16384 // info["bwd_run_len"]))
    assert swr.swr_carrier_elems(p) == 8 * 16 * 128 * 128


def test_backward_grid_targets():
    # the backward's default grid: one 8-wave group per CU at block 128 (256),
    # 4-wave groups at block 64 about 1024 (128 channels) or 8192 (64)
    info = swr.swr_launch_info(problem(B=8, T=4096, H=16, D=128, block=64))
    assert info["bwd_workgroups"] == 8 * 16 * (-(-4096 // info["bwd_run_len"]))
    assert 1024 <= info["bwd_workgroups"] < 2048
    info = swr.swr_launch_info(problem(B=16, T=8192, H=32, D=64, block=64))
    assert info["bwd_workgroups"] == 16 * 32 * (-(-8192 // info["bwd_run_len"]))
    assert 8192 <= info["bwd_workgroups"] < 16384


def test_carrier_elems():
    p = problem(B=2, T=250, H=3, D=64, block=64)
    assert swr.swr_carrier_elems(p) == 2 * 3 * 4 * 64     # ceil(250 / 64) = 4 blocks
    assert swr.load().swr_carrier_elems(ctypes.byref(problem(block=48))) == E_BLOCK


def test_offsets_beyond_32_bits_rejected():
    # a row stride whose 16-row span exceeds 2^31 bytes cannot be addressed
    huge = (1 << 27)
    assert fwd(problem(H=1, x_strides=(huge * 300, huge, huge))) == E_UNSUP


def test_launch_info_defaults():
    # headline workload: B=8, T=16384, H=16, D=128, block 128
    p = problem(B=8, T=16384, H=16, D=128, block=128)
    info = swr.swr_launch_info(p)
    # the forward's workgroups hold 2 heads each, the backward's one
    for k, heads in (("fwd", 2), ("bwd", 1)):
        rl, wg = info[k + "_run_len"], info[k + "_workgroups"]
        assert rl % 128 == 0 and wg == 8 * (16 // heads) * (-(-16384 // rl))
    assert info["fwd_workgroups"] == 512 and info["bwd_workgroups"] == 256   # 8-wave backward groups
    p = problem(B=1, T=1000, H=1, D=16, block=16, run_len=192)
    info = swr.swr_launch_info(p)
    assert info["fwd_run_len"] == info["bwd_run_len"] == 192
    assert info["fwd_workgroups"] == info["bwd_workgroups"] == 6          # H = 1: one head per group
    p = problem(B=3, T=1000, H=6, D=16, block=16, run_len=192)
    info = swr.swr_launch_info(p)
    assert info["fwd_workgroups"] == 3 * 3 * 6 and info["bwd_workgroups"] == 3 * 6 * 6
    # a problem too small to fill the forward's grid keeps one head per group
    p = problem(B=1, T=1024, H=4, D=64, block=64, dtype=F32)
    assert swr.swr_launch_info(p)["fwd_workgroups"] == 4 * 16
    p = problem(B=2, T=1000, H=5, D=16, block=16, run_len=192)        # odd H: one head per group
    assert swr.swr_launch_info(p)["fwd_workgroups"] == 2 * 5 * 6


def test_non_contiguous_layouts_accepted():
    # [B, H, T, D] storage described through strides is valid
    B, T, H, D = 2, 256, 4, 64
    p = problem(B=B, T=T, H=H, D=D, x_strides=(H * T * D, D, T * D), a_strides=(H * T, 1, T))
    assert swr.swr_launch_info(p)["fwd_run_len"] > 0


# ----------------------------------------------------------------------------- exact recurrence

H0, HL, WS, DH0, DHL = (GB * (i + 20) for i in range(5))


def xfwd(p, x=X, a=A, b=B_, c=C, h0=H0, y=Y, v_=V, hl=HL, ws=WS):
    v = ctypes.c_void_p
    return swr.load().swr_exact_forward(ctypes.byref(p), v(x), v(a), v(b), v(c), v(h0), v(y), v(v_),
                                        v(hl), v(ws), None)


def xbwd(p, x=X, a=A, b=B_, c=C, dy=DY, h0=H0, v_=V, dhl=DHL, dx=DX, da=DA, db=DB, dc=DC, dh0=DH0, ws=WS):
    v = ctypes.c_void_p
    return swr.load().swr_exact_backward(ctypes.byref(p), v(x), v(a), v(b), v(c), v(dy), v(h0), v(v_),
                                         v(dhl), v(dx), v(da), v(db), v(dc), v(dh0), v(ws), None)


def _agg_runs(T, seqs, bwd_run_len):
    # the exact backward's stage I halves the backward's runs while fewer
    # than 2048 groups would result (keeping a multiple of 64 tokens)
    agg = bwd_run_len
    while agg % 128 == 0 and seqs * (-(-T // agg)) < 2048:
        agg //= 2
    return -(-T // agg)


def test_exact_workspace_bytes():
    p = problem(B=8, T=16384, H=16, D=128, block=128)
    info = swr.swr_launch_info(p)
    nr = max(-(-16384 // info["fwd_run_len"]), -(-16384 // info["bwd_run_len"]),
             _agg_runs(16384, 8 * 16, info["bwd_run_len"]))
    assert nr == 16           # 1024-token aggregate runs: 2048 stage-I groups
    # the three-stage backward: per (batch, head) and run, aggregate end state,
    # entering state (D each), decay product; the one-pass forward: two counters
    # (16 floats), then per 128-token chunk a flag, a decay product and two end
    # states (D each) -- the larger of the two
    stages = 8 * 16 * nr * (2 * 128 + 1)
    chunks = 8 * 16 * (16384 // 128)
    chain = 16 + 2 * chunks + 2 * chunks * 128
    assert swr.swr_exact_workspace_bytes(p) == max(stages, chain) * 4 == chain * 4
    # float32 heads of 128 run the one-pass forward as two virtual heads of 64:
    # a flag and a decay product per chunk of each half
    pf = problem(B=8, T=16384, H=16, D=128, block=128, dtype=F32)
    chain32 = 16 + 2 * (2 * chunks) + 2 * chunks * 128
    assert swr.swr_exact_workspace_bytes(pf) == max(stages, chain32) * 4
    assert swr.swr_exact_workspace_bytes(problem(T=0)) == 0
    lib = swr.load()
    # a per-channel decay keeps one run decay product per channel
    pc = problem(B=2, T=256, H=4, D=64, block=64, per_channel=True)
    info = swr.swr_launch_info(pc)
    nr = max(-(-256 // info["fwd_run_len"]), -(-256 // info["bwd_run_len"]),
             _agg_runs(256, 2 * 4, info["bwd_run_len"]))
    assert swr.swr_exact_workspace_bytes(pc) == 2 * 4 * nr * (3 * 64) * 4
    # ... and its one-pass forward, per 128-token chunk of each 64-channel half
    # of a head, a flag (padded to 4) and a decay product, an aggregate and an
    # inclusive state per channel -- larger than the stages at the headline shape
    pcl = problem(B=8, T=16384, H=16, D=128, block=128, per_channel=True)
    n = 8 * 16 * 2 * 128
    assert swr.swr_exact_workspace_bytes(pcl) == (16 + n + 3 * n * 64) * 4
    assert lib.swr_exact_workspace_bytes(ctypes.byref(problem(block=48))) == E_BLOCK


def test_exact_validation():
    p = problem()
    # a per-channel decay takes x's layout and lane-vector alignment (bf16, D = 64: 8 bytes)
    assert xfwd(problem(per_channel=True), a=A + 2) == E_ALIGN
    assert xbwd(problem(per_channel=True), da=DA + 8) == E_ALIGN
    assert xfwd(problem(D=48)) == E_UNSUP and xbwd(problem(block=48)) == E_BLOCK
    for kw in ("x", "a", "b", "c", "y", "ws"):
        assert xfwd(p, **{kw: 0}) == E_NULL, kw
    for kw in ("x", "a", "b", "c", "dy", "v_", "dx", "da", "db", "dc", "ws"):
        assert xbwd(p, **{kw: 0}) == E_NULL, kw
    # states and workspace: 16-byte aligned
    for kw in ("h0", "hl", "v_", "ws"):
        assert xfwd(p, **{kw: GB * 40 + 8}) == E_ALIGN, kw
    for kw in ("h0", "dhl", "dh0", "v_", "ws"):
        assert xbwd(p, **{kw: GB * 40 + 8}) == E_ALIGN, kw
    assert xfwd(p, x=X + 4) == E_ALIGN and xbwd(p, dx=DX + 2) == E_ALIGN
    # outputs and the workspace must not overlap inputs or each other
    assert xfwd(p, hl=H0) == E_ALIAS
    assert xfwd(p, ws=X) == E_ALIAS
    assert xfwd(p, ws=Y + 64) == E_ALIAS
    assert xfwd(p, hl=V) == E_ALIAS
    assert xbwd(p, dh0=H0) == E_ALIAS
    assert xbwd(p, dh0=DHL) == E_ALIAS
    assert xbwd(p, ws=V) == E_ALIAS
    assert xbwd(p, ws=DA) == E_ALIAS
    assert xbwd(p, dx=DH0) == E_ALIAS
    # nothing to do for an empty batch or head set, even with NULL pointers
    for kw in (dict(B=0), dict(H=0)):
        assert xfwd(problem(**kw), 0, 0, 0, 0, 0, 0, 0, 0, 0) == OK
        assert xbwd(problem(**kw), 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0) == OK


def nfwd(p, x=X, a=A, b=B_, c=C, h0=H0, y=Y, v_=V, hl=HL):
    v = ctypes.c_void_p
    return swr.load().swr_exact_forward_noalloc(ctypes.byref(p), v(x), v(a), v(b), v(c), v(h0), v(y),
                                                v(v_), v(hl), None)


def test_exact_forward_noalloc_validation():
    # validated as swr_exact_forward is, every check before any HIP runtime call
    p = problem()
    for kw in ("x", "a", "b", "c", "y"):
        assert nfwd(p, **{kw: 0}) == E_NULL, kw
    for kw in ("h0", "hl", "v_"):
        assert nfwd(p, **{kw: GB * 40 + 8}) == E_ALIGN, kw
    assert nfwd(p, x=X + 4) == E_ALIGN
    assert nfwd(p, hl=H0) == E_ALIAS and nfwd(p, hl=V) == E_ALIAS and nfwd(p, y=X) == E_ALIAS
    assert nfwd(problem(D=48)) == E_UNSUP and nfwd(problem(block=48)) == E_BLOCK
    # a problem whose workspace exceeds the static array is refused with its own code
    assert swr.SWR_NOALLOC_SCRATCH_BYTES == 32 << 20
    assert "#define SWR_NOALLOC_SCRATCH_BYTES ((int64_t)32 << 20)" in open(HEADER).read()
    # (65536 sequences: more than the array for the one pass and the three stages)
    big = problem(B=512, T=64, H=128, D=128, block=128)
    assert swr.swr_exact_workspace_bytes(big) > swr.SWR_NOALLOC_SCRATCH_BYTES
    assert nfwd(big) == E_SCRATCH
    # one that only the three stages fit is not refused (it then reaches the
    # HIP runtime, which this machine lacks)
    mid = problem(B=16, T=16384, H=16, D=128, block=128)
    assert swr.swr_exact_workspace_bytes(mid) > swr.SWR_NOALLOC_SCRATCH_BYTES
    if NO_GPU:
        assert nfwd(mid) in (OK, E_HIP)
    assert "SWR_NOALLOC_SCRATCH_BYTES" in swr.swr_error_string(E_SCRATCH)
    # the headline shape fits
    assert swr.swr_exact_workspace_bytes(problem(B=8, T=16384, H=16, D=128, block=128)) <= 32 << 20
    # nothing to do for an empty batch or head set, even with NULL pointers
    for kw in (dict(B=0), dict(H=0)):
        assert nfwd(problem(**kw), 0, 0, 0, 0, 0, 0, 0, 0) == OK


@reaches_launch
@pytest.mark.parametrize("B,T,H,D,block,dtype,per_channel", [
    (1, 978811, 16, 128, 64, BF16, True),     # 4 GB a tensor
    (4, 737280, 7, 64, 16, F32, True),
    (16, 583738, 2, 64, 32, BF16, True),
    (8, 587840, 16, 64, 64, F32, False),
    (4, 1 << 20, 33, 16, 64, BF16, True),
])
def test_noalloc_takes_long_sequences(B, T, H, D, block, dtype, per_channel):
    # the forward's runs alone (about 512 workgroups) decide what the static
    # array holds, however finely a long sequence's backward is split
    p = problem(B=B, T=T, H=H, D=D, block=block, dtype=dtype, per_channel=per_channel)
    far = [(1 << 44) + (i << 40) for i in range(8)]
    assert nfwd(p, *far) in (OK, E_HIP)


# ----------------------------------------------------------------------------- recurrent decoding

ST = GB * 30


def stp(p, t0=0, x=X, a=A, b=B_, c=C, y=Y, st=ST):
    v = ctypes.c_void_p
    return swr.load().swr_step(ctypes.byref(p), t0, v(x), v(a), v(b), v(c), v(y), v(st), None)


def xstp(p, x=X, a=A, b=B_, c=C, y=Y, st=ST):
    v = ctypes.c_void_p
    return swr.load().swr_exact_step(ctypes.byref(p), v(x), v(a), v(b), v(c), v(y), v(st), None)


def dstate(p, a=A, v_=V, st=ST):
    v = ctypes.c_void_p
    return swr.load().swr_decode_state(ctypes.byref(p), v(a), v(v_), v(st), None)


def test_step_validation():
    p = problem(T=1)
    assert stp(p, t0=-1) == E_SHAPE
    for kw in ("x", "a", "b", "c", "y", "st"):
        assert stp(p, **{kw: 0}) == E_NULL, kw
        assert xstp(p, **{kw: 0}) == E_NULL, kw
    assert stp(p, st=ST + 8) == E_ALIGN and xstp(p, st=ST + 4) == E_ALIGN
    assert stp(p, x=X + 2) == E_ALIGN
    # a per-channel decay needs the whole head's lane slices aligned (D = 128 bf16: 16 bytes)
    assert stp(problem(T=1, D=128, per_channel=True), a=A + 8) == E_ALIGN
    assert stp(p, y=X) == E_ALIAS and stp(p, st=A) == E_ALIAS and stp(p, st=Y) == E_ALIAS
    assert xstp(p, st=C) == E_ALIAS
    assert stp(problem(T=1, block=48)) == E_BLOCK
    # no token or no sequence: nothing to do, even with NULL pointers
    assert stp(problem(T=0), 5, 0, 0, 0, 0, 0, 0) == OK
    assert xstp(problem(B=0, T=1), 0, 0, 0, 0, 0, 0) == OK


def test_decode_state_validation():
    p = problem()
    assert dstate(p, st=0) == E_NULL and dstate(p, a=0) == E_NULL and dstate(p, v_=0) == E_NULL
    assert dstate(p, st=ST + 4) == E_ALIGN and dstate(p, v_=V + 4) == E_ALIGN
    assert dstate(problem(D=128, per_channel=True), a=A + 8) == E_ALIGN
    assert dstate(p, st=V) == E_ALIAS and dstate(p, st=A) == E_ALIAS
    assert dstate(problem(B=0)) == OK


def test_small_heads_are_packed_when_adjacent():
    # heads of 16 (32) channels stored next to each other run four (two) to a
    # 64-channel virtual head: the launch covers H / 4 (H / 2) heads
    p = problem(B=1, T=4096, H=8, D=16, block=16, run_len=256)
    info = swr.swr_launch_info(p)
    assert info["fwd_workgroups"] == (8 // 4 // 2) * (4096 // 256)   # 2 virtual heads, 2 per group
    assert info["bwd_workgroups"] == (8 // 4) * (4096 // 256)
    p = problem(B=1, T=4096, H=8, D=32, block=32, run_len=256)
    assert swr.swr_launch_info(p)["bwd_workgroups"] == (8 // 2) * (4096 // 256)
    # not adjacent ([B, H, T, D] storage) or a head count that does not divide: one at a time
    B, T, H, D = 1, 4096, 8, 16
    p = problem(B=B, T=T, H=H, D=D, block=16, run_len=256, x_strides=(H * T * D, D, T * D), a_strides=(H * T, 1, T))
    assert swr.swr_launch_info(p)["bwd_workgroups"] == 8 * (4096 // 256)
    p = problem(B=1, T=4096, H=6, D=16, block=16, run_len=256)
    assert swr.swr_launch_info(p)["bwd_workgroups"] == 6 * (4096 // 256)
    # the exact workspace covers either plan
    p = problem(B=2, T=1000, H=8, D=16, block=16)
    assert swr.swr_exact_workspace_bytes(p) > 0


# ---------------------------------------------------------------------------- uniform window


def ufwd(p, x=X, a=A, b=B_, c=C, y=Y):
    v = ctypes.c_void_p
    return swr.load().swr_uniform_forward(ctypes.byref(p), v(x), v(a), v(b), v(c), v(y), None)


def ubwd(p, x=X, a=A, b=B_, c=C, dy=DY, dx=DX, da=DA, db=DB, dc=DC):
    v = ctypes.c_void_p
    return swr.load().swr_uniform_backward(ctypes.byref(p), v(x), v(a), v(b), v(c), v(dy), v(dx),
                                           v(da), v(db), v(dc), None)


def test_uniform_validation():
    p = problem()
    assert ufwd(p, y=0) == E_NULL and ubwd(p, da=0) == E_NULL
    assert ufwd(problem(block=48)) == E_BLOCK and ubwd(problem(D=48)) == E_UNSUP
    assert ufwd(problem(per_channel=True)) == E_UNSUP and ubwd(problem(per_channel=True)) == E_UNSUP
    assert ufwd(p, y=X) == E_ALIAS and ubwd(p, db=DX) == E_ALIAS and ubwd(p, da=A) == E_ALIAS
    assert ufwd(p, c=C + 2) == E_ALIGN and ubwd(p, da=DA + 2) == E_ALIGN
    assert ufwd(problem(run_len=96)) == E_UNSUP
    # a 128-channel head runs as two 64-channel halves: 8-byte lane slices in bf16
    p128 = problem(D=128)
    assert ufwd(p128, x=X + 8) != E_ALIGN and ufwd(p128, x=X + 4) == E_ALIGN
    assert ufwd(problem(B=0)) == OK and ubwd(problem(T=0), x=0, dx=0) == OK


@pytest.mark.parametrize("block", [16, 32, 64, 128])
@pytest.mark.parametrize("H,D", [(3, 64), (4, 128), (16, 16)])
def test_uniform_launch_plan(block, H, D):
    B, T = 2, 4096
    info = swr.swr_uniform_launch_info(problem(B=B, T=T, H=H, D=D, block=block, run_len=512))
    hv = H * (2 if D > 64 else 1)
    groups = B * -(-hv // (128 // block))
    assert info["fwd_run_len"] == info["bwd_run_len"] == 512
    assert info["fwd_workgroups"] == info["bwd_workgroups"] == groups * (T // 512)
    auto = swr.swr_uniform_launch_info(problem(B=B, T=T, H=H, D=D, block=block))
    assert auto["fwd_run_len"] % block == 0 and auto["bwd_run_len"] % block == 0


# ---------------------------------------------------------------------------- shared gates


def gfwd(p, group, gst, x=X, a=A, b=B_, c=C, y=Y):
    v = ctypes.c_void_p
    g = None if gst is None else (ctypes.c_int64 * 3)(*gst)
    return swr.load().swr_forward_shared_gates(ctypes.byref(p), group, g, v(x), v(a), v(b), v(c), v(y),
                                               None, None)


def gbwd(p, group, gst, x=X, a=A, b=B_, c=C, dy=DY, v_=V, dx=DX, da=DA, db=DB, dc=DC, ws=GB * 20):
    v = ctypes.c_void_p
    g = None if gst is None else (ctypes.c_int64 * 3)(*gst)
    return swr.load().swr_backward_shared_gates(ctypes.byref(p), group, g, v(x), v(a), v(b), v(c), v(dy),
                                                v(v_), v(dx), v(da), v(db), v(dc), v(ws), None)


def test_shared_gates_validation():
    B, T, H, D = 2, 256, 4, 64
    p = problem(B=B, T=T, H=H, D=D)
    gst = (T * 2 * D, 2 * D, D)          # [B, T, 2 groups, D]
    assert gfwd(p, 3, gst) == E_SHAPE and gfwd(p, 0, gst) == E_SHAPE
    assert gfwd(p, 2, None) == E_NULL
    assert gfwd(problem(B=B, T=T, H=H, D=D, per_channel=True), 2, gst) == E_UNSUP
    assert gfwd(p, 2, (T * 2 * D, 2 * D, D - 4)) in (E_SHAPE, E_ALIGN)
    assert gfwd(p, 2, (T * 2 * D, 2 * D + 2, D)) == E_ALIGN       # 4-byte rows, 8-byte lane slices
    assert gfwd(p, 2, gst, b=B_ + 4) == E_ALIGN
    assert gfwd(p, 2, gst, y=B_) == E_ALIAS
    assert gbwd(p, 2, gst, dc=C) == E_ALIAS
    assert gfwd(problem(B=0), 2, gst) == OK and gbwd(problem(T=0), 2, None) == OK
    # groups of up to 16 heads are summed inside the backward: no workspace
    assert swr.swr_shared_gates_workspace_bytes(p, 2) == 0
    with pytest.raises(swr.SwrError):
        swr.swr_shared_gates_workspace_bytes(p, 3)
    # larger groups go through a float32 workspace of every head's shares
    H32 = 32
    p32 = problem(B=B, T=T, H=H32, D=D)
    g32 = (T * D, D, D)                  # [B, T, 1 group, D]
    assert swr.swr_shared_gates_workspace_bytes(p32, 32) == 2 * B * T * H32 * D * 4
    assert gbwd(p32, 32, g32, ws=0) == E_NULL
    assert gbwd(p32, 32, g32, db=GB * 20) == E_ALIAS        # db inside the workspace


def test_forward_pairs_bf16_heads_of_64():
    # the forward runs bf16 heads of 64 channels two at a time (16-byte lane
    # slices); the backward and float32 keep one head per kernel head
    p = problem(B=2, T=4096, H=8, D=64, block=128, run_len=1024)
    info = swr.swr_launch_info(p)
    assert info["fwd_workgroups"] == 2 * (8 // 2 // 2) * 4      # pairs, two per workgroup
    assert info["bwd_workgroups"] == 2 * 8 * 4
    p = problem(B=2, T=4096, H=8, D=64, block=128, run_len=1024, dtype=F32)
    assert swr.swr_launch_info(p)["fwd_workgroups"] == 2 * (8 // 2) * 4
    p = problem(B=2, T=4096, H=7, D=64, block=128, run_len=1024)   # odd H: no pairs
    assert swr.swr_launch_info(p)["fwd_workgroups"] == 2 * 7 * 4


# ---- the Python binding refuses host tensors (the kernels would dereference
# their host addresses on the GPU); checked before the library is called.

def test_binding_refuses_host_tensors():
    torch = pytest.importorskip("torch")
    x = torch.zeros(1, 64, 2, 16, dtype=torch.bfloat16)
    a = torch.zeros(1, 64, 2, dtype=torch.bfloat16)
    gates = torch.zeros(1, 64, 1, 16, dtype=torch.bfloat16)
    calls = [
        lambda: swr.swr_forward(x, a, x, x, 16),
        lambda: swr.swr_carriers(x, a, x, 16),
        lambda: swr.swr_backward(x, a, x, x, x, torch.zeros(1), 16),
        lambda: swr.swr_exact_forward(x, a, x, x, 16),
        lambda: swr.swr_exact_backward(x, a, x, x, x, torch.zeros(1), 16),
        lambda: swr.swr_step(x, a, x, x, 16, 0),
        lambda: swr.swr_exact_step(x, a, x, x),
        lambda: swr.swr_decode_state(x, a, torch.zeros(1), 16),
        lambda: swr.swr_uniform_forward(x, a, x, x, 16),
        lambda: swr.swr_uniform_backward(x, a, x, x, x, 16),
        lambda: swr.swr_forward_shared_gates(x, a, gates, gates, 16, 2),
        lambda: swr.swr_backward_shared_gates(x, a, gates, gates, x, torch.zeros(1), 16, 2),
    ]
    for call in calls:
        with pytest.raises(ValueError, match="GPU tensor"):
            call()
