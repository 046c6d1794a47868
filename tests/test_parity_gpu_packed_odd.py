"""GPU parity of packed small heads where the head count does not fill the last
64-channel virtual head (its other lanes idle): every path against the oracle,
and nothing written past the real heads' outputs."""
import numpy as np
import pytest

import oracle
import workloads as W
from parity import assert_close, check_full, run_gpu, to_device, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # (B, T, H, D, block, dtype)
    (2, 2500, 7, 16, 16, "bf16"),      # 35000 tokens of heads: padded
    (1, 1000, 33, 16, 128, "bf16"),
    (9, 2000, 2, 16, 64, "bf16"),
    (3, 5461, 2, 16, 64, "f32"),       # 32766: the last that stays unpadded
    (2, 8192, 2, 16, 64, "f32"),       # 32768: the forward alone
    (3, 3700, 3, 32, 32, "bf16"),
    (2, 3300, 5, 32, 128, "f32"),
    (2, 300, 7, 16, 16, "bf16"),
]


@pytest.fixture(scope="module")
def swr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_13921_amd as lib
    lib.load()
    return lib


@pytest.mark.parametrize("B,T,H,D,block,dtype", CASES)
@pytest.mark.parametrize("carriers", [True, False])
def test_odd_head_counts(swr, B, T, H, D, block, dtype, carriers):
    prob = W.random_problem(181 + T + H, B, T, H, D, block, dtype, "sigmoid", 2.0)
    y, grads = run_gpu(swr, prob, residual=True, carriers=carriers)
    check_full(prob, y, grads, residual=True, what=f"packed odd {B}x{T}x{H}x{D} l{block} {dtype}")


def test_odd_head_counts_featurised(swr):
    prob = W.random_problem(182, 2, 3300, 5, 16, 32, "bf16", "sigmoid", 3.0, logits=True)
    feat = dict(sigmoid_decay=True, sigmoid_pregate=True)
    y, grads = run_gpu(swr, prob, **feat)
    check_full(prob, y, grads, what="packed odd sigmoid", **feat)


def _guarded(shape, dtype=torch.float32):
    """A tensor of this shape inside a larger one, and the values around it."""
    n = int(np.prod(shape))
    buf = torch.full((n + 2048,), 7.0, dtype=dtype, device="cuda")
    return buf[1024:1024 + n].view(shape), (buf[:1024], buf[1024 + n:])


@pytest.mark.parametrize("B,T,H,D,block,dtype", CASES)
def test_exact_odd_head_counts(swr, B, T, H, D, block, dtype):
    prob = W.random_problem(183 + T + H, B, T, H, D, block, dtype, "sigmoid", 3.0)
    x, a, b, c, dy = (to_device(getattr(prob, n), dtype) for n in ("x", "a", "b", "c", "dy"))
    rng = np.random.default_rng(T)
    h0, dhl = (rng.standard_normal((B, H, D)).astype(np.float32) for _ in range(2))
    h0d, dhld = torch.from_numpy(h0).cuda(), torch.from_numpy(dhl).cuda()
    y, gy = _guarded((B, T, H, D), x.dtype)
    v, gv = _guarded((B, H, -(-T // block), D))
    hl, gh = _guarded((B, H, D))
    outs, guards = zip(*(_guarded(s, d) for s, d in (((B, T, H, D), x.dtype), ((B, T, H), torch.float32),
                                                     ((B, T, H, D), x.dtype), ((B, T, H, D), x.dtype))))
    swr.swr_exact_forward(x, a, b, c, block, h0=h0d, y=y, carriers=v, h_last=hl)
    *_, dh0 = swr.swr_exact_backward(x, a, b, c, dy, v, block, h0=h0d, dh_last=dhld, outputs=outs, want_dh0=True)
    torch.cuda.synchronize()
    for g in (gy, gv, gh) + guards:
        assert all(bool((t == 7.0).all()) for t in g)
    ref_y, ref_hl = oracle.exact_forward(prob.x, prob.a, prob.b, prob.c, h0)
    refs = oracle.exact_backward(prob.x, prob.a, prob.b, prob.c, prob.dy, h0, dhl)
    assert_close(to_host(y), ref_y, dtype, "y")
    assert_close(to_host(hl), ref_hl, dtype, "h_last")
    for name, got, ref in zip(("dx", "da", "db", "dc", "dh0"), tuple(outs) + (dh0,), refs):
        assert_close(to_host(got), ref, dtype, name)


@pytest.mark.parametrize("B,T,H,D,block,dtype", CASES)
def test_odd_head_counts_write_only_their_outputs(swr, B, T, H, D, block, dtype):
    prob = W.random_problem(184 + T + H, B, T, H, D, block, dtype, "sigmoid", 2.0)
    x, a, b, c, dy = (to_device(getattr(prob, n), dtype) for n in ("x", "a", "b", "c", "dy"))
    y, gy = _guarded((B, T, H, D), x.dtype)
    v, gv = _guarded((B, H, -(-T // block), D))
    outs, guards = zip(*(_guarded(s, d) for s, d in (((B, T, H, D), x.dtype), ((B, T, H), torch.float32),
                                                     ((B, T, H, D), x.dtype), ((B, T, H, D), x.dtype))))
    swr.swr_forward(x, a, b, c, block, y=y, carriers=v)
    swr.swr_backward(x, a, b, c, dy, v, block, outputs=outs)
    torch.cuda.synchronize()
    for g in (gy, gv) + guards:
        assert all(bool((t == 7.0).all()) for t in g)
    check_full(prob, y, outs, what="packed odd guarded")


def _strided_like(t, strides, dtype=None):
    """t's values in memory of these strides."""
    r = torch.empty_strided(t.shape, strides, dtype=dtype or t.dtype, device=t.device)
    return r.copy_(t)


@pytest.mark.parametrize("H,D,log2_stride", [(3, 16, 28), (3, 16, 29), (4, 16, 28), (2, 32, 30)])
def test_decays_of_far_apart_heads(swr, H, D, log2_stride):
    # a's and da's heads lie 2^31 bytes and more from the first: past a lane's 32-bit offset
    B, T, block = 2, 8192, 64
    prob = W.random_problem(185 + H, B, T, H, D, block, "bf16", "sigmoid", 3.0)
    x, a, b, c, dy = (to_device(getattr(prob, n), "bf16") for n in ("x", "a", "b", "c", "dy"))
    far = (T, 1, 1 << log2_stride)
    a = _strided_like(a, far)
    y, v = swr.swr_forward(x, a, b, c, block, save_carriers=True)
    outs = [torch.empty_like(x), torch.empty_strided((B, T, H), far, dtype=torch.float32, device="cuda"),
            torch.empty_like(x), torch.empty_like(x)]
    outs[1].fill_(float("nan"))
    for carriers in (v, None):
        grads = swr.swr_backward(x, a, b, c, dy, carriers, block, outputs=outs)
        torch.cuda.synchronize()
        check_full(prob, y, grads, what=f"far heads {H}x{D} 2^{log2_stride}")
    ye, ve, hl = swr.swr_exact_forward(x, a, b, c, block, save_carriers=True, want_h_last=True)
    grads = swr.swr_exact_backward(x, a, b, c, dy, ve, block, outputs=outs)
    torch.cuda.synchronize()
    ref_y, ref_hl = oracle.exact_forward(prob.x, prob.a, prob.b, prob.c)
    assert_close(to_host(ye), ref_y, "bf16", "y")
    assert_close(to_host(hl), ref_hl, "bf16", "h_last")
    for name, got, ref in zip(("dx", "da", "db", "dc"), grads, oracle.exact_backward(prob.x, prob.a, prob.b, prob.c,
                                                                                    prob.dy)):
        assert_close(to_host(got), ref, "bf16", name)


def _form(t, form):
    """t's values in another storage that the calls accept: heads-first, rows
    longer than their heads, or aligned for one head's lanes but not the packed
    ones' (heads of D channels: D / 16 elements off)."""
    if form == "heads first":
        return _strided_like(t, (t.stride(0), 1, t.shape[1]) if t.dim() == 3 else t.stride())
    if form == "long rows":
        w = t.stride(1)
        return _strided_like(t, (t.shape[1] * (w + 64), w + 64) + t.stride()[2:])
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
    r = buf[t.shape[3] // 16 if t.dim() == 4 else 1:][:t.numel()].view(t.shape)
    return r.copy_(t)


@pytest.mark.parametrize("B,T,H,D,block", [(2, 2500, 7, 16, 16), (3, 3700, 3, 32, 32), (1, 11000, 7, 16, 128)])
@pytest.mark.parametrize("form", ["heads first", "long rows", "misaligned"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_odd_head_counts_in_other_storage(swr, B, T, H, D, block, form, dtype):
    # (heads first: of a and da alone; misaligned: the heads run one by one)
    prob = W.random_problem(186 + T + H, B, T, H, D, block, dtype, "sigmoid", 3.0)
    x, a, b, c, dy = (_form(to_device(getattr(prob, n), dtype), form) for n in ("x", "a", "b", "c", "dy"))
    y, v = swr.swr_forward(x, a, b, c, block, save_carriers=True)
    for carriers in (v, None):
        grads = swr.swr_backward(x, a, b, c, dy, carriers, block)
        torch.cuda.synchronize()
        assert grads[1].stride() == a.stride()
        check_full(prob, y, grads, what=f"odd {form} {dtype}")
    ye, ve, hl = swr.swr_exact_forward(x, a, b, c, block, save_carriers=True, want_h_last=True)
    grads = swr.swr_exact_backward(x, a, b, c, dy, ve, block)
    torch.cuda.synchronize()
    ref_y, ref_hl = oracle.exact_forward(prob.x, prob.a, prob.b, prob.c)
    assert_close(to_host(ye), ref_y, dtype, "y")
    assert_close(to_host(hl), ref_hl, dtype, "h_last")
    for name, got, ref in zip(("dx", "da", "db", "dc"), grads, oracle.exact_backward(prob.x, prob.a, prob.b, prob.c,
                                                                                    prob.dy)):
        assert_close(to_host(got), ref, dtype, name)
