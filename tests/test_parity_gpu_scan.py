"""GPU parity of the exact recurrence's carrier scan over the runs at the edges
of its split into segments: one batch of loads for all runs, fewer runs than
segments, one batch of loads a segment, and segments of several batches
(run_len forces short runs; packed heads of 16 channels run the three stages in
both directions)."""
import numpy as np
import pytest

import oracle
import workloads as W
from parity import assert_close, to_device, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("runs", [1, 2, 7, 8, 9, 15, 17, 127, 128, 129, 511, 513, 1100])
@pytest.mark.parametrize("per_channel", [False, True])
def test_scan_over_runs(runs, per_channel):
    import paper_2512_13921_amd as swr
    # (the per-channel forward runs in one pass: its backward is the scan's)
    B, H, D, l = 2, 4, 16, 16
    T = 64 * runs - 5
    prob = W.random_problem(70 + runs, B, T, H, D, l, "f32", "exp_softplus", per_channel=per_channel)
    x, a, b, c, dy = (to_device(getattr(prob, n), "f32") for n in ("x", "a", "b", "c", "dy"))
    rng = np.random.default_rng(runs)
    h0, dhl = (rng.standard_normal((B, H, D)).astype(np.float32) for _ in range(2))
    h0d, dhld = torch.from_numpy(h0).cuda(), torch.from_numpy(dhl).cuda()
    y, v, hl = swr.swr_exact_forward(x, a, b, c, l, h0=h0d, save_carriers=True, want_h_last=True, run_len=64)
    grads = swr.swr_exact_backward(x, a, b, c, dy, v, l, h0=h0d, dh_last=dhld, want_dh0=True, run_len=64)
    torch.cuda.synchronize()
    ref_y, ref_hl = oracle.exact_forward(prob.x, prob.a, prob.b, prob.c, h0)
    refs = oracle.exact_backward(prob.x, prob.a, prob.b, prob.c, prob.dy, h0, dhl)
    assert_close(to_host(y), ref_y, "f32", f"{runs} runs: y")
    assert_close(to_host(hl), ref_hl, "f32", f"{runs} runs: h_last")
    for name, got, ref in zip(("dx", "da", "db", "dc", "dh0"), grads, refs):
        assert_close(to_host(got), ref, "f32", f"{runs} runs: {name}")


@pytest.mark.parametrize("runs", [128, 1100])
@pytest.mark.parametrize("per_channel", [False, True])
def test_segments_whose_product_overflows_from_a_zero_state(runs, per_channel):
    # 1.2^64 a run: from 7 runs on a product passes float32's range, while the
    # states that it multiplies are zero and every result is finite
    import paper_2512_13921_amd as swr
    B, H, D, l, T = 2, 4, 16, 16, 64 * runs
    prob = W.random_problem(90 + runs, B, T, H, D, l, "f32", "sigmoid", 2.0, per_channel=per_channel)
    prob.a[:, 200:T - 200] = np.float32(1.2)
    prob.x[:, :T - 200] = 0
    prob.dy[:, 200:] = 0
    x, a, b, c, dy = (to_device(getattr(prob, n), "f32") for n in ("x", "a", "b", "c", "dy"))
    ref_y, ref_hl = oracle.exact_forward(prob.x, prob.a, prob.b, prob.c)
    hs, _ = oracle.exact_forward(prob.x, prob.a, prob.b, np.ones_like(prob.c))
    v = torch.from_numpy(hs[:, l - 1::l].transpose(0, 2, 1, 3).astype(np.float32)).cuda().contiguous()
    grads = swr.swr_exact_backward(x, a, b, c, dy, v, l, want_dh0=True, run_len=64)
    torch.cuda.synchronize()
    refs = oracle.exact_backward(prob.x, prob.a, prob.b, prob.c, prob.dy)
    for name, got, ref in zip(("dx", "da", "db", "dc", "dh0"), grads, refs):
        assert_close(to_host(got), ref, "f32", name)
    if per_channel:   # (whose forward runs in one pass, without the scan)
        return
    y, hl = swr.swr_exact_forward(x, a, b, c, l, want_h_last=True, run_len=64)
    torch.cuda.synchronize()
    assert_close(to_host(y), ref_y, "f32", "y")
    assert_close(to_host(hl), ref_hl, "f32", "h_last")


def test_segments_whose_product_overflows_from_a_small_state():
    # a state of 1e-30 grows by 1.25^512 = 4e49 over one segment of 8 runs (packed
    # heads of 16, three stages both ways), backward from the other end alike
    import paper_2512_13921_amd as swr
    B, H, D, l, T = 1, 4, 16, 16, 64 * 128
    prob = W.random_problem(91, B, T, H, D, l, "f32", "sigmoid", 2.0)
    prob.a[:, :512] = prob.a[:, T - 512:] = np.float32(1.25)
    prob.x[:], prob.dy[:] = 0, 0
    state = np.full((B, H, D), 1e-30, np.float32)
    x, a, b, c, dy = (to_device(getattr(prob, n), "f32") for n in ("x", "a", "b", "c", "dy"))
    st = torch.from_numpy(state).cuda()
    _, v = swr.swr_exact_forward(x, a, b, c, l, h0=st, save_carriers=True, run_len=64)
    dx, *_ = swr.swr_exact_backward(x, a, b, c, dy, v, l, h0=st, dh_last=st, run_len=64)
    torch.cuda.synchronize()
    # h after token 511, and the adjoint of token T - 513: each of the 512
    # products rounds by 2^-24 at most, which makes 3.1e-5
    ref = float(state[0, 0, 0]) * 1.25 ** 512
    for got in (to_host(v)[:, :, 511 // l], to_host(dx)[:, T - 513] / prob.b[:, T - 513]):
        assert np.all(np.abs(got / ref - 1) < 4e-5)
