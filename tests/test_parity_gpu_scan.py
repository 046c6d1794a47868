"""GPU parity of the exact recurrence's carrier scan over the runs at the edges
of its split into segments: fewer runs than segments, one batch of loads a
segment, and segments of several batches (run_len forces short runs; packed
heads of 16 channels run the three stages in both directions)."""
import numpy as np
import pytest

import oracle
import workloads as W
from parity import assert_close, to_device, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("runs", [1, 2, 15, 17, 127, 128, 129, 511, 513, 1100])
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
