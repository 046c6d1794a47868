"""GPU parity of the exact recurrence on both sides of the sizes where its
schedule changes: a single run (up to 128 tokens), the three stages (long
chains or many chunks of few bytes), the one-pass chains; and the count of
look-back waits that gave up, which reads zero whichever schedule ran."""
import numpy as np
import pytest

import oracle
import workloads as W
from parity import assert_close, to_device, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # (B, T, H, D, block, dtype, per_channel)
    (1, 1, 3, 64, 64, "bf16", False),        # a single run, down to one token
    (2, 127, 3, 128, 16, "bf16", False),
    (2, 128, 2, 64, 128, "f32", False),
    (1, 100, 5, 32, 32, "f32", True),
    (2, 128, 8, 16, 64, "bf16", False),      # ... of packed heads
    (1, 128, 2, 128, 64, "bf16", True),      # ... of 64-channel halves
    (1, 64, 3, 128, 32, "f32", False),       # float32 heads of 128: a single run forward up to 64 tokens
    (1, 65, 3, 128, 32, "f32", False),       # and a chain of one chunk from there on
    (1, 129, 2, 64, 128, "bf16", False),     # pairs at l = 128: one pass up to 10 chunks
    (1, 129, 2, 64, 32, "bf16", False),      # three-stage forward, one-pass backward
    (1, 1280, 2, 64, 128, "bf16", False),    # 10 chunks
    (1, 1281, 2, 64, 128, "bf16", False),    # 11 chunks: three stages
    (1, 4096, 2, 64, 64, "bf16", False),     # the backward's last chain of 32 chunks
    (1, 4097, 2, 64, 64, "bf16", False),     # and its first 33 chunks in three stages
    (2, 8192, 3, 64, 128, "f32", False),     # float32: 64 chunks, 12.6 MB (backward one-pass)
    (1, 8100, 3, 64, 16, "f32", False),      # float32: 64 chunks, three stages
    (1, 8000, 3, 64, 16, "f32", False),      # float32: 63 chunks, one pass
    (1, 8100, 3, 128, 16, "f32", False),     # float32 heads of 128: one pass at any length
    (1, 8000, 3, 128, 16, "f32", False),
    (1, 50000, 4, 128, 128, "bf16", False),  # a row of 1024 bytes: three stages, over 24 MB
    (1, 50000, 6, 64, 128, "bf16", False),   # a row of 768 bytes: pairs would chain
    (1, 33000, 3, 128, 64, "f32", False),    # over 24 MB and 1024 bytes: one pass
    (1, 6017, 6, 128, 64, "bf16", False),    # a row of 1536 bytes, 48 chunks: three stages
    (1, 6016, 6, 128, 64, "bf16", False),    # 47 chunks: one pass
    (1, 6017, 7, 128, 64, "bf16", False),    # a longer row: one pass
    (1, 600, 32, 64, 64, "bf16", False),     # pairs, a row of 4096 bytes, few bytes: three stages
    (1, 600, 34, 64, 64, "bf16", False),     # of more: one pass past 512 tokens
    (2, 512, 32, 64, 64, "bf16", False),     # (three stages up to there, to 8192 bytes)
    (1, 513, 48, 64, 64, "bf16", False),
    (1, 1281, 5, 64, 32, "bf16", False),     # heads of 64 of an odd count: 11 chunks, three stages
    (1, 1280, 5, 64, 32, "bf16", False),     # 10 chunks, one pass
    (1, 400, 121, 64, 16, "bf16", False),    # 484 chunks in all, three stages
    (1, 400, 119, 64, 16, "bf16", False),    # 476 chunks, one pass
    (1, 950, 33, 32, 64, "bf16", False),     # heads of 32 one at a time: 264 chunks, three stages
    (1, 950, 31, 32, 64, "bf16", False),     # 248 chunks, one pass
]


@pytest.mark.parametrize("B,T,H,D,block,dtype,per_channel", CASES)
@pytest.mark.parametrize("states", [False, True])
def test_exact_schedules(B, T, H, D, block, dtype, per_channel, states):
    import paper_2512_13921_amd as swr
    prob = W.random_problem(T + D, B, T, H, D, block, dtype, "sigmoid", 3.0, per_channel=per_channel)
    x, a, b, c, dy = (to_device(getattr(prob, n), dtype) for n in ("x", "a", "b", "c", "dy"))
    rng = np.random.default_rng(T)
    h0, dhl = (rng.standard_normal((B, H, D)).astype(np.float32) if states else None for _ in range(2))
    dev = lambda t: None if t is None else torch.from_numpy(t).cuda()
    p = swr.make_problem(B, T, H, D, block, 1 if dtype == "bf16" else 0, x.stride()[:3],
                         x.stride()[:3] if per_channel else a.stride(), per_channel=per_channel)
    ws = torch.full((swr.swr_exact_workspace_bytes(p) // 4,), float("nan"), device="cuda")
    count = lambda: int(ws.view(torch.int32)[1].item())
    y, v, hl = swr.swr_exact_forward(x, a, b, c, block, h0=dev(h0), save_carriers=True, want_h_last=True,
                                     workspace=ws)
    torch.cuda.synchronize()
    if not per_channel and not (D <= 32 and H % (64 // D) == 0):   # (packed heads never chain)
        assert count() == 0
    grads = swr.swr_exact_backward(x, a, b, c, dy, v, block, h0=dev(h0), dh_last=dev(dhl), want_dh0=True,
                                   workspace=ws)
    torch.cuda.synchronize()
    if not per_channel and D == 64:
        assert count() == 0
    ref_y, ref_hl = oracle.exact_forward(prob.x, prob.a, prob.b, prob.c, h0)
    refs = oracle.exact_backward(prob.x, prob.a, prob.b, prob.c, prob.dy, h0, dhl)
    assert_close(to_host(y), ref_y, dtype, "y")
    assert_close(to_host(hl), ref_hl, dtype, "h_last")
    ends = [min(T, (t + 1) * block) - 1 for t in range(-(-T // block))]
    if T <= 8192:
        hs, _ = oracle.exact_forward(prob.x, prob.a, prob.b, np.ones_like(prob.c), h0)
        assert_close(to_host(v), hs[:, ends].transpose(0, 2, 1, 3), dtype, "carriers")
    for name, got, ref in zip(("dx", "da", "db", "dc", "dh0"), grads, refs):
        assert_close(to_host(got), ref, dtype, name)


FORMS = [
    # (B, T, H, D, block, dtype, per_channel)
    (2, 100, 6, 64, 64, "bf16", False),      # a single run
    (1, 128, 3, 128, 128, "f32", True),      # ... of 64-channel halves
    (2, 77, 8, 16, 16, "bf16", False),       # ... of packed heads (stored heads first: one at a time)
    (1, 4999, 6, 64, 16, "bf16", False),     # three stages of pairs
    (2, 1500, 5, 128, 128, "bf16", False),   # one pass
    (1, 3000, 3, 32, 32, "bf16", True),      # one pass, three stages back
]


@pytest.mark.parametrize("B,T,H,D,block,dtype,per_channel", FORMS)
@pytest.mark.parametrize("form", ["logits", "heads first", "long rows"])
def test_exact_schedules_in_other_forms(B, T, H, D, block, dtype, per_channel, form):
    import paper_2512_13921_amd as swr
    logits = form == "logits"
    prob = W.random_problem(T + D + 1, B, T, H, D, block, dtype, "sigmoid", 3.0, per_channel=per_channel, logits=logits)
    feat = dict(sigmoid_decay=logits, sigmoid_pregate=logits)

    def dev(n):
        t = to_device(getattr(prob, n), dtype)
        if form == "heads first":
            return t.transpose(1, 2).contiguous().transpose(1, 2)
        if form == "long rows":
            w = t.stride(1)
            return torch.empty_strided(t.shape, (T * (w + 64), w + 64) + t.stride()[2:], dtype=t.dtype,
                                       device="cuda").copy_(t)
        return t

    x, a, b, c, dy = (dev(n) for n in ("x", "a", "b", "c", "dy"))
    rng = np.random.default_rng(T)
    h0, dhl = (rng.standard_normal((B, H, D)).astype(np.float32) for _ in range(2))
    h0d, dhld = torch.from_numpy(h0).cuda(), torch.from_numpy(dhl).cuda()
    y, v, hl = swr.swr_exact_forward(x, a, b, c, block, h0=h0d, residual=True, save_carriers=True, want_h_last=True,
                                     **feat)
    grads = swr.swr_exact_backward(x, a, b, c, dy, v, block, h0=h0d, dh_last=dhld, residual=True, want_dh0=True, **feat)
    torch.cuda.synchronize()
    ref_y, ref_hl = oracle.exact_forward(prob.x, prob.a, prob.b, prob.c, h0, residual=True, **feat)
    refs = oracle.exact_backward(prob.x, prob.a, prob.b, prob.c, prob.dy, h0, dhl, residual=True, **feat)
    assert_close(to_host(y), ref_y, dtype, "y")
    assert_close(to_host(hl), ref_hl, dtype, "h_last")
    for name, got, ref in zip(("dx", "da", "db", "dc", "dh0"), grads, refs):
        assert_close(to_host(got), ref, dtype, name)


def test_time_out_path_of_the_chains(monkeypatch):
    # Both one-pass schedules (paired-head forward, backward) at a size that
    # chains, with the poll limit forced to 0 from the host: the kernels end,
    # every finite output is the normal call's, a count comes with NaNs.
    import paper_2512_13921_amd as swr
    prob = W.random_problem(17, 1, 64 * 128, 64, 64, 128, "bf16", "sigmoid", 3.0)
    x, a, b, c, dy = (to_device(getattr(prob, n), "bf16") for n in ("x", "a", "b", "c", "dy"))
    ws = torch.zeros(16 << 20, dtype=torch.int32, device="cuda")

    def both(v=None):
        y, v_, hl = swr.swr_exact_forward(x, a, b, c, 128, save_carriers=True, want_h_last=True, workspace=ws)
        torch.cuda.synchronize()
        n = int(ws[1].item())
        g = swr.swr_exact_backward(x, a, b, c, dy, v_ if v is None else v, 128, workspace=ws)
        torch.cuda.synchronize()
        return (y, v_, hl), n, g, int(ws[1].item())

    ref_f, n0, ref_b, n1 = both()
    assert n0 == 0 and n1 == 0
    monkeypatch.setenv("SWR_CHAIN_SPIN_LIMIT", "0")
    got_f, nf, got_b, nb = both(ref_f[1])
    monkeypatch.delenv("SWR_CHAIN_SPIN_LIMIT")
    for got, ref, n in ((got_f, ref_f, nf), (got_b, ref_b, nb)):
        for u, w in zip(got, ref):
            fin = torch.isfinite(u)
            assert torch.equal(u[fin], w[fin])
            assert n > 0 or bool(fin.all())
        assert n == 0 or not bool(torch.isfinite(got[0]).all())
    again_f, n0, again_b, n1 = both()
    assert n0 == 0 and n1 == 0
    for u, w in zip(again_f + tuple(again_b), ref_f + tuple(ref_b)):
        assert torch.equal(u, w)
