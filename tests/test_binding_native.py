"""The binding's native marshalling against its Python path: the same results
on ordinary calls, and every call that Python refuses still refused by it."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture()
def swr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_13921_amd as lib
    lib.load()
    return lib


class _Nothing:
    """A native module that handles no call."""
    def __getattr__(self, name):
        return lambda *args: None


def _inputs(dtype, per_channel=False, layout="bthd", B=2, T=150, H=4, D=64):
    g = torch.Generator(device="cuda").manual_seed(3)
    def t(*shape):
        r = torch.randn(shape, generator=g, device="cuda").to(dtype)
        return r.transpose(1, 2).contiguous().transpose(1, 2) if layout == "bhtd" else r
    x, b, c, dy = (t(B, T, H, D) for _ in range(4))
    a = torch.sigmoid(t(B, T, H, D) if per_channel else t(B, T, H))
    return x, a, b, c, dy, t(B, T, H // 2, D), t(B, T, H // 2, D)


def _calls(swr, x, a, b, c, dy, gb, gc):
    h = torch.randn(x.shape[0], x.shape[2], x.shape[3], device="cuda")
    y, v = swr.swr_forward(x, a, b, c, 32, residual=True, save_carriers=True)
    yield y, v
    yield swr.swr_forward(x, a, b, c, 32, sigmoid_decay=True, sigmoid_pregate=True)
    yield swr.swr_backward(x, a, b, c, dy, v, 32)
    yield swr.swr_backward(x, a, b, c, dy, None, 32, run_len=128)
    h.fill_(0.5)
    ye, ve, hl = swr.swr_exact_forward(x, a, b, c, 32, h0=h, save_carriers=True, want_h_last=True)
    yield ye, ve, hl
    yield swr.swr_exact_forward(x, a, b, c, 32)
    yield swr.swr_exact_backward(x, a, b, c, dy, ve, 32, h0=h, dh_last=h, want_dh0=True)
    yield swr.swr_exact_backward(x, a, b, c, dy, ve, 32)
    st = swr.swr_decode_state(x, a, v, 32)
    yield st.clone()
    yield swr.swr_step(x[:, :2], a[:, :2], b[:, :2], c[:, :2], 32, 7, st)
    yield swr.swr_exact_step(x[:, :2], a[:, :2], b[:, :2], c[:, :2], h)
    if a.dim() == 3:
        yield swr.swr_uniform_forward(x, a, b, c, 32)
        yield swr.swr_uniform_backward(x, a, b, c, dy, 32, residual=True)
        yg, vg = swr.swr_forward_shared_gates(x, a, gb, gc, 32, 2, save_carriers=True)
        yield yg, vg
        yield swr.swr_forward_shared_gates(x, a, gb, gc, 32, 2)
        yield swr.swr_backward_shared_gates(x, a, gb, gc, dy, vg, 32, 2)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("per_channel,layout", [(False, "bthd"), (True, "bthd"), (False, "bhtd")])
def test_native_and_python_paths_agree(swr, monkeypatch, dtype, per_channel, layout):
    inputs = _inputs(dtype, per_channel, layout)
    native = list(_calls(swr, *inputs))
    monkeypatch.setattr(swr, "_native", (swr._lib, _Nothing()))
    python = list(_calls(swr, *inputs))
    torch.cuda.synchronize()
    assert len(native) == len(python)
    for i, (u, w) in enumerate(zip(native, python)):
        u, w = (r if isinstance(r, tuple) else (r,) for r in (u, w))
        assert len(u) == len(w), i
        for p, q in zip(u, w):
            assert p.dtype == q.dtype and p.stride() == q.stride() and torch.equal(p, q), i


def test_refusals_are_the_python_path_s(swr):
    x, a, b, c, dy, gb, gc = _inputs(torch.bfloat16)
    half = x.half()
    with pytest.raises(ValueError, match="share shape, dtype and strides"):
        swr.swr_forward(x, a, b, c.transpose(1, 2).contiguous().transpose(1, 2), 32)
    with pytest.raises(ValueError, match="share shape, dtype and strides"):
        swr.swr_forward(x, a, b.float(), c, 32)
    with pytest.raises(TypeError, match="a must have the dtype of x"):
        swr.swr_forward(x, a.float(), b, c, 32)
    with pytest.raises(TypeError, match="unsupported dtype torch.float16"):
        swr.swr_forward(half, half[..., 0].contiguous(), half, half, 32)
    with pytest.raises(ValueError, match="x must be"):
        swr.swr_forward(x[0], a, b, c, 32)
    with pytest.raises(ValueError, match="a must be .B, T, H."):
        swr.swr_forward(x, a[:, :5], b, c, 32)
    with pytest.raises(ValueError, match="carriers must be"):
        swr.swr_backward(x, a, b, c, dy, torch.zeros(1, device="cuda"), 32)
    with pytest.raises(ValueError, match="needs the exact forward"):
        swr.swr_exact_backward(x, a, b, c, dy, None, 32)
    with pytest.raises(ValueError, match="h0 must be"):
        swr.swr_exact_forward(x, a, b, c, 32, h0=torch.zeros(3, device="cuda"))
    with pytest.raises(ValueError, match="state must be"):
        swr.swr_step(x, a, b, c, 32, 0, torch.zeros(3, device="cuda"))
    with pytest.raises(ValueError, match="group must divide"):
        swr.swr_forward_shared_gates(x, a, gb, gc, 32, 3)
    with pytest.raises(ValueError, match="shared gates must be"):
        swr.swr_forward_shared_gates(x, a, b, c, 32, 2)
    for call in (lambda: swr.swr_forward(x, a, b, c, 48), lambda: swr.swr_forward(x, a, b, c, 32, run_len=7),
                 lambda: swr.swr_step(x, a, b, c, 32, -1, torch.zeros(2, 4, 2, 64, device="cuda")),
                 lambda: swr.swr_forward(x, a, b, c, 32, y=x), lambda: swr.swr_uniform_forward(x, a, b, c, 8)):
        with pytest.raises(swr.SwrError):
            call()
    torch.cuda.synchronize()


def test_stream_argument_and_current_stream(swr):
    x, a, b, c, dy, _, _ = _inputs(torch.bfloat16)
    ref = swr.swr_forward(x, a, b, c, 32)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    y1 = swr.swr_forward(x, a, b, c, 32, stream=s)
    with torch.cuda.stream(s):
        y2 = swr.swr_forward(x, a, b, c, 32)
    torch.cuda.synchronize()
    assert torch.equal(y1, ref) and torch.equal(y2, ref)


def _workspace_calls(swr):
    """The calls that allocate a workspace of their own, as functions of the stream."""
    x, a, b, c, dy, _, _ = _inputs(torch.bfloat16, T=700, H=32)
    gb, gc = b[:, :, :1].contiguous(), c[:, :, :1].contiguous()   # one gate for 32 heads: summed in a workspace
    _, ve = swr.swr_exact_forward(x, a, b, c, 32, save_carriers=True)
    _, vg = swr.swr_forward_shared_gates(x, a, gb, gc, 32, 32, save_carriers=True)
    return (lambda s: swr.swr_exact_forward(x, a, b, c, 32, save_carriers=True, want_h_last=True, stream=s),
            lambda s: swr.swr_exact_backward(x, a, b, c, dy, ve, 32, want_dh0=True, stream=s),
            lambda s: swr.swr_backward_shared_gates(x, a, gb, gc, dy, vg, 32, 32, stream=s))


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("call", range(3))
def test_a_call_s_own_workspace_is_its_stream_s(swr, monkeypatch, native, call):
    # The caller never sees the workspace, so nothing it does can keep the next
    # allocation off it: it has to be memory of the stream the kernels run on.
    if not native:
        monkeypatch.setattr(swr, "_native", (swr._lib, _Nothing()))
    run = _workspace_calls(swr)[call]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    s = torch.cuda.Stream()
    before = {m["address"] for m in torch.cuda.memory_snapshot()}
    run(s)
    torch.cuda.synchronize()
    assert any(m["stream"] == s.cuda_stream and m["address"] not in before for m in torch.cuda.memory_snapshot())


@pytest.mark.parametrize("native", [True, False])
def test_calls_on_another_stream_among_allocations_here(swr, monkeypatch, native):
    if not native:
        monkeypatch.setattr(swr, "_native", (swr._lib, _Nothing()))
    calls = _workspace_calls(swr)
    refs = [run(None) for run in calls]
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    for run, ref in zip(calls, refs):
        with torch.cuda.stream(s):
            torch.cuda._sleep(20_000_000)
        outs = run(s)
        filled = [torch.full((n,), float("nan"), device="cuda") for n in (1 << 10, 1 << 14, 1 << 18, 1 << 20, 1 << 22)]
        torch.cuda.synchronize()
        for u, w in zip(outs, ref):
            assert torch.equal(u, w)
        del filled


def test_a_state_of_zeros_is_filled_on_the_call_s_stream(swr):
    # the current stream is still busy when the step on another stream reads its state
    x, a, b, c, *_ = _inputs(torch.bfloat16, T=2)
    steps = (lambda s: swr.swr_step(x, a, b, c, 32, 0, stream=s), lambda s: swr.swr_exact_step(x, a, b, c, stream=s))
    for step in steps:
        y, st = step(None)
        torch.cuda.synchronize()
        unlike = torch.full_like(st, 7.0)   # what the next state's memory holds
        torch.cuda.synchronize()
        del unlike
        s = torch.cuda.Stream()
        torch.cuda._sleep(200_000_000)
        y2, st2 = step(s)
        with torch.cuda.stream(s):
            same = torch.equal(y2, y) and torch.equal(st2, st)
        torch.cuda.synchronize()
        assert same
