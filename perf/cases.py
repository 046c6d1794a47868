"""Performance cases of the Sliding Window Recurrence library.

Each case is one unit of work that a user of the library has it do, called
through the Python binding (``paper_2512_13921_amd``):

* ``train``: a training step's two calls, ``swr_forward`` with the block
  carriers saved and ``swr_backward`` with them (or, with ``carriers`` false,
  a forward that saves nothing and a backward that recomputes them);
* ``layer``: the same through the autograd function, with the Phalanx layer's
  featurisation (sigmoid of the decay and pre-gate logits) and residual;
* ``prefill``: inference over a prompt, the forward and the decoding state;
* ``generate``: a prompt, then tokens decoded one at a time;
* ``exact``: forward and backward of the untruncated recurrence from an
  initial state, with the final state and its gradient;
* ``uniform``: forward and backward of the uniform window;
* ``gates``: forward and backward with the gates shared by groups of heads.
"""
import math

import torch

import paper_2512_13921_amd as swr

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(kind, B, T, H, D, block, dtype="bf16", decay="head", name=None, **more):
    case = {"kind": kind, "B": B, "T": T, "H": H, "D": D, "block": block, "dtype": dtype,
            "decay": decay, **more}
    return case if name is None else {"name": name, **case}


def listed():
    return [
        # The smallest call: a unit test's or a debugging run's float32 layer.
        # Launch latency and host time count, not bytes.
        _case("train", 1, 1024, 4, 64, 64, "f32", name="train_tiny_f32", recipe="sigmoid2"),
        # Serving: a short prompt for a batch of 8, then 16 tokens one by one.
        _case("generate", 8, 1024, 16, 128, 128, name="generate_16", recipe="exp", new=16),
        # The Phalanx layer in a training step of ordinary size, through autograd.
        _case("layer", 8, 4096, 16, 128, 64, name="layer_T4096", recipe="sigmoid3", residual=True),
        # The benchmark's shape: a large training step, one decay per head.
        _case("train", 8, 16384, 16, 128, 128, name="train_T16384", recipe="exp"),
        # Long-context inference: one sequence of 131072 tokens.
        _case("prefill", 1, 131072, 32, 64, 128, name="prefill_T131072", recipe="exp"),
        # A model of width 2048 with 32 heads of 64, batch 16.
        _case("train", 16, 8192, 32, 64, 64, name="train_width2048", recipe="sigmoid5"),
        # The paper's own mixer: 128 heads of 16 channels, block 16.
        _case("train", 1, 16384, 128, 16, 16, name="train_paper_mixer", recipe="sigmoid3", residual=True),
        # A full diagonal: one decay per token, head and channel.
        _case("train", 4, 8192, 16, 128, 128, decay="channel", name="train_per_channel", recipe="exp"),
        # The untruncated recurrence that the window approximates.
        _case("exact", 8, 16384, 16, 128, 128, name="exact_T16384", recipe="exp"),
        # The paper's other truncation, at an ordinary size.
        _case("uniform", 8, 4096, 16, 128, 64, name="uniform_T4096", recipe="sigmoid3"),
        # Gates shared by groups of 4 heads, as grouped-query attention shares keys.
        _case("gates", 16, 8192, 32, 64, 64, name="gates_width2048", recipe="sigmoid5", group=4),
        # An odd shape: odd head count and length, a head width that is no power
        # of two, heads-first storage, float32, nothing saved but the inputs.
        _case("train", 3, 5003, 5, 96, 32, "f32", name="train_ragged_f32", recipe="sigmoid3",
              layout="bhtd", carriers=False),
    ]


def draw(rng):
    kind = rng.choice(("train", "train", "layer", "prefill", "generate", "exact", "exact", "uniform", "gates"))
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    natural = (16, 32, 64, 128)
    any_width = (16, 32, 48, 64, 80, 96, 112, 128, 128, 256)
    D = rng.choice(any_width if kind in ("train", "layer") else natural)
    H = rng.choice((1, 2, 3, 4, 5, 7, 8, 12, 16, 16, 24, 32, 32) if D >= 64 else (4, 7, 8, 16, 33, 64, 128))
    block = rng.choice((16, 32, 64, 128))
    more = {"recipe": rng.choice(("exp", "sigmoid2", "sigmoid3", "sigmoid5"))}
    decay = "head"
    if kind in ("train", "exact") and rng.random() < 0.25:
        decay = "channel"
    if kind == "gates":
        H = rng.choice((2, 4, 8, 12, 16, 32))
        more["group"] = rng.choice([g for g in (1, 2, 4, 8) if H % g == 0])
    if kind == "train":
        more["carriers"] = rng.random() < 0.75
    if kind in ("train", "layer", "uniform"):
        more["residual"] = rng.random() < 0.5
    if kind in ("train", "exact", "uniform", "gates") and rng.random() < 0.25:
        more["layout"] = "bhtd"
    # Elements of one [B, T, H, D] tensor, spread over their logarithm up to a
    # share of the largest listed case's 2^28.
    top = 24 if kind == "generate" else 26 if dtype == "f32" or decay == "channel" else 27
    n = 2.0 ** rng.uniform(17, top)
    B = min(rng.choice((1, 1, 2, 3, 4, 8, 16)), max(1, int(n / (64 * H * D))))
    T = min(262144, max(17, int(n / (B * H * D))))
    if rng.random() < 0.5:   # half of them whole multiples of 64, the others as they fall
        T = max(64, T // 64 * 64)
    if kind == "generate":
        more["new"] = rng.choice((1, 4, 16, 32))
    return _case(kind, B, T, H, D, block, dtype, decay, **more)


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, case):
    """Standard normals of shape [B, T, H, .], stored in the case's layout."""
    dt = _DTYPES[case["dtype"]]
    if case.get("layout") == "bhtd":
        B, T, H, D = shape
        return torch.randn((B, H, T, D), generator=g, dtype=dt, device="cuda").transpose(1, 2)
    return torch.randn(shape, generator=g, dtype=dt, device="cuda")


def _decay(g, shape, case):
    """Decays (or, for the layer, their logits) by the workloads' recipes."""
    z = torch.randn(shape, generator=g, dtype=torch.float32, device="cuda")
    if case["recipe"] == "exp":
        delta = torch.rand(shape, generator=g, dtype=torch.float32, device="cuda") * 0.099 + 1e-3
        a = torch.exp(-torch.nn.functional.softplus(z) * delta)
        if case["kind"] == "layer":
            a = z + 3.0
    else:
        z = z + float(case["recipe"][len("sigmoid"):])
        a = z if case["kind"] == "layer" else torch.sigmoid(z)
    a = a.to(_DTYPES[case["dtype"]])
    if case.get("layout") == "bhtd":   # a has x's order of dimensions in memory
        a = a.transpose(1, 2).contiguous().transpose(1, 2)
    return a


def prepare(case, seed):
    g = _generator(seed)
    B, T, H, D = case["B"], case["T"], case["H"], case["D"]
    T += case.get("new", 0)
    G = H // case.get("group", 1)
    s = {"case": case,
         "x": _normal(g, (B, T, H, D), case),
         "b": _normal(g, (B, T, G, D), case),
         "c": _normal(g, (B, T, G, D), case),
         "a": _decay(g, (B, T, H, D) if case["decay"] == "channel" else (B, T, H), case)}
    if case["kind"] not in ("prefill", "generate"):
        s["dy"] = _normal(g, (B, T, H, D), case)
    if case["kind"] == "exact":
        s["h0"] = torch.randn((B, H, D), generator=g, dtype=torch.float32, device="cuda")
        s["dh_last"] = torch.randn((B, H, D), generator=g, dtype=torch.float32, device="cuda")
    if case["kind"] == "layer":
        for n in ("x", "a", "b", "c"):
            s[n].requires_grad_(True)
    return s


# ----------------------------------------------------------------------------
# One pass
# ----------------------------------------------------------------------------


def run(state):
    case = state["case"]
    kind, block = case["kind"], case["block"]
    x, a, b, c = state["x"], state["a"], state["b"], state["c"]
    residual = case.get("residual", False)
    if kind == "train":
        if case.get("carriers", True):
            y, v = swr.swr_forward(x, a, b, c, block, residual, save_carriers=True)
        else:
            y, v = swr.swr_forward(x, a, b, c, block, residual), None
        dx, da, db, dc = swr.swr_backward(x, a, b, c, state["dy"], v, block, residual)
        out = {"y": y, "dx": dx, "da": da, "db": db, "dc": dc}
        return out if v is None else {**out, "v": v}
    if kind == "layer":
        y = swr.SWRFunction.apply(x, a, b, c, block, residual, True, True)
        dx, da, db, dc = torch.autograd.grad(y, (x, a, b, c), state["dy"])
        return {"y": y.detach(), "dx": dx, "da": da, "db": db, "dc": dc}
    if kind == "prefill":
        y, v = swr.swr_forward(x, a, b, c, block, save_carriers=True)
        return {"y": y, "state": swr.swr_decode_state(x, a, v, block)}
    if kind == "generate":
        T, new = case["T"], case["new"]
        xp, ap, bp, cp = (t[:, :T] for t in (x, a, b, c))
        y, v = swr.swr_forward(xp, ap, bp, cp, block, save_carriers=True)
        st = swr.swr_decode_state(xp, ap, v, block)
        tokens = []
        for t in range(T, T + new):
            yt, st = swr.swr_step(x[:, t:t + 1], a[:, t:t + 1], b[:, t:t + 1], c[:, t:t + 1], block, t, st)
            tokens.append(yt)
        return {"y": y, "state": st, "tokens": tokens}
    if kind == "exact":
        y, v, h_last = swr.swr_exact_forward(x, a, b, c, block, h0=state["h0"], save_carriers=True,
                                             want_h_last=True)
        dx, da, db, dc, dh0 = swr.swr_exact_backward(x, a, b, c, state["dy"], v, block, h0=state["h0"],
                                                     dh_last=state["dh_last"], want_dh0=True)
        return {"y": y, "v": v, "h_last": h_last, "dx": dx, "da": da, "db": db, "dc": dc, "dh0": dh0}
    if kind == "uniform":
        y = swr.swr_uniform_forward(x, a, b, c, block, residual)
        dx, da, db, dc = swr.swr_uniform_backward(x, a, b, c, state["dy"], block, residual)
        return {"y": y, "dx": dx, "da": da, "db": db, "dc": dc}
    if kind == "gates":
        group = case["group"]
        y, v = swr.swr_forward_shared_gates(x, a, b, c, block, group, save_carriers=True)
        dx, da, db, dc = swr.swr_backward_shared_gates(x, a, b, c, state["dy"], v, block, group)
        return {"y": y, "v": v, "dx": dx, "da": da, "db": db, "dc": dc}
    raise ValueError(f"unknown kind {kind!r}")


# ----------------------------------------------------------------------------
# Work, tolerance and the values in 64 bits
# ----------------------------------------------------------------------------


def work(case):
    """Bytes and operations of one pass: every call's inputs read once and its
    outputs written once (the forward and the backward are two calls, with
    the loss between them, so each reads x, a, b and c)."""
    kind = case["kind"]
    es = 2 if case["dtype"] == "bf16" else 4
    B, T, H, D = case["B"], case["T"], case["H"], case["D"]
    rows = B * T * H
    n, ng = rows * D, rows * D // case.get("group", 1)
    na = n if case["decay"] == "channel" else rows
    v = B * H * math.ceil(T / case["block"]) * D * 4
    if kind == "uniform" or not case.get("carriers", True):
        v = 0
    st = B * H * D * 4
    fwd = (2 * n + 2 * ng + na) * es + v
    bwd = (3 * n + 4 * ng + na) * es + na * (es if kind == "layer" else 4) + v
    # multiply-adds per element: pre-gate, recurrence and read-out; the
    # backward recomputes the states and runs the adjoint recurrence, the
    # four gradients on top.  The uniform window runs each over two blocks.
    f, w = 4 * n, 14 * n
    if kind == "prefill":
        return {"bytes": fwd + 2 * st + v // max(1, math.ceil(T / case["block"])), "flops": f}
    if kind == "generate":
        k = case["new"]
        token = (4 * D + 1) * B * H * es + 4 * st   # a step reads and writes its two states
        return {"bytes": fwd + 4 * st + k * token, "flops": f + 6 * k * B * H * D}
    if kind == "exact":
        return {"bytes": fwd + bwd + 5 * st, "flops": f + w}
    if kind == "uniform":
        return {"bytes": fwd + bwd, "flops": 2 * (f + w)}
    return {"bytes": fwd + bwd, "flops": f + w}


def tolerance(case):
    # About four times what the calls differ from the 64-bit values by: bf16
    # outputs are rounded once (2^-9 of a value at most, 1.7e-3 in the 2-norm);
    # float32 outputs carry the rounding of float32 sums over two blocks or,
    # exact, over the decay's memory.
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 2e-6, "max": 4e-5}


def _blocks(t, l, fill):
    """[B, T, H, .] -> l tensors [B, nb, H, .], the tokens at each offset of their block."""
    B, T = t.shape[:2]
    nb = -(-T // l)
    if nb * l != T:
        pad = torch.full((B, nb * l - T) + t.shape[2:], fill, dtype=t.dtype, device=t.device)
        t = torch.cat((t, pad), 1)
    return t.reshape((B, nb, l) + t.shape[2:]).unbind(2)


def _unblocks(ts, T):
    t = torch.stack(ts, 2)
    return t.reshape((t.shape[0], -1) + t.shape[3:])[:, :T]


def _shift(v, first=None):
    first = torch.zeros_like(v[:, :1]) if first is None else first
    return torch.cat((first, v[:, :-1]), 1)


def _states(kind, a, u, l, h0=None):
    """The states h [B, T, H, D], and the local end states of the blocks."""
    T = u.shape[1]
    A, U = _blocks(a, l, 1.0), _blocks(u, l, 0.0)
    w, ws = torch.zeros_like(U[0]), []
    for p in range(l):
        w = A[p] * w + U[p]
        if kind == "uniform":
            ws.append(w)
    v = w
    if kind == "uniform":   # plus the tail of the previous block that the window still holds
        tails, S, R = [None] * l, torch.zeros_like(v), torch.ones_like(A[0])
        for p in reversed(range(l)):
            tails[p] = S
            S = S + R * U[p]
            R = R * A[p]
        g, hs = torch.ones_like(A[0]), []
        for p in range(l):
            g = g * A[p]
            hs.append(ws[p] + g * _shift(tails[p]))
        return _unblocks(hs, T), v
    if kind == "exact":     # the carrier recurrence over the blocks
        P = A[0]
        for p in range(1, l):
            P = P * A[p]
        h, entering = h0, []
        for t in range(v.shape[1]):
            entering.append(h)
            h = P[:, t] * h + v[:, t]
        e = torch.stack(entering, 1)
    else:                   # the jagged window: the previous block's local end state
        e = _shift(v)
    hs = []
    for p in range(l):
        e = A[p] * e + U[p]
        hs.append(e)
    return _unblocks(hs, T), v


def exact(case, seed):
    s = prepare(case, seed)
    kind, l, T = case["kind"], case["block"], s["x"].shape[1]
    grads = "dy" in s
    x, a, b, c = (s[n].detach().double().requires_grad_(grads) for n in ("x", "a", "b", "c"))
    av, bv, cv = (torch.sigmoid(a), torch.sigmoid(b), c) if kind == "layer" else (a, b, c)
    if av.dim() == 3:
        av = av.unsqueeze(-1)
    if kind == "gates":
        bv, cv = (t.repeat_interleave(case["group"], 2) for t in (bv, cv))
    h0 = s["h0"].double().requires_grad_(True) if kind == "exact" else None
    h, v = _states(kind, av, bv * x, 128 if kind == "exact" else l, h0)
    y = cv * h
    if case.get("residual", False):
        y = y + x
    if kind in ("prefill", "generate"):
        n = case["T"]
        nb = -(-n // l)
        hp, vp = (h, v) if n == T else _states(kind, av[:, :n], (bv * x)[:, :n], l)
        last = torch.stack((hp[:, -1], vp[:, nb - 1]), 2)   # (e, s) after the prompt
        if kind == "prefill":
            return {"y": y, "state": last}
        # the state after the last token; a block that is complete has not yet
        # been exchanged for the next one
        at = -(-T // l) - 1
        return {"y": y[:, :n], "state": torch.stack((h[:, -1], v[:, at]), 2),
                "tokens": [y[:, t:t + 1] for t in range(n, T)]}
    loss = (y * s["dy"].double()).sum()
    if kind != "exact":
        dx, da, db, dc = torch.autograd.grad(loss, (x, a, b, c))
        out = {"y": y, "dx": dx, "da": da, "db": db, "dc": dc}
        if kind == "gates" or (kind == "train" and case.get("carriers", True)):
            out["v"] = v.transpose(1, 2)
        return {n: t.detach() for n, t in out.items()}
    loss = loss + (h[:, -1] * s["dh_last"].double()).sum()
    dx, da, db, dc, dh0 = torch.autograd.grad(loss, (x, a, b, c, h0))
    ends = [min(T, (t + 1) * l) - 1 for t in range(-(-T // l))]
    out = {"y": y, "v": h[:, ends].transpose(1, 2), "h_last": h[:, -1],
           "dx": dx, "da": da, "db": db, "dc": dc, "dh0": dh0}
    return {n: t.detach() for n, t in out.items()}
