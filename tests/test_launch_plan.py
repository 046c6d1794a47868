"""Launch plans (CPU only): every run length is a multiple of the sweep's step
that covers the sequence, a grid of a few rounds of resident workgroups never
starts another round, one plan of each kind is pinned by its numbers, and
packed heads stay within their bounds."""
import pytest

import paper_2512_13921_amd as swr


def _info(B, T, H, D, block, per_channel=False, uniform=False):
    p = swr.make_problem(B, T, H, D, block, swr.SWR_DTYPE_BF16, (T * H * D, H * D, D),
                         (T * H * D, H * D, D) if per_channel else (T * H, H, 1), per_channel=per_channel)
    return swr.swr_uniform_launch_info(p) if uniform else swr.swr_launch_info(p)


@pytest.mark.parametrize("T", [1, 16, 100, 128, 129, 1000, 4999, 61554])
@pytest.mark.parametrize("B,H", [(1, 1), (3, 7), (4, 7), (16, 32), (40, 64)])
@pytest.mark.parametrize("D,block,cap", [(128, 128, 256), (64, 128, 256), (64, 64, 512), (128, 16, 512), (48, 32, 512)])
def test_backward_plan(T, B, H, D, block, cap):
    i = _info(B, T, H, D, block)
    step = 128 if block == 128 else 64
    run, work = i["bwd_run_len"], i["bwd_workgroups"]
    runs = -(-T // run)
    assert run % step == 0 and work == B * H * runs
    assert run - step < T          # no run starts past the sequence
    units, nsteps = B * H, -(-T // step)
    rounds = -(-work // cap)
    if rounds <= 4 and units * T // 512 < 2 * cap:   # as many runs as these rounds hold
        assert run // step == -(-nsteps // min(nsteps, max(1, rounds * cap // units)))
    if units <= cap and T >= 64 * step * cap // units:
        assert work >= cap // 2    # a long sequence fills the machine


@pytest.mark.parametrize("B,H,T", [(4, 7, 61554), (3, 7, 49920), (1, 5, 112439), (2, 30, 8000)])
def test_uniform_backward_fits_one_round(B, H, T):
    i = _info(B, T, H, 64, 128, uniform=True)
    assert i["bwd_workgroups"] <= 256
    assert i["bwd_run_len"] % 128 == 0


# Packed small heads: a lane's 32-bit offsets add its head's share of a, da and
# the carriers.  Past 2^31 bytes the heads run one by one, whose bases are 64-bit.

def _packed(B, T, H, D, block, dtype=swr.SWR_DTYPE_BF16, sa_t=None, sa_h=None):
    sa_t = H if sa_t is None else sa_t
    sa_h = 1 if sa_h is None else sa_h
    p = swr.make_problem(B, T, H, D, block, dtype, (T * H * D, H * D, D), (max(T * sa_t, H * sa_h), sa_t, sa_h))
    i = swr.swr_launch_info(p)
    units = i["bwd_workgroups"] // -(-T // i["bwd_run_len"])
    assert units in (B * H, B * -(-H * D // 64))
    return units == B * -(-H * D // 64)


@pytest.mark.parametrize("H,D", [(3, 16), (4, 16), (7, 16), (3, 32), (2, 32)])
def test_packed_heads_bound_the_decays_offsets(H, D):
    lim, pack = 2 ** 31 - 1, 64 // D
    last = (lim - 64) // (4 * (pack - 1))               # 16 tokens of stride 1 and the last head's share
    assert _packed(2, 8192, H, D, 64, sa_t=1, sa_h=last)
    assert not _packed(2, 8192, H, D, 64, sa_t=1, sa_h=last + 1)
    assert not _packed(2, 8192, H, D, 64, sa_t=1, sa_h=2 ** 29)
    last = (lim - (pack - 1) * 4) // 64                 # rows of a far apart, heads next to each other
    assert _packed(1, 16384, H, D, 64, sa_t=last)
    if last + 1 <= lim // 64:                           # (else refused, as one head's offsets are)
        assert not _packed(1, 16384, H, D, 64, sa_t=last + 1)


@pytest.mark.parametrize("H,D,block", [(3, 16, 16), (4, 16, 128), (5, 32, 32), (2, 32, 64)])
def test_packed_heads_bound_the_carriers_offsets(H, D, block):
    blocks = (2 ** 31 - 1) // 256                       # 64 channels of float32 a block
    assert _packed(1, blocks * block - 1, H, D, block)
    assert not _packed(1, (blocks + 1) * block, H, D, block)


@pytest.mark.parametrize("B,T,H,D,block,dtype,per_channel", [
    (64, 1670942336, 12, 16, 64, swr.SWR_DTYPE_BF16, False),
    (64, 686221184, 33, 32, 64, swr.SWR_DTYPE_F32, True),
    (64, 78976637, 128, 112, 32, swr.SWR_DTYPE_BF16, True),
])
def test_short_runs_of_very_long_sequences_fit_a_launch(B, T, H, D, block, dtype, per_channel):
    # runs of 256 tokens would make more workgroups than a launch takes
    xs = (T * H * D, D, T * D)
    p = swr.make_problem(B, T, H, D, block, dtype, xs, xs if per_channel else (T * H, 1, T), per_channel=per_channel)
    plans = [swr.swr_launch_info(p)] if per_channel else [swr.swr_launch_info(p), swr.swr_uniform_launch_info(p)]
    for i in plans:
        assert 0 < i["fwd_workgroups"] < 2 ** 31 and 0 < i["bwd_workgroups"] < 2 ** 31
    if D != 112:
        assert swr.swr_exact_workspace_bytes(p) > 0


@pytest.mark.parametrize("D,block,sigmoid,packed", [(32, 64, True, False), (32, 128, True, True), (32, 64, False, True),
                                                    (16, 64, True, True)])
def test_odd_counts_with_sigmoids(D, block, sigmoid, packed):
    B, T, H = 2, 8192, 3
    p = swr.make_problem(B, T, H, D, block, swr.SWR_DTYPE_BF16, (T * H * D, H * D, D), (T * H, H, 1),
                         sigmoid_decay=sigmoid)
    i = swr.swr_launch_info(p)
    assert i["bwd_workgroups"] // -(-T // i["bwd_run_len"]) == (B * -(-H * D // 64) if packed else B * H)


@pytest.mark.parametrize("T,packed", [(10922, False), (10923, True)])
def test_odd_counts_in_the_forward_of_long_blocks(T, packed):
    i = swr.swr_launch_info(swr.make_problem(2, T, 3, 16, 128, swr.SWR_DTYPE_BF16, (T * 48, 48, 16), (T * 3, 3, 1)))
    assert i["fwd_workgroups"] // -(-T // i["fwd_run_len"]) == (2 if packed else 6)


@pytest.mark.parametrize("B,T,H,D,block,dtype,per_channel,sigmoid,run,work", [
    (8, 16384, 16, 128, 128, "bf16", False, False, 8192, 256),   # 8 waves: one round of 256
    (3, 20000, 7, 64, 128, "bf16", False, False, 1792, 252),     # ... never just past one
    (8, 4096, 16, 128, 64, "bf16", False, False, 512, 1024),     # 4 waves: runs of 512, whole rounds of 512
    (1, 16384, 4, 64, 64, "bf16", False, False, 128, 512),       # too short for these: one round
    (2, 8192, 33, 64, 64, "f32", False, False, 128, 4224),       # float32 lanes of 4: a grid of at most 8192
    (2, 8192, 33, 64, 64, "bf16", False, True, 128, 4224),       # and bf16 with the sigmoids
    (2, 8192, 33, 64, 64, "bf16", False, False, 576, 990),       # ... without: about 512, whole rounds
    (4, 8192, 16, 32, 64, "bf16", True, False, 64, 8192),        # a decay per channel, 2 channels a lane
    (1, 16384, 128, 16, 16, "bf16", False, False, 384, 1376),    # packed heads: runs of about 256
])
def test_pinned_backward_plans(B, T, H, D, block, dtype, per_channel, sigmoid, run, work):
    xs = (T * H * D, H * D, D)
    p = swr.make_problem(B, T, H, D, block, swr.SWR_DTYPE_BF16 if dtype == "bf16" else swr.SWR_DTYPE_F32, xs,
                         xs if per_channel else (T * H, H, 1), per_channel=per_channel, sigmoid_decay=sigmoid)
    i = swr.swr_launch_info(p)
    assert (i["bwd_run_len"], i["bwd_workgroups"]) == (run, work)
