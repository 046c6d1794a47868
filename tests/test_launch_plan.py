"""Launch plans of the backward sweeps (CPU only): every run length is a
multiple of the sweep's step that covers the sequence, and a grid of a few
rounds of resident workgroups never starts another round."""
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
