"""GPU parity of swr_decode_state at the edges of its token split: last blocks
of 1 to 128 tokens (one token a lane, or 32 rows a pass), both decay modes."""
import pytest

import oracle
import workloads as W
from parity import assert_close, to_device, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("last", [1, 31, 33, 63, 64, 65, 127, 128])
@pytest.mark.parametrize("D,dtype,per_channel,logits", [(128, "bf16", False, False), (16, "f32", True, False),
                                                        (64, "bf16", True, True), (32, "f32", False, True)])
def test_decode_state_last_block_lengths(last, D, dtype, per_channel, logits):
    import paper_2512_13921_amd as swr
    prob = W.random_problem(900 + last, 1, 128 + last, 5, D, 128, dtype, "sigmoid", 3.0, with_dy=False,
                            per_channel=per_channel, logits=logits)
    x, a, b, c = (to_device(getattr(prob, n), dtype) for n in "xabc")
    _, v = swr.swr_forward(x, a, b, c, 128, save_carriers=True, sigmoid_decay=logits)
    st = swr.swr_decode_state(x, a, v, 128, sigmoid_decay=logits)
    torch.cuda.synchronize()
    _, ref = oracle.step(prob.x, prob.a, prob.b, prob.c, None, 0, 128, sigmoid_decay=logits)
    assert_close(to_host(st), ref, dtype, f"decode state, last block of {last}")


def test_decode_state_of_more_sequences_than_a_grid_of_waves():
    # 2^26 waves would be 2^32 threads, more than a launch takes
    import paper_2512_13921_amd as swr
    B, H, D = 4099, 16384, 16
    x = torch.empty((B, 1, H, D), dtype=torch.bfloat16, device="cuda")
    a = torch.full((B, 1, H), 0.5, dtype=torch.bfloat16, device="cuda")
    v = torch.rand((B, H, 1, D), device="cuda")
    st = swr.swr_decode_state(x, a, v, 16)
    torch.cuda.synchronize()
    # one token: both states are the first block's carrier
    assert torch.equal(st[:, :, 0], v[:, :, 0]) and torch.equal(st[:, :, 1], v[:, :, 0])
