"""Row lengths other than the binding's: the ABI asks for rows of a multiple of
16 bytes, and a saved state may be of any such length."""
import pytest

from tests.gpu_harness import Pair, log

pytestmark = pytest.mark.gpu


def least_ld(P, dtype):
    per16 = 8 if dtype == "bf16" else 4
    return (P + per16 - 1) // per16 * per16


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_whole_buffers_of_the_least_row_length_are_restored(dtype):
    """A state saved as whole [n, ld] buffers goes back into a context of that
    row length, and the run goes on as one that was never stopped."""
    import torch

    log("case whole buffers restored %s" % dtype)
    n, P = 8, 20_001
    ld = least_ld(P, dtype)
    full = Pair(n, P, "two_peer", dtype, precisions=("f32",))
    for t in range(2):
        full.local_step()
        full.gossip_round(t)
    saved = {}
    for k in ("x", "y", "m", "v", "u", "zp"):
        saved[k] = torch.zeros((n, ld), dtype=full.gpu.bufs[k].dtype, device="cuda")
        saved[k][:, :P].copy_(full.gpu.bufs[k][:, :P])
    counters, step = full.gpu.counters(), full.step
    resumed = Pair(n, P, "two_peer", dtype, precisions=(), ld=saved["x"].shape[1])
    resumed.oracles = {}  # compared with `full`
    resumed.grads = torch.empty_like(full.grads)  # the seeded gradients go by the whole buffer
    for k, v in saved.items():
        resumed.gpu.bufs[k].copy_(v)
    resumed.gpu.set_counters(*counters)
    resumed.step = step
    for t in range(2, 4):
        for run in (full, resumed):
            run.local_step()
            run.gossip_round(t)
    for k in ("x", "m", "v", "u", "zp"):
        assert torch.equal(full.gpu.bufs[k][:, :P], resumed.gpu.bufs[k][:, :P]), k
    assert full.gpu.consensus_error() == resumed.gpu.consensus_error()
