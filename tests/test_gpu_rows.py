"""Row lengths other than the binding's: the ABI asks for rows of a multiple of
16 bytes, and a saved state may be of any such length."""
import numpy as np
import pytest

from tests.gpu_harness import Pair, log, reduction_close

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


LEAST = [
    # n, P, graph, form, dtype, gamma, fused
    (4, 1_000, "ring", "eq", "f32", 0.1, True),  # rows without padding, 4000 bytes each
    (7, 1_000, "exponential", "eq", "bf16", 0.1, False),  # without padding, 2000 bytes
    (16, 4_099, "two_peer", "alg1", "bf16", 0.0, True),
    (24, 777, "one_peer", "eq", "bf16", 0.2, True),
    (33, 516, "complete", "dadam", "f32", 0.0, False),  # without padding, two whole tiles and 4 columns
    (40, 1_032, "random_regular", "local_dadam", "bf16", 0.0, False),  # without padding
    (64, 260, "complete", "eq", "f32", 0.1, True),  # without padding
]


@pytest.mark.parametrize("n,P,graph,form,dtype,gamma,fused", LEAST)
def test_rows_of_the_least_length(n, P, graph, form, dtype, gamma, fused):
    """Local steps, rounds and reductions on rows that are aligned to 16 bytes
    only and follow one another without a gap or with the least one: every
    stored value is the oracle's, so nothing runs over into the next worker."""
    import torch

    log("case least rows n=%d P=%d %s %s %s" % (n, P, graph, form, dtype))
    pair = Pair(n, P, graph, dtype, gamma=gamma, form=form, precisions=("f32",), ld=least_ld(P, dtype))
    assert pair.gpu.ld == least_ld(P, dtype)
    some = (np.arange(n) % 3 != 1).astype(np.uint8)
    o = pair.oracles["f32"]
    mean = torch.empty(pair.gpu.ld, dtype=pair.gpu.x.dtype, device="cuda")
    for t in range(3):
        pair.local_step(some if t == 1 else None)
        if fused:
            pair.local_step_gossip_round(t, some)
        else:
            pair.check_state(names=("m", "v"), y_rows=np.flatnonzero(some), tag="before round %d" % t)
            pair.gossip_round(t)
        reduction_close(pair.gpu.consensus_error(), o.consensus_error(), "round %d" % t)
    pair.check_state(tag="least rows")  # asserts identical bits
    for a, b in ((0, P), (1, P - 1), (P // 2 + 1, P // 2 + 8)):
        reduction_close(pair.gpu.consensus_error_cols(a, b), o.consensus_error(slice(a, b)), "cols [%d,%d)" % (a, b))
    pair.gpu.replica_mean(mean)
    got = mean[:P].view(torch.int16 if dtype == "bf16" else torch.int32).cpu().numpy()
    assert np.array_equal(got, np.asarray(o.replica_mean()).view(got.dtype))
