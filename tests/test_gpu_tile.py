"""The tile round kernel against the planned one (both are the same arithmetic
in the same order per element, so every stored value is bit-identical; the two
statistics are fp64 sums in another order, so they agree to far less than an
fp32 rounding).  Sizes sit at the edges of a tile (256 columns) and of the
workers per wave (1, 2, 4 or 8, by n and by the number of tiles)."""
import os

import numpy as np
import pytest

import gasloc_inputs as gi

pytestmark = pytest.mark.gpu

EDGES = [
    # n, P, graph, form, dtype, gamma, fused
    (1, 255, "ring", "eq", "f32", 0.1, True),
    (2, 257, "one_peer", "alg1", "bf16", 0.0, True),
    (15, 1, "exponential", "eq", "bf16", 0.1, False),
    (16, 256, "two_peer", "local_dadam", "f32", 0.0, False),
    (17, 511, "complete", "eq", "f32", 0.1, True),
    (32, 513, "random_regular", "alg1", "f32", 0.0, False),
    (33, 1023, "complete", "dadam", "bf16", 0.0, False),
    (63, 259, "exponential", "eq", "f32", 0.0, True),
    (64, 1025, "complete", "alg1", "bf16", 0.0, True),
    (64, 254, "one_peer", "local_dadam", "bf16", 0.0, False),
]
MANY_TILES = 64 * 256 * 256 + 3  # past the line at 64 tiles per CU, with a ragged last tile
LARGE = [
    (5, "ring", "eq", "bf16", 0.1, True),
    (16, "complete", "eq", "f32", 0.1, True),
    (17, "two_peer", "alg1", "bf16", 0.0, True),
    (32, "exponential", "local_dadam", "f32", 0.0, False),
    (33, "complete", "dadam", "f32", 0.0, False),
    (61, "two_peer", "eq", "bf16", 0.1, True),
]


def _rounds(kernel, n, P, graph, form, dtype, gamma, fused, rounds=2, mu=gi.OUTER_MOMENTUM):
    import torch

    import paper_2606_11081_amd as g

    before = os.environ.pop("GASLOC_GOSSIP_KERNEL", None)
    try:
        if kernel:
            os.environ["GASLOC_GOSSIP_KERNEL"] = kernel
        run = g.GASLoC(n, P, topology=graph, seed=5, degree=4, param_dtype=dtype, outer_lr=gi.OUTER_LR,
                       outer_momentum=mu, consensus_momentum=gamma, round_form=form)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(n + P)
        run.x.normal_(0.0, 0.02, generator=gen)
        grads = torch.empty((n, run.ld), dtype=torch.float32, device="cuda").normal_(0.0, 1.0, generator=gen)
        some = (np.arange(n) % 3 != 1).astype(np.uint8)  # heterogeneous local steps
        stats = []
        for t in range(rounds):
            run.local_step(grads, gi.LOCAL_LR, some if t % 2 == 0 else 1 - some)
            if fused:
                run.local_step_gossip_round(grads, gi.LOCAL_LR, t, some)
            else:
                run.gossip_round(t)
            stats += [run.consensus_error(), run.pseudo_gradient_sq()]
        out = {k: run.bufs[k][:, :P].clone() for k in ("x", "m", "v", "u", "zp") if run.bufs[k] is not None}
        run.close()
        return out, np.array(stats)
    finally:
        os.environ.pop("GASLOC_GOSSIP_KERNEL", None)
        if before is not None:
            os.environ["GASLOC_GOSSIP_KERNEL"] = before


def _compare(n, P, *case, **options):
    import torch

    a, sa = _rounds(None, n, P, *case, **options)
    b, sb = _rounds("planned", n, P, *case, **options)
    for k in a:
        view = torch.int16 if a[k].dtype == torch.bfloat16 else torch.int32
        assert torch.equal(a[k].contiguous().view(view), b[k].contiguous().view(view)), k
    # n P fp64 terms, all non-negative up to a cancellation of at most log2(n + 1) bits
    np.testing.assert_allclose(sa, sb, rtol=n * P * 2.0 ** -52)


@pytest.mark.parametrize("n,P,graph,form,dtype,gamma,fused", EDGES)
def test_tile_edges(n, P, graph, form, dtype, gamma, fused):
    print("case tile edges n=%d P=%d %s %s %s" % (n, P, graph, form, dtype), flush=True)
    _compare(n, P, graph, form, dtype, gamma, fused)


@pytest.mark.parametrize("n,graph,form,dtype,gamma,fused", LARGE)
def test_tile_workers_per_wave(n, graph, form, dtype, gamma, fused):
    print("case tile workers per wave n=%d %s %s %s" % (n, graph, form, dtype), flush=True)
    _compare(n, MANY_TILES, graph, form, dtype, gamma, fused)


TWO_PER_CU = 2 * 256 * 256 + 3  # past the line at two tiles per CU (beyond 32 workers), with a ragged last tile
BEYOND_32 = [  # 8 waves with 5, 6, 7 and 8 workers each, whole and not
    (33, "two_peer", "local_dadam", "bf16", 0.0, False),
    (40, "exponential", "alg1", "bf16", 0.0, True),
    (41, "complete", "eq", "bf16", 0.0, False),
    (48, "one_peer", "alg1", "f32", 0.0, False),
    (49, "two_peer", "eq", "f32", 0.1, True),
    (56, "ring", "dadam", "bf16", 0.0, False),
    (57, "two_peer", "alg1", "f32", 0.0, True),
    (63, "exponential", "local_dadam", "f32", 0.0, False),
    (64, "complete", "dadam", "bf16", 0.0, False),
    (64, "two_peer", "eq", "bf16", 0.1, False),
]


@pytest.mark.parametrize("n,graph,form,dtype,gamma,fused", BEYOND_32)
def test_tile_eight_waves(n, graph, form, dtype, gamma, fused):
    print("case tile eight waves n=%d %s %s %s" % (n, graph, form, dtype), flush=True)
    _compare(n, TWO_PER_CU, graph, form, dtype, gamma, fused)


@pytest.mark.parametrize("n,form,dtype,fused", [(20, "alg1", "bf16", False), (32, "local_dadam", "bf16", False),
                                                (31, "eq", "bf16", False), (26, "alg1", "f32", True)])
def test_tile_four_workers_per_wave(n, form, dtype, fused):
    """The batches of four workers per wave that go out at once, and those that do not."""
    print("case tile four workers per wave n=%d %s %s" % (n, form, dtype), flush=True)
    _compare(n, MANY_TILES, "two_peer", form, dtype, 0.0, fused)


@pytest.mark.parametrize("n,dtype", [(9, "f32"), (10, "bf16"), (17, "bf16"), (20, "f32")])
def test_tile_three_workers_per_wave(n, dtype):
    print("case tile three workers per wave n=%d %s" % (n, dtype), flush=True)
    _compare(n, MANY_TILES, "two_peer", "eq", dtype, 0.1, True)


@pytest.mark.parametrize("mu", [0.0, 0.9])
@pytest.mark.parametrize("n,P", [(40, TWO_PER_CU), (64, TWO_PER_CU), (28, MANY_TILES)])
@pytest.mark.parametrize("form,dtype", [("alg1", "bf16"), ("local_dadam", "f32"), ("eq", "bf16")])
def test_tile_with_and_without_outer_momentum(form, dtype, n, P, mu):
    """u present and absent: it is loaded with the values or with the rows, by form and workers per wave."""
    print("case tile momentum n=%d %s %s mu=%g" % (n, form, dtype, mu), flush=True)
    _compare(n, P, "two_peer", form, dtype, 0.0, False, mu=mu)
