"""Calls around a round on the GPU: a round recorded in a HIP graph, the
consensus error reduced afresh, the network average's division, calls after a
failed HIP call of the program's own."""
import numpy as np
import pytest

import gasloc_inputs as gi

pytestmark = pytest.mark.gpu


def _context(n, P, form, dtype, gamma, stream):
    import paper_2606_11081_amd as g

    return g.GASLoC(n, P, topology="complete", param_dtype=dtype, outer_lr=gi.OUTER_LR,
                    outer_momentum=gi.OUTER_MOMENTUM, consensus_momentum=gamma, round_form=form, stream=stream)


def _bits(t):
    import torch

    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


@pytest.mark.parametrize("n,P,form,dtype,gamma", [(8, 1_500, "eq", "f32", 0.1), (40, 300, "eq", "bf16", 0.0),
                                                  (17, 513, "dadam", "f32", 0.0)])
def test_recorded_complete_round_keeps_its_graph(n, P, form, dtype, gamma):
    """Replays of a recorded round whose rows are all equal mix with the
    recorded entries, also after rounds with another graph on the context."""
    import torch

    print("case recorded complete round n=%d P=%d %s %s" % (n, P, form, dtype), flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        run = _context(n, P, form, dtype, gamma, stream)
        ref = _context(n, P, form, dtype, gamma, stream)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(n * P)
        names = [k for k in ("x", "y", "m", "v", "u", "zp") if run.bufs[k] is not None]
        start = {k: torch.empty((n, P), device="cuda").normal_(0.0, 0.02, generator=gen).to(run.bufs[k].dtype)
                 for k in names}
        ring = (np.arange(0, 3 * n + 1, 3, dtype=np.int32),
                np.concatenate([np.sort([(i - 1) % n, i, (i + 1) % n]) for i in range(n)]).astype(np.int32),
                np.full(3 * n, 1.0 / 3.0, np.float32))

        def restore(r):
            for k in names:
                r.bufs[k][:, :P].copy_(start[k])
            r.set_counters(np.full(n, 7, np.int64), np.ones(n, np.uint8), 3)

        restore(ref)
        ref.gossip_round(3)
        want = {k: _bits(ref.bufs[k][:, :P]) for k in names}
        stats = (ref.consensus_error(), ref.pseudo_gradient_sq())

        run.gossip_round(3)  # warm-up
        restore(run)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            run.gossip_round(3)
        for replay in range(3):
            restore(run)
            graph.replay()
            for k in names:
                assert torch.equal(_bits(run.bufs[k][:, :P]), want[k]), (replay, k)
            run.gossip_round(4, ring)  # eager work between the replays
            stream.synchronize()
        restore(run)
        graph.replay()
        assert run.pseudo_gradient_sq() == stats[1]
        run.gossip_round(3)
        restore(run)
        run.gossip_round(3)
        assert (run.consensus_error(), run.pseudo_gradient_sq()) == stats
        run.close()
        ref.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [2, 11, 33, 64])
def test_consensus_error_afresh_is_the_rounds(n, dtype):
    """One column: the error that a round keeps, the one reduced afresh and the
    stated arithmetic (deviations from worker 0, fp64, each operation rounded
    on its own, workers in order) are the same number."""
    import torch

    print("case consensus error afresh n=%d %s" % (n, dtype), flush=True)
    import paper_2606_11081_amd as g

    run = g.GASLoC(n, 1, topology="ring", param_dtype=dtype, outer_lr=gi.OUTER_LR, outer_momentum=gi.OUTER_MOMENTUM,
                   consensus_momentum=0.1)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    grads = torch.empty((n, run.ld), device="cuda")
    run.x.normal_(0.0, 1.0, generator=gen)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    for t in range(12):
        grads.normal_(0.0, 1.0, generator=gen)
        run.local_step_gossip_round(grads, gi.LOCAL_LR, t)
        fused = run.consensus_error()
        afresh = run.consensus_error_cols(0, 1)
        g.gasloc_consensus_error_cols_noalloc(run.x, dtype, n, run.ld, 0, 1, out)
        x = run.x[:, 0].double().cpu().numpy()
        s = q = np.float64(0.0)
        for v in x[1:]:
            d = v - x[0]
            s += d
            q += d * d
        assert fused == afresh == float(out) == q - s * s * (1.0 / np.float64(n)), t
    run.close()


def test_calls_after_a_failed_hip_call_of_the_program():
    """A HIP call of the program's own that failed, and whose error the program
    has handled, fails no call of the library and is still there to be read."""
    import torch

    print("case calls after a failed HIP call", flush=True)
    import paper_2606_11081_amd as g

    n, P = 4, 1_000
    lib = g.library()  # its symbols and those of the HIP runtime it is linked to
    x = torch.zeros(n, P, device="cuda")
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    grads = torch.ones(n, g.padded_ld(P, "f32"), device="cuda")
    mean = torch.empty(P, device="cuda")
    bufs = g.alloc_buffers(n, P)
    bufs["x"].zero_()
    torch.cuda.synchronize()
    lib.hipGetLastError()
    failed = lib.hipSetDevice(1 << 20)  # no such GPU: refused by the runtime, nothing reaches the device
    assert failed != 0
    try:
        ctx = g.gasloc_init(n, P, g.make_topology_struct("complete", 0, 3), g.make_hparams(), bufs["x"], bufs["y"],
                            bufs["m"], bufs["v"], bufs["u"], bufs["zp"], bufs["ld"],
                            torch.cuda.current_stream().cuda_stream)
        g.gasloc_local_step(ctx, grads, grads.shape[1], None, 1e-3)
        g.gasloc_gossip_round(ctx, None, 0)
        assert g.gasloc_consensus_error(ctx) == 0.0
        assert g.gasloc_consensus_error_cols(ctx, 0, P) == 0.0
        g.gasloc_replica_mean(ctx, mean)
        g.gasloc_destroy(ctx)
        g.gasloc_consensus_error_cols_noalloc(x, "f32", n, P, 0, P, out)
    finally:
        left = lib.hipGetLastError()  # cleared for the tests that follow
    assert left in (0, failed)
    assert float(out) == 0.0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_replica_mean_is_the_rounded_quotient(dtype):
    """For every worker count the average is the fp64 sum in worker order over
    n, correctly rounded, then rounded to the parameters: random values,
    infinities, NaN, signed zeros, subnormals and the largest finite ones."""
    import torch

    print("case replica mean quotient %s" % dtype, flush=True)
    import paper_2606_11081_amd as g

    P = 2_051
    pdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator()
    gen.manual_seed(3)
    special = torch.tensor([0.0, -0.0, float("inf"), float("-inf"), float("nan"), 1e-45, -1e-45, 1e-38, 3.3895314e38,
                            -3.3895314e38])
    for n in range(1, 65):
        x = torch.randn(n, P, generator=gen) * torch.exp(4.0 * torch.randn(n, P, generator=gen))
        x[:, : len(special)] = special  # every worker the same
        pick = torch.randint(0, len(special), (n, 200), generator=gen)
        x[:, 100:300] = special[pick]  # and mixed
        x = x.to(pdt)
        run = g.GASLoC(n, P, topology="ring", param_dtype=dtype)
        run.x[:, :P].copy_(x)
        out = torch.empty(run.ld, dtype=pdt, device="cuda")
        run.replica_mean(out)
        s = torch.zeros(P, dtype=torch.float64)
        for i in range(n):
            s = s + x[i].double()
        want = (s / n).float().to(pdt)
        got = out[:P].cpu()
        run.close()
        nan = torch.isnan(want)
        assert torch.equal(torch.isnan(got), nan), n
        assert torch.equal(_bits(got[~nan]), _bits(want[~nan])), n
