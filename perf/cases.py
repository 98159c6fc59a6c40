"""Timed cases of the GASLoC round: what a training program has the library do.

A training program keeps n worker replicas on the GPU and, round after round,
runs the workers' local AdamW steps, folds the last of them into the gossip
round (or runs the round by itself), reads the consensus error and the
pseudo-gradient norm, and now and then takes the network average.  A case is
one such pass, mid-run: optimizer state that has seen a hundred steps,
parameters around N(0, 0.02^2) that differ between workers, gradients around
N(0, 1).

Fields of a case:
  pass      "steps": H local steps; "round": H local steps and a gossip round;
            "average": the network average and the consensus error of x
  n, P      workers, parameters
  graph     kind of communication graph; its random kinds draw a new graph
            every round
  form      "eq" (Eq. 1 and 2), "alg1" (Algorithm 1), "dadam", "local_dadam"
  dtype     storage of the parameters ("f32" or "bf16"; all state is fp32)
  gamma     consensus momentum (eq only)
  H         local steps in the pass
  fused     the last local step and the round in one call
  half      only half of the workers take the local steps (heterogeneous H_i)
  read      the pass ends by reading the consensus error and the
            pseudo-gradient norm, as a program that logs them does
"""
import numpy as np
import torch

import paper_2606_11081_amd as g

LR, BETA1, BETA2, EPS, WD = 4e-3, 0.9, 0.95, 1e-8, 0.1
ETA, MU, DEGREE = 0.7, 0.9, 3
ROUNDS_DONE = 10
GRAPHS = ("ring", "complete", "exponential", "one_peer_exp", "one_peer", "two_peer", "random_regular")


def _case(name, **fields):
    c = {"name": name, "pass": "round", "graph": "ring", "form": "eq", "dtype": "f32", "gamma": 0.1, "H": 1,
         "fused": True, "half": False, "read": True}
    c.update(fields)
    return c


def listed():
    return [
        # the smallest call: a toy replica, all launches and host work (the size of the smoke check)
        _case("ring-n4-p4099", n=4, P=4099),
        # the smallest workload: everything fits the last-level cache
        _case("ring-n4-p1m", n=4, P=1_048_576),
        # odd n and P, a form whose last step cannot be fused
        _case("localdadam-n11-p1m", n=11, P=1_000_003, graph="two_peer", form="local_dadam", gamma=0.0, fused=False,
              read=False),
        # the n=8 workload at its full size (134M-class replicas), one local step per round
        _case("exp-n8-p124m", n=8, P=124_000_000, graph="exponential"),
        # the inner loop: nine of ten launches of the n=16 workload
        _case("steps-n16-p100m", **{"pass": "steps"}, n=16, P=100_000_000, graph="one_peer_exp", read=False),
        # the end of an n=16 round: a local step, then the last one fused into the round
        _case("onepeerexp-n16-p100m", n=16, P=100_000_000, graph="one_peer_exp", H=2),
        # the paper's best graph, bf16 parameters, the iterate form of Algorithm 1
        _case("alg1-2peer-n16-p50m-bf16", n=16, P=50_000_000, graph="two_peer", form="alg1", dtype="bf16", gamma=0.0),
        # the n=32 workload's round: a random 3-regular graph every round, bf16 parameters
        _case("regular3-n32-p40m-bf16", n=32, P=40_000_000, graph="random_regular", dtype="bf16"),
        # the n=64 workload's round: a random matching, workers with different H_i, no consensus momentum
        _case("matching-n64-p25m", n=64, P=25_000_000, graph="one_peer", gamma=0.0, fused=False, half=True),
        # DiLoCo: every worker averages with all others
        _case("diloco-n32-p25m-bf16", n=32, P=25_000_000, graph="complete", dtype="bf16"),
        # a dense graph whose rows all differ
        _case("exp-n32-p12m", n=32, P=12_000_000, graph="exponential", fused=False, read=False),
        # evaluation and checkpoints: the network average, and how far the workers are from it
        _case("average-n16-p50m-bf16", **{"pass": "average"}, n=16, P=50_000_000, dtype="bf16", read=False),
    ]


def _log_uniform(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    """A case of the listed ones' ranges: 2 to 64 workers, a thousand to a hundred million parameters per worker,
    up to 4e8 replica-parameters, every graph, form, storage type and way to end a round."""
    n = max(2, min(64, round(_log_uniform(rng, 2, 64.4))))
    graph = rng.choice(GRAPHS)
    if graph == "random_regular":
        n = max(4, n - n % 2)
    P = int(_log_uniform(rng, 1000, min(1e8, 4e8 / n)))
    c = {"pass": rng.choice(("round",) * 7 + ("steps", "steps", "average")), "n": n, "P": P, "graph": graph,
         "form": rng.choice(("eq",) * 5 + ("alg1", "dadam", "local_dadam")), "dtype": rng.choice(("f32", "bf16")),
         "H": rng.choice((1, 1, 2)), "half": rng.random() < 0.25, "read": rng.random() < 0.5}
    c["gamma"] = rng.choice((0.1, 0.1, 0.0)) if c["form"] == "eq" else 0.0
    c["fused"] = c["form"] in ("eq", "alg1") and rng.random() < 0.7
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _active(case, seed):
    """Workers that take the local steps (None: all of them)."""
    if not case["half"]:
        return None
    a = np.zeros(case["n"], np.uint8)
    a[np.random.RandomState(seed % (1 << 31)).permutation(case["n"])[:max(1, case["n"] // 2)]] = 1
    return a


def _step_counts(case):
    return 100 + np.arange(case["n"], dtype=np.int64)


def _fill(bufs, grads, case, seed):
    """Fills columns [0, P) of the given buffers (None: not wanted) from the seed, row by row."""
    x = bufs["x"]
    n, P, dev = x.shape[0], case["P"], x.device
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(std):
        return torch.empty(P, dtype=torch.float32, device=dev).normal_(0.0, std, generator=gen)

    start = normal(0.02)
    for i in range(n):
        xi = start + normal(0.002)
        x[i, :P].copy_(xi)
        if bufs.get("y") is not None:
            bufs["y"][i, :P].copy_(xi + normal(0.01))
        bufs["m"][i, :P].copy_(normal(0.3))
        bufs["v"][i, :P].copy_(torch.empty(P, dtype=torch.float32, device=dev).uniform_(0.6, 1.4, generator=gen))
        if bufs.get("u") is not None:
            bufs["u"][i, :P].copy_(normal(0.01))
        if bufs.get("zp") is not None:
            bufs["zp"][i, :P].copy_(xi + normal(0.005))
        if grads is not None:
            grads[i, :P].copy_(normal(1.0) + 0.1 * (i % 3 - 1))


def prepare(case, seed):
    run_ = g.GASLoC(case["n"], case["P"], topology=case["graph"], seed=seed % (1 << 31), degree=DEGREE,
                    param_dtype=case["dtype"], beta1=BETA1, beta2=BETA2, eps=EPS, weight_decay=WD, outer_lr=ETA,
                    outer_momentum=MU, consensus_momentum=case["gamma"], round_form=case["form"])
    average = case["pass"] == "average"
    grads = None if average else torch.empty((case["n"], run_.ld), dtype=torch.float32, device="cuda")
    _fill(run_.bufs, grads, case, seed)
    in_steps = np.full(case["n"], case["pass"] == "steps", np.uint8)  # "steps" is in the middle of an inner loop
    run_.set_counters(_step_counts(case), in_steps, ROUNDS_DONE)
    mean = torch.empty(run_.ld, dtype=run_.x.dtype, device="cuda") if average else None
    return {"case": dict(case), "run": run_, "grads": grads, "active": _active(case, seed), "t": ROUNDS_DONE,
            "mean": mean}


def run(state):
    case, r, P = state["case"], state["run"], state["case"]["P"]
    if case["pass"] == "average":
        r.replica_mean(state["mean"])
        return {"mean": state["mean"][:P], "consensus_error": r.consensus_error_cols(0, P)}
    grads, active, H = state["grads"], state["active"], case["H"]
    if case["pass"] == "steps":
        for _ in range(H):
            r.local_step(grads, LR, active)
        return {k: r.bufs[k][:, :P] for k in ("y", "m", "v")}
    for _ in range(H - 1 if case["fused"] else H):
        r.local_step(grads, LR, active)
    t = state["t"]
    state["t"] += 1
    if case["fused"]:
        r.local_step_gossip_round(grads, LR, t, active)
    else:
        r.gossip_round(t)
    out = {k: r.bufs[k][:, :P] for k in ("x", "m", "v", "u", "zp") if r.bufs[k] is not None}
    if case["read"]:
        out["consensus_error"] = r.consensus_error()
        out["pseudo_gradient_sq"] = r.pseudo_gradient_sq()
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct ones may differ
# --------------------------------------------------------------------------

def _entries(case):
    """Entries per row of the mixing matrix."""
    n = case["n"]
    per = {"ring": 3, "complete": n, "exponential": 1 + (n - 1).bit_length(), "one_peer_exp": 2, "one_peer": 2,
           "two_peer": 3, "random_regular": DEGREE + 1}
    return min(n, per[case["graph"]])


def work(case):
    n, P, sp = case["n"], case["P"], 2 if case["dtype"] == "bf16" else 4
    rp = n * P
    if case["pass"] == "average":  # x for the average, the average, x for the consensus error
        return {"bytes": 2 * rp * sp + P * sp, "flops": 5 * rp}
    moving = (max(1, n // 2) if case["half"] else n) * P
    own_steps = case["H"] - (1 if case["pass"] == "round" and case["fused"] else 0)
    nbytes = own_steps * moving * (2 * sp + 20)  # y, g, m, v read; y, m, v written
    flops = case["H"] * moving * 18
    if case["pass"] == "round":
        with_u = case["form"] != "dadam"
        nbytes += rp * (2 * sp + (8 if with_u else 0) + (8 if case["gamma"] else 0))  # x, u, zp read and written
        if own_steps:
            nbytes += moving * sp  # y
        if case["fused"]:
            nbytes += moving * 20  # g, m, v read; m, v written
        flops += rp * (2 * _entries(case) + 16)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # fp32 passes are 4e-8 to 1.2e-7 off the 64-bit ones.  A bf16 store that rounds the other way moves that element
    # by up to 2^-7 of it (and the momentum that is fed from it by as much); bf16 passes are 1.7e-3 to 3.7e-3 off
    # the 64-bit ones, whose iterates are not rounded, and two correct ones differ where they round differently.
    if case["dtype"] == "bf16":
        return {"rel": 2e-3, "max": 0.1}
    return {"rel": 5e-7, "max": 1e-5}


# --------------------------------------------------------------------------
# the same pass in 64 bits, in plain torch
# --------------------------------------------------------------------------

_M64 = (1 << 64) - 1


def _mix64(v):
    v = ((v ^ (v >> 30)) * 0xBF58476D1CE4E5B9) & _M64
    v = ((v ^ (v >> 27)) * 0x94D049BB133111EB) & _M64
    return v ^ (v >> 31)


class _SplitMix64:
    """The published generator, seeded for round t of a schedule."""

    def __init__(self, seed, t):
        self.state = _mix64(seed ^ _mix64(t))

    def below(self, bound):
        while True:
            self.state = (self.state + 0x9E3779B97F4A7C15) & _M64
            r = _mix64(self.state)
            if r >= (1 << 64) % bound:
                return r % bound

    def permutation(self, count):
        a = list(range(count))
        for i in range(count - 1, 0, -1):
            j = self.below(i + 1)
            a[i], a[j] = a[j], a[i]
        return a


def _mixing_matrix(graph, n, seed, t):
    """W of round t, dense, with the fp32 weights that a round uses."""
    rng = _SplitMix64(seed, t)
    near = [{i} for i in range(n)]

    def link(a, b):
        near[a].add(b)
        near[b].add(a)

    if graph == "ring":
        for i in range(n):
            link(i, (i + 1) % n)
    elif graph == "complete":
        near = [set(range(n)) for _ in range(n)]
    elif graph == "exponential":
        for i in range(n):
            near[i] |= {(i + (1 << k)) % n for k in range((n - 1).bit_length())}
    elif graph == "one_peer_exp":
        hop = 1 << (t % (n - 1).bit_length())
        for i in range(n):
            near[i].add((i + hop) % n)
    elif graph == "one_peer":
        s = rng.permutation(n)
        for k in range(0, n - 1, 2):
            link(s[k], s[k + 1])
    elif graph == "two_peer":
        s = rng.permutation(n)
        for k in range(n):
            link(s[k], s[(k + 1) % n])
    else:  # pairing model: points of the workers' half edges, until no loop and no double edge comes out
        while True:
            s = rng.permutation(n * DEGREE)
            pairs = [(s[q] // DEGREE, s[q + 1] // DEGREE) for q in range(0, n * DEGREE, 2)]
            if all(a != b for a, b in pairs) and len({frozenset(p) for p in pairs}) == len(pairs):
                break
        for a, b in pairs:
            link(a, b)
    W = np.zeros((n, n), np.float32)
    for i in range(n):
        W[i, sorted(near[i])] = np.float32(1.0 / len(near[i]))
    return W.astype(np.float64)


def _exact_steps(c, y, m, v, grads, moving):
    """H local steps of the workers in `moving`, in place; c: the step constants by worker and step."""
    for s1, c2 in c:
        for i in moving:
            w = y[i] * (1.0 - float(np.float32(LR)) * float(np.float32(WD)))
            b1, b2 = float(np.float32(BETA1)), float(np.float32(BETA2))
            m[i].mul_(b1).add_(grads[i], alpha=1.0 - b1)
            v[i].mul_(b2).addcmul_(grads[i], grads[i], value=1.0 - b2)
            y[i] = w - s1[i] * m[i] / (v[i].sqrt() / c2[i] + float(np.float32(EPS)))


def exact(case, seed):
    n, P, dev = case["n"], case["P"], "cuda"
    pdt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    form, kind = case["form"], case["pass"]

    def buf(dtype=torch.float32, wanted=True):
        return torch.empty((n, P), dtype=dtype, device=dev) if wanted else None

    with_u = form != "dadam"
    bufs = {"x": buf(pdt), "y": buf(pdt), "m": buf(), "v": buf(), "u": buf(wanted=with_u),
            "zp": buf(wanted=case["gamma"] != 0.0)}
    grads = buf(wanted=kind != "average")
    _fill(bufs, grads, case, seed)
    names = {"average": (), "steps": ("y", "m", "v")}.get(kind, ("x", "m", "v") + (("u",) if with_u else ()) +
                                                          (("zp",) if case["gamma"] else ()))
    out = {k: torch.empty((n, P), dtype=torch.float64, device=dev) for k in names}
    mean = torch.empty(P, dtype=torch.float64, device=dev) if kind == "average" else None
    active = _active(case, seed)
    moving = range(n) if active is None else [int(i) for i in np.flatnonzero(active)]
    b1, b2 = float(np.float32(BETA1)), float(np.float32(BETA2))
    consts = []
    for h in range(case["H"]):
        k = (_step_counts(case) + h + 1).astype(np.float64)
        consts.append((float(np.float32(LR)) / (1.0 - b1 ** k), np.sqrt(1.0 - b2 ** k)))
    W = None
    if kind == "round":
        W = torch.from_numpy(_mixing_matrix(case["graph"], n, seed % (1 << 31), ROUNDS_DONE)).to(dev)
        row_sum = W.sum(1, keepdim=True)
    eta, mu, gamma = (float(np.float32(q)) for q in (ETA, MU, case["gamma"]))
    ce, pg = 0.0, 0.0
    chunk = max(1, (1 << 27) // n)
    for p0 in range(0, P, chunk):
        p1 = min(P, p0 + chunk)
        d = {k: b[:, p0:p1].double() for k, b in bufs.items() if b is not None and (kind != "average" or k == "x")}
        x = d["x"]
        if kind == "average":
            mean[p0:p1] = x.mean(0)
            ce += float((x - x.mean(0)).square().sum())
            continue
        y = d["y"] if kind == "steps" else x.clone()
        _exact_steps(consts, y, d["m"], d["v"], grads[:, p0:p1].double(), moving)
        if kind == "steps":
            d["y"] = y
        else:
            pg += float((x - y).square().sum())

            def outer(base, delta):  # Nesterov; leaves the new momentum in d["u"]
                d["u"] = mu * d["u"] + delta
                return base - eta * (delta + mu * d["u"])

            if form == "eq":
                z = outer(x, x - y)
                d["x"] = W @ z
                if gamma:
                    d["x"] += gamma * (z - d["zp"])
                    d["zp"] = z
            elif form == "alg1":
                d["x"] = outer(x, row_sum * x - W @ y)
            elif form == "dadam":
                d["x"] = W @ x + (y - x)
            else:
                d["x"] = outer(y, row_sum * x - W @ x)
            stored = d["x"].to(pdt).double()
            ce += float((stored - stored.mean(0)).square().sum())
        for k in names:
            out[k][:, p0:p1] = d[k]
    if kind == "average":
        return {"mean": mean, "consensus_error": ce}
    if kind == "round" and case["read"]:
        out["consensus_error"], out["pseudo_gradient_sq"] = ce, pg
    return out
