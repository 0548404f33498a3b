"""The work that is timed: what programs that train with this library have it do, through its public entry points.

Four kinds of case:

  train         a network in the middle of its training: one factor-update period (four minibatches, one of which
                updates the Fisher factors), fresh minibatches, the updated weights read back at the end
  replicas      several replicas of a network on one GPU, each stepped on a stream of its own, and the parameter average
                over them; with `reset` the average is followed by a step that builds every Fisher factor anew from its
                first minibatch, as the processes of a distributed run do after each averaging
  precondition  the preconditioner on its own, for a program that has its own network: four calls on fresh matrices
                (the call works in place, so each is copied into the buffer that the caller hands over)
  simple        the stateless preconditioner (factors from the other rows of the same minibatch), four calls

Everything is fp32 with 32-bit labels, which is all the library takes.
"""
import math

import torch

import paper_1410_7455_amd as ng

LR = 0.002                # a rate of the later epochs: at the first epochs' 0.01 a rounding difference grows fast from step to step
MAX_CHANGE = 0.075        # with renormalised p-norm layers it keeps the summed-gradient steps stable
CALLS = 4                 # minibatches (calls) of one pass: one update period
WARM = 12                 # minibatches before the first pass: the first ten update their factors on every call
ALPHA, HISTORY, EPSILON = 4.0, 2000.0, 1e-10

# Speech-shaped network with renormalised p-norm layers: 360 -> 4 x (3000 -> 300) -> 5000
SPEECH = dict(input=360, hidden=3000, layers=5, classes=5000, nonlin="pnorm", group=10, minibatch=512, rank_in=20, rank_out=80, period=4)


def listed():
    return [
        # the smallest call: a tiny tanh network, where launches and host work are everything
        dict(name="train_tiny_tanh", kind="train", method="online", input=40, hidden=128, layers=3, classes=50, nonlin="tanh", group=10,
             minibatch=64, rank_in=4, rank_out=8, period=4),
        # a small p-norm network whose sizes are multiples of nothing
        dict(name="train_small_ragged", kind="train", method="online", input=52, hidden=230, layers=3, classes=203, nonlin="pnorm", group=10,
             minibatch=93, rank_in=5, rank_out=13, period=4),
        # the everyday case
        dict(name="train_speech_pnorm", kind="train", method="online", **SPEECH),
        # the largest network: six layers of 2048 tanh units, 8000 classes, minibatches of 1024
        dict(name="train_wide_tanh", kind="train", method="online", input=440, hidden=2048, layers=7, classes=8000, nonlin="tanh", group=10,
             minibatch=1024, rank_in=20, rank_out=80, period=4),
        # the everyday network with the stateless method in place of the online one
        dict(name="train_speech_simple", kind="train", method="simple", **SPEECH),
        # several models trained side by side on one GPU, averaged without forgetting their factors
        dict(name="replicas_interleaved", kind="replicas", replicas=8, reset=False, **SPEECH),
        # the restart behind an averaging point: every factor is built anew
        dict(name="replicas_restart", kind="replicas", replicas=2, reset=True, **SPEECH),
        # the preconditioner alone: a layer-input matrix, factor updated on every call
        dict(name="precondition_input_r20", kind="precondition", rows=512, dim=3001, rank=20, ones=True, period=1),
        # an output-derivative matrix, factor updated on every call
        dict(name="precondition_output_r80", kind="precondition", rows=512, dim=5000, rank=80, ones=False, period=1),
        # the same with the usual period: one call of four updates
        dict(name="precondition_output_r80_p4", kind="precondition", rows=512, dim=5000, rank=80, ones=False, period=4),
        # few rows, a dimension and a rank that are multiples of nothing
        dict(name="precondition_small_ragged", kind="precondition", rows=63, dim=205, rank=13, ones=True, period=4),
        # the stateless method alone
        dict(name="simple_output", kind="simple", rows=512, dim=5000, ones=False),
    ]


def _log(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "replicas", "precondition", "precondition", "precondition", "simple"])
    if kind in ("train", "replicas"):
        # the input dimension is a multiple of four, as the library asks; a minibatch has more rows than the largest rank
        nonlin, group = rng.choice([("tanh", 10), ("pnorm", 10), ("pnorm", 5)])
        if nonlin == "tanh":
            hidden = _log(rng, 100, 2048)
        else:
            hidden = group * _log(rng, 30, 300)
        rank_in, rank_out = _log(rng, 4, 30), _log(rng, 6, 90)
        smallest_input = rank_in + 1
        if nonlin == "pnorm":   # the rank stays below every matrix' dimension
            rank_in = min(rank_in, hidden // group - 1)
        rank_out = min(rank_out, hidden - 1)
        case = dict(kind=kind, input=4 * _log(rng, max(10, smallest_input // 4 + 1), 110), hidden=hidden, layers=rng.randint(2, 6),
                    classes=_log(rng, 100, 6000), nonlin=nonlin, group=group, minibatch=_log(rng, 2 * rank_out + 20, 700), rank_in=rank_in,
                    rank_out=min(rank_out, 90), period=4)
        if kind == "train":
            case["method"] = rng.choice(["online", "online", "simple"])
        else:
            case["reset"] = rng.random() < 0.3
            case["replicas"] = rng.randint(2, 3 if case["reset"] else 5)
        return case
    if kind == "precondition":
        rank = _log(rng, 4, 96)
        return dict(kind=kind, rows=_log(rng, max(50, 2 * rank), 1024), dim=_log(rng, max(100, 3 * rank), 6000), rank=rank,
                    ones=rng.random() < 0.5, period=rng.choice([1, 4]))
    return dict(kind=kind, rows=_log(rng, 50, 700), dim=_log(rng, 100, 5000), ones=rng.random() < 0.5)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _sizes(case):
    dims = [case["input"]] + [case["hidden"]] * (case["layers"] - 1) + [case["classes"]]
    nonlin = [ng.NGSGD_PNORM if case["nonlin"] == "pnorm" else ng.NGSGD_TANH] * (case["layers"] - 1)
    step = case["hidden"] // case["group"] if case["nonlin"] == "pnorm" else case["hidden"]
    in_dims = [case["input"]] + [step] * (case["layers"] - 1)
    return dims, nonlin, in_dims


def _minibatches(case, g, count):
    """Features with a mean and scale per dimension, labels with a Zipf law over the classes."""
    d, n, c = case["input"], case["minibatch"], case["classes"]
    mean = torch.rand(d, generator=g, device="cuda") * 4.0 - 2.0
    scale = torch.rand(d, generator=g, device="cuda") * 1.5 + 0.5
    x = torch.randn(count, n, d, generator=g, device="cuda") * scale + mean
    law = torch.arange(1, c + 1, dtype=torch.float32, device="cuda") ** -1.1
    y = torch.multinomial(law, count * n, replacement=True, generator=g).to(torch.int32).view(count, n)
    return list(zip(x.unbind(0), y.unbind(0)))


def _network(case, g, side_streams=0):
    dims, nonlin, in_dims = _sizes(case)
    net = ng.Network(dims, nonlin, case["minibatch"], case["group"], case["rank_in"], case["rank_out"], ALPHA, HISTORY, EPSILON, case["period"],
                     renorm=case["nonlin"] == "pnorm", max_change_per_sample=MAX_CHANGE, method=case.get("method", "online"),
                     side_streams=side_streams)
    for layer in range(case["layers"]):
        w = torch.zeros(dims[layer + 1], in_dims[layer] + 1, device="cuda")
        body = torch.randn(dims[layer + 1], in_dims[layer], generator=g, device="cuda") / math.sqrt(in_dims[layer])
        # Not zero in the softmax layer: its first derivatives, one-hot minus nearly uniform, would have many equal singular
        # values, and the factors built from them would not be unique.  Behind wide tanh layers full size makes the first
        # steps unstable.
        small = layer == case["layers"] - 1 and case["nonlin"] == "tanh"
        w[:, :-1] = body * 0.1 if small else body
        net.set_params(layer, w)
    return net


def _pool_size(case):
    """Minibatches kept: few are learnt by heart when they come round again, and their derivatives then vanish."""
    return max(32, min(256, int(2e8 / (4.0 * case["minibatch"] * case["input"]))))


def _matrices(case, g, count):
    """Rows with covariance Q diag(1/k^2) Q^T, Q a product of reflections; the bias input as the last column if `ones`."""
    n, d = case["rows"], case["dim"]
    k = torch.arange(1, d + 1, dtype=torch.float32, device="cuda")
    vs = [v / v.norm() for v in torch.randn(4, d, generator=g, device="cuda").unbind(0)]
    out = []
    for _ in range(count):
        m = torch.randn(n, d, generator=g, device="cuda") / k
        for v in vs:
            m -= 2.0 * torch.outer(m @ v, v)
        if case["ones"]:
            m[:, -1] = 1.0
        buf = torch.zeros(n, (d + 3) // 4 * 4, device="cuda")   # rows start on 16-byte boundaries
        buf[:, :d] = m
        out.append(buf)
    return out


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "train":
        net = _network(case, g)
        pool = _minibatches(case, g, _pool_size(case))
        for x, y in pool[:WARM]:
            net.step(x, y, LR)
        net.join()
        return dict(case=case, net=net, pool=pool, at=WARM)
    if kind == "replicas":
        nets = [_network(case, _gen(seed), side_streams=1) for _ in range(case["replicas"])]   # the same model in all
        pool = _minibatches(case, g, max(2 * WARM, _pool_size(case) // 2))
        streams = [torch.cuda.Stream() for _ in nets]
        ready = torch.cuda.Event()
        ready.record()
        for r, (net, s) in enumerate(zip(nets, streams)):
            s.wait_event(ready)
            for i in range(WARM):
                x, y = pool[(r + i * len(nets)) % len(pool)]
                net.step(x, y, LR, stream=s)
            net.join(s)
        torch.cuda.synchronize()
        return dict(case=case, nets=nets, streams=streams, pool=pool, at=WARM * len(nets))
    ld = (case["dim"] + 3) // 4 * 4
    mats = _matrices(case, g, 12)
    bufs = [torch.empty(case["rows"], ld, device="cuda") for _ in range(CALLS)]
    state = dict(case=case, mats=mats, bufs=bufs, at=0)
    if kind == "precondition":
        state["pre"] = ng.Preconditioner(case["dim"], case["rank"], case["rows"], ALPHA, HISTORY, EPSILON, update_period=case["period"])
        for m in mats:
            bufs[0].copy_(m)
            state["pre"].precondition(bufs[0][:, : case["dim"]])
    else:
        state["pre"] = ng.SimplePreconditioner(case["rows"], case["dim"])
    return state


def _run_train(state):
    net, pool, case = state["net"], state["pool"], state["case"]
    logprob = torch.empty(CALLS, dtype=torch.float64, device="cuda")
    for i in range(CALLS):
        x, y = pool[(state["at"] + i) % len(pool)]
        net.step(x, y, LR, logprob_out=logprob[i:])
    state["at"] += CALLS
    return [logprob] + [net.get_params(layer) for layer in range(case["layers"])]


def _run_replicas(state):
    """Without reset: a period of minibatches on every replica, then the average. With reset: the average of what
    the replicas trained so far, then the first minibatch of their next round (which initialises every factor)."""
    nets, streams, pool, case = state["nets"], state["streams"], state["pool"], state["case"]
    main = torch.cuda.current_stream()
    count = 1 if case["reset"] else CALLS
    logprob = torch.empty(len(nets), count, dtype=torch.float64, device="cuda")
    if case["reset"]:
        ng.average(nets, reset_preconditioners=True)
    for s in streams:
        s.wait_stream(main)
    for i in range(count):
        for r, (net, s) in enumerate(zip(nets, streams)):
            x, y = pool[(state["at"] + i * len(nets) + r) % len(pool)]
            net.step(x, y, LR, logprob_out=logprob[r, i:], stream=s)
    state["at"] += count * len(nets)
    for s in streams:
        main.wait_stream(s)
    if not case["reset"]:
        ng.average(nets, reset_preconditioners=False)
        nets = nets[:1]   # all hold the average
    return [logprob] + [net.get_params(layer) for net in nets for layer in range(case["layers"])]


def _run_precondition(state):
    pre, case = state["pre"], state["case"]
    gamma = torch.empty(CALLS, device="cuda")
    norms = torch.empty(CALLS, case["rows"], device="cuda")
    for i, buf in enumerate(state["bufs"]):
        buf.copy_(state["mats"][(state["at"] + i) % len(state["mats"])])
        pre.precondition(buf[:, : case["dim"]], gamma=gamma[i:], rownorm2=norms[i])
    state["at"] += CALLS
    return [gamma, norms] + [buf[:, : case["dim"]] for buf in state["bufs"]]


def run(state):
    kind = state["case"]["kind"]
    if kind == "train":
        return _run_train(state)
    if kind == "replicas":
        return _run_replicas(state)
    return _run_precondition(state)


def _factor(n, d, r, updates, calls):
    """(bytes, flops) of the online method's factor: W read on each call and written by an update."""
    flops = calls * 4.0 * n * d * r + updates * (2.0 * n * d * r + 4.0 * r * r * d + 2.0 * r * r * n)
    return 4.0 * r * d * (calls + updates), flops


def _simple(n, d):
    m = min(n, d)
    return n * float(d) * m + 2.0 * m ** 3 + 2.0 * n * float(d) * m   # half the Gram matrix, the inverse, Q


def _step(case, calls, updates):
    """(bytes, flops) of `calls` minibatches: weights and factors in and out, features and labels in, three products per layer."""
    dims, _, in_dims = _sizes(case)
    n = case["minibatch"]
    nbytes, flops = calls * n * (case["input"] + 1) * 4.0, 0.0
    for layer, (i, o) in enumerate(zip(in_dims, dims[1:])):
        nbytes += calls * 8.0 * o * (i + 1)
        flops += calls * 2.0 * n * o * ((i + 1) * 2 + (i if layer else 0))
        if case.get("method") == "simple":
            flops += calls * (_simple(n, i + 1) + _simple(n, o))
        else:
            for d, r in ((i + 1, case["rank_in"]), (o, case["rank_out"])):
                b, f = _factor(n, d, r, updates, calls)
                nbytes, flops = nbytes + b, flops + f
    return nbytes, flops


def work(case):
    kind = case["kind"]
    if kind == "train":
        nbytes, flops = _step(case, CALLS, CALLS / case["period"])
    elif kind == "replicas":
        dims, _, in_dims = _sizes(case)
        nbytes, flops = _step(case, *((1, 1) if case["reset"] else (CALLS, CALLS / case["period"])))
        nbytes += 8.0 * sum(o * (i + 1) for i, o in zip(in_dims, dims[1:]))
        if case["reset"]:   # the eigen-decomposition behind each initial factor: 4/3 n^3 to reduce, 2 n^2 R for the vectors
            for i, o in zip(in_dims, dims[1:]):
                for d, r in ((i + 1, case["rank_in"]), (o, case["rank_out"])):
                    m = min(d, case["minibatch"])
                    flops += 1.0 * d * case["minibatch"] * m + 4.0 / 3.0 * m ** 3 + 2.0 * m * m * r
        nbytes, flops = nbytes * case["replicas"], flops * case["replicas"]
    elif kind == "precondition":
        nbytes, flops = _factor(case["rows"], case["dim"], case["rank"], CALLS / case["period"], CALLS)
        nbytes += CALLS * 8.0 * case["rows"] * case["dim"]
    else:
        nbytes, flops = CALLS * 8.0 * case["rows"] * case["dim"], CALLS * _simple(case["rows"], case["dim"])
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the largest difference from the same passes in 64 bits (warm-up included), over the listed and drawn cases."""
    if case["kind"] == "simple":
        return {"rel": 1e-5, "max": 2.2e-3}      # 1.6e-6, 5.4e-4
    if case["kind"] == "precondition":
        return {"rel": 5e-5, "max": 7e-3}        # 1.2e-5, 1.7e-3: 12 calls before the pass, each updating the factor the next one uses
    if case.get("method") == "simple":
        return {"rel": 4e-5, "max": 6e-4}        # 8e-6, 1.6e-4
    if case["nonlin"] == "tanh":
        return {"rel": 1e-3, "max": 0.18}        # 2.7e-4, 4.7e-2: one row of the softmax layer, a class seen once
    return {"rel": 4e-3, "max": 9e-2}            # 9.8e-4, 2.2e-2
