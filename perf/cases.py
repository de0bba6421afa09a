"""The work this library is used for, as cases that can be prepared, run and compared.

Most cases are one forward pass of a Mixture-of-Experts layer around its experts, as a model calls it: `route_xw` (projection,
SoftTopk scores, integer rewards, assignment under capacities, gates, dispatch lists), `dispatch_tokens` (the expert input buffers)
and `combine` (the gate-weighted sum of what the experts return).  The experts themselves belong to the model; here they are the
identity, so the layer's result for token i is (sum of its gates) * x_i.  That result does not depend on the order of a token's
slots, which the exact assignment leaves open, while every pair, gate, list and position has to be right to produce it.

The other cases are the router's backward pass (load-balance loss and derivative of the gates) and the top-2 step with Sinkhorn.
"""
import math

import torch

import paper_2508_12801_amd as ms

DEVICE = "cuda:0"
SINKHORN_TAU, SINKHORN_ITERATIONS = 0.05, 20
AUX_WEIGHT = 0.01


def _layer(name, T, d, E, k, factor, bias, dtype="bf16", t=1.0, assignment="exact"):
    """`factor`: the experts' capacity over T*k/E, the mean number of tokens per expert.  `bias`: how uneven the experts' popularity is."""
    case = dict(kind="layer", T=T, d=d, E=E, k=k, factor=factor, bias=bias, dtype=dtype, t=t, assignment=assignment)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest batch anyone routes: a unit test, an interactive request; launches and host work are all of it
        _layer("layer 64 tokens, 8 experts", 64, 64, 8, 2, 1.0, "none", dtype="fp32", t=0.0),
        # a serving step: a few hundred sequences decode one token each through a fine-grained layer
        _layer("layer 256 tokens, 64 experts", 256, 2048, 64, 8, 1.25, "zipf"),
        # one training sequence batch through a coarse top-2 layer, capacity exactly k*n/e
        _layer("layer 4096 tokens, top 2 of 16", 4096, 1024, 16, 2, 1.0, "normal"),
        # a width and an expert count that fit no tile, fp32 throughout, a token count with a remainder everywhere
        _layer("layer 10007 tokens, fp32, ragged", 10007, 1000, 96, 6, 1.1, "normal", dtype="fp32"),
        # fine-grained layers of training size, tight capacity and uneven expert popularity
        _layer("layer 16384 tokens, top 8 of 64", 16384, 2048, 64, 8, 1.0, "zipf"),
        # the same with a quarter of the demand dropped for lack of room
        _layer("layer 16384 tokens, 3/4 room", 16384, 2048, 64, 8, 0.75, "zipf"),
        # more, narrower experts
        _layer("layer 16384 tokens, 256 experts", 16384, 2048, 256, 8, 1.0, "zipf"),
        # capacity factor 1.25 and balanced experts: the assignment is nearly free, the data movement is the layer
        _layer("layer 32768 tokens, room to spare", 32768, 2048, 64, 8, 1.25, "none"),
        # the batch of a GPU in the method's own training runs, with its fast assignment (iterative rerouting)
        _layer("layer 44032 tokens, rerouting", 44032, 1024, 64, 2, 1.0, "zipf", assignment="iter"),
        # the largest batch: prefill or training of 65536 tokens over 128 experts
        _layer("layer 65536 tokens, top 8 of 128", 65536, 2048, 128, 8, 1.0, "zipf"),
        # the router's backward pass for that batch
        dict(name="backward 65536 tokens", kind="backward", T=65536, E=128, k=8),
        # scores, the top-1 choice, Sinkhorn on the residual and gates: the method's approximate top-2 step
        dict(name="sinkhorn 4096 tokens", kind="sinkhorn", T=4096, E=16),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: any number of tokens, expert counts on and off the powers of two, widths on and off the tiles."""
    kind = rng.choices(("layer", "backward", "sinkhorn"), (10, 1, 1))[0]
    T = _log_uniform(rng, 64, 65536)
    if kind == "backward":
        return dict(kind=kind, T=T, E=rng.choice((8, 16, 24, 32, 48, 64, 96, 128)), k=rng.randint(1, 8))
    if kind == "sinkhorn":
        return dict(kind=kind, T=T, E=rng.choice((8, 12, 16, 32, 48, 64)))
    # more experts than 128, and batches with less room than demand, come in batches of up to 16384 tokens
    E = rng.choice((8, 16, 20, 32, 48, 64, 64, 96, 128) + ((160, 256) if 1024 <= T <= 16384 else ()))
    k = rng.choice((1, 2, 2, 4, 6, 8))
    factor = rng.choice((1.0, 1.0, 1.0, 1.1, 1.25, 1.5) + ((0.75,) if T <= 16384 and E <= 64 else ()))
    dtype = rng.choices(("bf16", "fp32"), (4, 1))[0]
    most = 2048 if dtype == "bf16" else 1024
    d = 64 * rng.randint(1, most // 64) if rng.random() < 0.7 else 8 * rng.randint(8, most // 8)
    return _layer(None, T, d, E, k, factor, rng.choice(("none", "normal", "zipf")), dtype=dtype, t=rng.choice((0.0, 1.0, 1.0)),
                  assignment=rng.choices(("exact", "iter"), (5, 1))[0])


def _capacity(case):
    return min(case["T"], max(1, math.ceil(case["factor"] * case["T"] * case["k"] / case["E"] - 1e-9)))


def _expert_bias(kind, E, gen):
    """Per-expert logit offsets: none, i.i.d. with variance 1/2, or a Zipf(1.2) popularity scaled to [0, 2]."""
    if kind == "none":
        return None
    if kind == "normal":
        return torch.randn(E, generator=gen, device=DEVICE) * math.sqrt(0.5)
    w = torch.arange(1, E + 1, device=DEVICE, dtype=torch.float64) ** -1.2
    b = 2.0 * (w - w[-1]) / (w[0] - w[-1])
    return b[torch.randperm(E, generator=gen, device=DEVICE)].float()


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    T, E = case["T"], case["E"]
    if case["kind"] == "layer":
        d, dtype = case["d"], torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        x = torch.randn(T, d, generator=gen, device=DEVICE).to(dtype)
        W = (torch.randn(d, E, generator=gen, device=DEVICE) / math.sqrt(d)).to(dtype)
        return dict(case=case, x=x, W=W, bias=_expert_bias(case["bias"], E, gen), C=_capacity(case))
    logits = torch.randn(T, E, generator=gen, device=DEVICE) + _expert_bias("zipf" if case["kind"] == "backward" else "normal", E, gen)
    if case["kind"] == "sinkhorn":
        return dict(case=case, logits=logits, C=math.ceil(2 * T / E))
    # what the forward pass left behind, and the gradient of the loss with respect to every gate
    k = case["k"]
    fwd = ms.route_logits(logits, k, math.ceil(T * k / E), assignment="iter", allow_not_converged=True)
    dgates = torch.randn(T, k, generator=gen, device=DEVICE)
    return dict(case=case, logits=logits, scores=fwd["scores"], assign=fwd["assign"], offsets=fwd["expert_offsets"], dgates=dgates)


def run(state):
    case = state["case"]
    if case["kind"] == "layer":
        x, E, k, C = state["x"], case["E"], case["k"], state["C"]
        r = ms.route_xw(x, state["W"], state["bias"], k, C, t=case["t"], assignment=case["assignment"])
        expert_in = ms.dispatch_tokens(x, r["expert_offsets"], r["disp_token"], E, C)
        y = ms.combine(expert_in, r["assign"], r["token_pos"], r["gates"])
        return dict(scores=r["scores"], y=y, pairs=r["stats"]["flow_value"], total=float(r["stats"]["total_score_q"]))
    if case["kind"] == "sinkhorn":
        scores, q = ms.softtopk(state["logits"], 2, 1.0)
        a = ms.assign_top1_sinkhorn(scores, state["C"], SINKHORN_TAU, SINKHORN_ITERATIONS)
        return dict(scores=scores, q=q, assign=a["assign"], gates=ms.gates(scores, a["assign"]))
    aux = ms.aux_loss(state["scores"], state["offsets"], AUX_WEIGHT)
    dlogits = ms.gates_backward(state["logits"], state["scores"], state["assign"], state["dgates"], aux["dscores_col"])
    return dict(loss=aux["loss"], mean_scores=aux["mean_scores"], dscores_col=aux["dscores_col"], dlogits=dlogits)


def work(case):
    T, E = case["T"], case["E"]
    if case["kind"] == "backward":
        k = case["k"]
        return {"bytes": 4 * (3 * T * E + 2 * T * k + 4 * E), "flops": 8 * T * E}
    if case["kind"] == "sinkhorn":
        # the residual affinities are a function of the scores; each of the iterations needs every entry twice
        return {"bytes": 4 * (3 * T * E + 4 * T), "flops": (4 * SINKHORN_ITERATIONS + 12) * T * E}
    d, k, C, size = case["d"], case["k"], _capacity(case), 2 if case["dtype"] == "bf16" else 4
    pairs = min(T * k, E * C)
    routing = (T * d + d * E) * size + 3 * 4 * T * E + 4 * (5 * T * k + 3 * E)   # x, W; logits, scores, rewards; five lists of pairs
    movement = (E * C * d + pairs * d) * size + 4 * T * d                        # expert buffers out and back, the layer's result
    return {"bytes": routing + movement, "flops": 2 * T * d * E + 2 * pairs * d}


def tolerance(case):
    if case["kind"] == "backward":
        return {"rel": 1e-5, "max": 1e-3}
    if case["kind"] == "sinkhorn":
        # 20 iterations of fp32 sums: the plan is good to about 1e-4 of its row's maximum, so a second choice may fall either way
        # where two experts are that close, and the gate with it
        return {"rel": 5e-3, "max": 0.9, "differ": 2e-3}
    # The scores agree to about 1e-6.  The assignment is the exact optimum of rewards rounded to integers: another order of the
    # projection's sums moves some of them by one unit, and optima that differ in no unit of score exist as well; either way a few
    # tokens in ten thousand change an expert, and their rows of y with it; experts whose logits are that close swap their ranks
    # and with them their multipliers.
    return {"rel": 3e-3, "max": 0.6}
