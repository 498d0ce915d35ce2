"""The work this library is used for, as measurable cases over its public Python entry points.

A case is a dict of plain values: what is called ("kind"), its sizes and its options.

  forward   one inference pass of the layer (ssm_scan_fwd), e.g. over imagined trajectories
  train     forward and gradient pass of the layer (ssm_scan_fwd, ssm_scan_bwd) over a batch of replay windows
  block     the same for the S5 block: layer and half-GLU gate (ssm_block_fwd, ssm_block_bwd)
  rollout   an imagined roll-out in step mode: the plan of the current parameters, `L` dependent steps, then
            the adjoint steps in reverse order (ssm_step_prepare, ssm_step, ssm_step_bwd)
  returns   the critic's lambda-return and its gradient (ssm_lambda_return, ssm_lambda_return_bwd)
  scan      the resettable scan and its reverse on projected elements (ssm_scan_states, ssm_scan_states_reverse)

Sizes: `Bt` sequences (trajectories) of `L` steps, layer width `H`, `P` complex states.  Everything is float32 /
complex64, the only types the library takes.  The distributions are those of
paper_2502_20168_amd/workloads.py, drawn on the GPU.
"""
import math

import torch

from paper_2502_20168_amd import binding as ssm

GAMMA, LAMBDA = 0.997, 0.95

MAX_TRAIN_WORK = 32768 * 512 * 512      # tokens * H * P of the largest listed case


def _case(name, kind, Bt, L, H=0, P=0, p_reset=0.0, first=False, x0=False, slow=False, want_x=True):
    return {"name": name, "kind": kind, "Bt": Bt, "L": L, "H": H, "P": P, "p_reset": p_reset, "first": first,
            "x0": x0, "slow": slow, "want_x": want_x}


def listed():
    return [
        # a single small layer, two short sequences: acting in the environment, where latency counts
        _case("forward_tiny", "forward", 2, 64, 32, 32),
        # a small world model on a short replay window (the small benchmark configuration)
        _case("train_small", "train", 16, 64, 256, 256, p_reset=0.02, first=True),
        # the headline benchmark: the batch of one world-model update
        _case("train_worldmodel", "train", 16, 256, 512, 512, p_reset=0.01, first=True),
        # few, very long sequences with slow decay
        _case("train_long", "train", 4, 4096, 256, 256, p_reset=0.001, first=True, slow=True),
        # wide and short: imagination from 1024 start states; only y and the last state are wanted
        _case("forward_imagination", "forward", 1024, 16, 512, 512, x0=True, want_x=False),
        # replay windows of no convenient length, with widths that no tile divides
        _case("train_ragged", "train", 20, 300, 500, 250, p_reset=0.02, x0=True),
        # the wide layer of the vision task on windows that are not whole tiles of steps
        _case("train_wide", "train", 24, 200, 1024, 512, p_reset=0.01, first=True),
        # the headline batch eight times over: a large update on one GPU
        _case("train_large", "train", 128, 256, 512, 512, p_reset=0.01, first=True),
        # one S5 block of the vision task: layer and gate, 32 windows of 128 steps
        _case("block_vision", "block", 32, 128, 1024, 512, p_reset=0.01, first=True),
        # actor-critic stage: 1024 trajectories rolled out 16 steps, with the actor's gradients
        _case("rollout", "rollout", 1024, 16, 512, 512, x0=True),
        # targets of the critic for 65536 imagined trajectories of horizon 16
        _case("returns", "returns", 65536, 16),
        # the scan on its own, on elements projected elsewhere: long sequences
        _case("scan_long", "scan", 4, 4096, 0, 256, p_reset=0.001, first=True, slow=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng):
    w = _log_uniform(rng, 32, 1024)
    return max(64, w // 64 * 64) if rng.random() < 0.5 else w


def _length(rng, lo, hi):
    if rng.random() < 0.5:
        return 1 << rng.randint(int(math.log2(lo)), int(math.log2(hi)))
    return _log_uniform(rng, lo, hi)


def draw(rng):
    kind = rng.choice(("forward", "train", "train", "train", "block", "rollout", "returns", "scan"))
    flags = {"p_reset": rng.choice((0.0, 0.001, 0.01, 0.02)), "first": rng.random() < 0.5, "x0": rng.random() < 0.5}
    if kind == "returns":
        return _unnamed(_case("", kind, _log_uniform(rng, 256, 65536), rng.randint(2, 64)))
    if kind == "rollout":
        return _unnamed(_case("", kind, _log_uniform(rng, 16, 2048), rng.randint(4, 16), _width(rng), _width(rng), **flags))
    while True:
        tokens = _log_uniform(rng, 128, 32768)
        L = _length(rng, 16, 4096)
        Bt = max(1, tokens // L)
        H, P = _width(rng), _width(rng)
        if kind == "scan":
            H = 0
        if 128 <= Bt * L <= 32768 and Bt * L * H * P <= MAX_TRAIN_WORK // 2:
            break
    want_x = kind != "forward" or rng.random() < 0.5
    return _unnamed(_case("", kind, Bt, L, H, P, slow=L >= 1024, want_x=want_x, **flags))


def _unnamed(case):
    del case["name"]
    return case


def prepare(case, seed):
    kind, Bt, L, H, P = case["kind"], case["Bt"], case["L"], case["H"], case["P"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    uniform = lambda lo, hi, *shape: torch.rand(shape, generator=gen, device="cuda") * (hi - lo) + lo
    cnormal = lambda std, *shape: torch.complex(normal(*shape) * std, normal(*shape) * std)
    s = {"case": case}
    if kind == "returns":
        even = (torch.arange(Bt, device="cuda") % 2 == 0)[None, :]
        s["reward"], s["value"], s["dret"] = normal(L, Bt), normal(L, Bt), normal(L, Bt)
        # sampled continuation flags for the even trajectories, probabilities for the odd ones
        s["cont"] = torch.where(even, (uniform(0, 1, L, Bt) >= 0.05).float(), uniform(0, 1, L, Bt))
        return s
    decay = (0.001, 0.1) if case["slow"] else (0.1, 1.0)
    s["Lambda"] = torch.complex(-uniform(*decay, P), uniform(0.0, math.pi, P))
    s["log_delta"] = uniform(math.log(1e-3), math.log(1e-1), P)
    flags = uniform(0, 1, Bt, L) < case["p_reset"]
    if case["first"]:
        flags[:, 0] = True
    s["is_first"] = flags.to(torch.uint8) if case["first"] or case["p_reset"] > 0 else None
    s["x0"] = cnormal(1.0, Bt, P) if case["x0"] else None
    if kind == "scan":
        s["A_bar"], _ = ssm.ssm_discretize(s["Lambda"], None, s["log_delta"])
        s["v"], s["gx"] = cnormal(0.05, Bt, L, P), cnormal(0.05, Bt, L, P)
        s["ws_f"], s["ws_b"] = ssm.alloc_workspace(Bt, L, 1, P, False), ssm.alloc_workspace(Bt, L, 1, P, True)
        return s
    s["B"], s["C"], s["D"] = cnormal(H ** -0.5, P, H), cnormal(H ** -0.5, H, P), normal(H)
    s["u"], s["dy"] = normal(Bt, L, H), normal(Bt, L, H)
    if kind == "rollout":
        # step mode takes one step of all trajectories at a time
        s["u"], s["dy"] = s["u"].transpose(0, 1).contiguous(), s["dy"].transpose(0, 1).contiguous()
        if s["is_first"] is not None:
            s["is_first"] = s["is_first"].t().contiguous()
        return s
    if kind == "block":
        s["W"] = normal(H, H) * H ** -0.5
        for key, bwd in (("ws_f", False), ("ws_b", True)):
            s[key] = torch.empty(ssm.ssm_block_workspace_bytes(Bt, L, H, P, bwd), dtype=torch.uint8, device="cuda")
        return s
    s["ws_f"] = ssm.alloc_workspace(Bt, L, H, P, False)
    if kind == "train":
        s["ws_b"] = ssm.alloc_workspace(Bt, L, H, P, True)
    return s


def run(state):
    return _RUN[state["case"]["kind"]](state)


def _forward(s):
    return ssm.ssm_scan_fwd(s["Lambda"], s["B"], s["C"], s["D"], s["log_delta"], s["u"], s["is_first"], s["x0"],
                            want_x=s["case"]["want_x"], workspace=s["ws_f"])


def _train(s):
    fwd = _forward(s)
    bwd = ssm.ssm_scan_bwd(s["Lambda"], s["B"], s["C"], s["D"], s["log_delta"], s["u"], s["is_first"], s["x0"],
                           fwd["x"], s["dy"], workspace=s["ws_b"])
    return {**fwd, **bwd}


def _block(s):
    par = (s["Lambda"], s["B"], s["C"], s["D"], s["log_delta"], s["W"], s["u"], s["is_first"], s["x0"])
    fwd = ssm.ssm_block_fwd(*par, workspace=s["ws_f"])
    bwd = ssm.ssm_block_bwd(*par, fwd["x"], fwd["y"], fwd["gate"], s["dy"], workspace=s["ws_b"])
    return {**fwd, **bwd}


def _rollout(s):
    P, steps = s["case"]["P"], s["case"]["L"]
    # the parameters have changed since the last roll-out: a new plan
    plan = ssm.ssm_step_prepare(s["Lambda"], s["B"], s["C"], s["log_delta"])
    first = s["is_first"]
    x, xs, ys = s["x0"], [], []
    for t in range(steps):
        x, y = ssm.ssm_step(plan, s["D"], s["u"][t], x, None if first is None else first[t], P=P)
        xs.append(x)
        ys.append(y)
    dx, dus = None, []
    for t in reversed(range(steps)):
        gx, du, dx = ssm.ssm_step_bwd(plan, s["D"], s["dy"][t], dx, None if first is None else first[t], P=P)
        dus.append(du)
    return {"x": xs[-1], "y": ys, "du": dus, "gx": gx, "dx": dx}


def _returns(s):
    ret = ssm.ssm_lambda_return(s["reward"], s["cont"], s["value"], GAMMA, LAMBDA)
    return (ret,) + ssm.ssm_lambda_return_bwd(s["cont"], s["value"], ret, s["dret"], GAMMA, LAMBDA)


def _scan(s):
    # both calls work in place; the elements are copied so that every pass scans the same ones
    x, x_last = ssm.ssm_scan_states(s["A_bar"], s["v"].clone(), s["is_first"], s["x0"], workspace=s["ws_f"])
    chi, dA, dx0 = ssm.ssm_scan_states_reverse(s["A_bar"], s["gx"].clone(), x, s["is_first"], s["x0"], workspace=s["ws_b"])
    return {"x": x, "x_last": x_last, "chi": chi, "dA_bar": dA, "dx0": dx0}


_RUN = {"forward": _forward, "train": _train, "block": _block, "rollout": _rollout, "returns": _returns, "scan": _scan}


def work(case):
    """Bytes and operations (of 32-bit products and sums) that one pass cannot do without."""
    kind, Bt, L, H, P = case["kind"], case["Bt"], case["L"], case["H"], case["P"]
    T = Bt * L
    if kind == "returns":
        return {"bytes": 4 * T * (4 + 4), "flops": 13 * T}
    flags = T if case["first"] or case["p_reset"] > 0 else 0
    ends = 8 * Bt * P * (2 if case["x0"] else 1)                       # x_last, x0
    if kind == "scan":
        return {"bytes": 32 * T * P + 2 * ends + flags, "flops": 24 * T * P}
    par = 16 * P * H + 12 * P + 4 * H                                  # B, C; Lambda, log_delta; D
    product = 4 * T * P * H                                            # one projection
    if kind == "forward":
        return {"bytes": 4 * T * 2 * H + (8 * T * P if case["want_x"] else 0) + flags + ends + par,
                "flops": 2 * product + 8 * T * P}
    if kind == "rollout":
        return {"bytes": 4 * T * 4 * H + 8 * Bt * P * (4 if case["x0"] else 3) + flags + par, "flops": 4 * product + 16 * T * P}
    train = {"bytes": 4 * T * 4 * H + 8 * T * P + flags + 2 * ends + 2 * par, "flops": 6 * product + 24 * T * P}
    if kind == "block":
        # further: out and the gate stored, W and its gradient
        train["bytes"] += 4 * T * 2 * H + 8 * H * H
        train["flops"] += 6 * T * H * H
    return train


def tolerance(case):
    # Sums of float32 products: a few 1e-6 of the norm for the activations.  The gradients of Lambda and log_delta sum
    # over all tokens terms that largely cancel, behind a recurrence that carries rounding over 1 / (1 - |A_bar|) steps.
    if case["kind"] == "returns":
        return {"rel": 1e-6}
    if case["kind"] in ("forward", "rollout"):
        return {"rel": 2e-5}
    return {"rel": 1e-4}
