"""The calls whose time this library is judged by: optimizer steps of real sizes through its public entry points.

A case is one call of a training loop's optimizer on the weights it has in hand: a single matrix (`step`), a stack of
same-shape layers (`strided`, or `batched` by pointers), a call with options (`ex`), or a model's whole layer stack in one
call (`groups`). One pass updates W and M in place from G, as each training step does.
"""
import math

import torch

from paper_2512_16928_amd import binding

MU, LR, STEPS = 0.95, 0.02, 5
QUINTIC = (3.4445, -4.7750, 2.0315)
EPS = 1e-7

#: The shapes of a grouped call, as (rows, cols, matrices): all 96 matrices of the 1B-style stack, one layer of the 7B-style
#: stack, and one layer of a small model.
STACKS = {
    "1b": ((2048, 2048, 64), (8192, 2048, 16), (2048, 8192, 16)),
    "1b-layer": ((2048, 2048, 4), (8192, 2048, 1), (2048, 8192, 1)),
    "7b-layer": ((4096, 4096, 4), (11008, 4096, 2), (4096, 11008, 1)),
    "304m": ((1024, 1024, 64), (4096, 1024, 16), (1024, 4096, 16)),
    "304m-layer": ((1024, 1024, 4), (4096, 1024, 1), (1024, 4096, 1)),
}


def listed():
    return [
        # the smallest: one 256 x 256 fp32 layer, where launches and latency are everything
        {"name": "one-256-fp32", "call": "ex", "rows": 256, "cols": 256, "batch": 1, "alpha": 0.25, "w": "f32", "g": "f32"},
        # a loop over parameters calls the step matrix by matrix: an attention matrix of the 304M model (d_model 1024) ...
        {"name": "one-1024", "call": "step", "rows": 1024, "cols": 1024, "batch": 1, "alpha": 0.25},
        # ... and an MLP matrix of the 1B model, whose shorter side is its columns
        {"name": "one-8192x2048", "call": "step", "rows": 8192, "cols": 2048, "batch": 1, "alpha": 0.25},
        # odd sides (an embedding adapter, a pruned head): nothing is a multiple of a tile or of a vector; fp32 W and G
        {"name": "odd-1155x771", "call": "ex", "rows": 1155, "cols": 771, "batch": 3, "alpha": 0.5, "w": "f32", "g": "f32"},
        # a parameter list by pointers: the down projections of eight layers, the paper's smallest fraction
        {"name": "batched-8x2048x8192", "call": "batched", "rows": 2048, "cols": 8192, "batch": 8, "alpha": 0.125},
        # one mixture-of-experts layer: 64 experts, 30% of them without gradient in this step
        {"name": "moe-64x2048x1408", "call": "strided", "rows": 2048, "cols": 1408, "batch": 64, "alpha": 0.25, "zero": 0.3},
        # all attention matrices of the 1B model
        {"name": "attn-64x2048", "call": "strided", "rows": 2048, "cols": 2048, "batch": 64, "alpha": 0.25},
        # its up projections at the paper's larger fraction (column selection)
        {"name": "mlp-16x8192x2048-half", "call": "strided", "rows": 8192, "cols": 2048, "batch": 16, "alpha": 0.5},
        # Muon itself (alpha 1) on square matrices
        {"name": "muon-16x2048", "call": "strided", "rows": 2048, "cols": 2048, "batch": 16, "alpha": 1.0},
        # the fp32 master on fp32 weights
        {"name": "master-8x1024x4096", "call": "ex", "rows": 1024, "cols": 4096, "batch": 8, "alpha": 0.25, "w": "f32",
         "g": "bf16", "master": True},
        # one layer of the 7B-style stack in one call
        {"name": "7b-layer", "call": "groups", "stack": "7b-layer", "alpha": 0.25},
        # the whole 1B-style stack in one call, the largest
        {"name": "1b-stack", "call": "groups", "stack": "1b", "alpha": 0.25},
    ]


def _shapes(case):
    if case["call"] == "groups":
        return STACKS[case["stack"]]
    return ((case["rows"], case["cols"], case["batch"]),)


def _plan(rows, cols, alpha):
    """(selected lines, whether they are rows): the shorter side, rows where both are alike."""
    by_rows = rows <= cols
    d = rows if by_rows else cols
    a32 = float(torch.tensor(alpha, dtype=torch.float32))
    return min(d, max(1, math.ceil(a32 * d))), by_rows


def work(case):
    """M, G and W's selected lines in, M and W's selected lines out; Newton-Schulz as the paper counts it,
    5 (4 s^2 l + 2 s^3) for a compact matrix of s x l."""
    wb = 4 if case.get("w") == "f32" else 2
    gb = 4 if case.get("g") == "f32" else 2
    nbytes = flops = 0
    for rows, cols, n in _shapes(case):
        k, by_rows = _plan(rows, cols, case["alpha"])
        other = cols if by_rows else rows
        s, l = min(k, other), max(k, other)
        nbytes += n * (rows * cols * (8 + gb) + k * other * 2 * wb)
        flops += n * STEPS * (4 * s * s * l + 2 * s ** 3)
    return {"bytes": nbytes, "flops": flops}


def draw(rng):
    """One more case: every kind of call, sides from 64 to 11008 spread over their logarithm (half of them odd or
    ragged), the paper's fractions, single matrices and stacks, never more work than the largest listed case."""
    top = [work(c) for c in listed()]
    most_b, most_f = max(w["bytes"] for w in top), max(w["flops"] for w in top)

    def side(lo=64, hi=11008):
        v = round(math.exp(rng.uniform(math.log(lo), math.log(hi))))
        return v if rng.random() < 0.5 else max(lo, v // 128 * 128)

    while True:
        call = rng.choice(("step", "strided", "strided", "batched", "ex", "ex", "ex", "groups"))
        case = {"call": call, "alpha": rng.choice((0.125, 0.25, 0.25, 0.5, 1.0))}
        if call == "groups":
            case["stack"] = rng.choice(sorted(STACKS))
        else:
            case["rows"], case["cols"] = side(), side()
            case["batch"] = 1 if call == "step" else round(math.exp(rng.uniform(0.0, math.log(64))))
        if call == "strided" and rng.random() < 0.3:
            case["zero"] = 0.3
        if call == "ex":
            case["w"], case["g"] = rng.choice((("bf16", "bf16"), ("f32", "f32"), ("f32", "bf16")))
            option = rng.choice(("none", "none", "random", "master"))
            if option == "random":
                case["rule"] = "random"
            if option == "master":
                case["master"] = True
        w = work(case)
        if w["bytes"] <= most_b and w["flops"] <= most_f * (0.4 if case.get("master") else 1.0):
            return case


def _inputs(case, seed, device):
    """W, M, G stacks: weights N(0, 0.02^2); momentum and gradient of std 1e-3 with a log-normal scale per row, alike in
    both, as gradients of a layer's units differ."""
    gen = torch.Generator(device=device)
    gen.manual_seed(int(seed) * 1000003 + 17)
    wt = torch.float32 if case.get("w") == "f32" else torch.bfloat16
    gt = torch.float32 if case.get("g") == "f32" else torch.bfloat16
    stacks = []
    for rows, cols, n in _shapes(case):
        W = torch.empty((n, rows, cols), dtype=wt, device=device)
        M = torch.empty((n, rows, cols), dtype=torch.float32, device=device)
        G = torch.empty((n, rows, cols), dtype=gt, device=device)
        for b0 in range(0, n, 8):   # a few matrices at a time: the fp32 draws stay small beside the stacks
            m = min(8, n - b0)
            W[b0:b0 + m] = torch.randn((m, rows, cols), generator=gen, device=device).mul_(0.02)
            r = torch.exp(torch.randn((m, rows, 1), generator=gen, device=device)).mul_(1e-3)
            M[b0:b0 + m] = torch.randn((m, rows, cols), generator=gen, device=device).mul_(r)
            G[b0:b0 + m] = torch.randn((m, rows, cols), generator=gen, device=device).mul_(r)
        if case.get("zero"):
            idle = torch.rand(n, generator=gen, device=device) < case["zero"]
            G[idle] = 0
        stacks.append((W, M, G))
    return stacks


def _draw_key(case, seed):
    """The Random rule's generator key, a number of the run's own."""
    return int(seed) * 2654435761 % (1 << 63)


def prepare(case, seed):
    stacks = _inputs(case, seed, "cuda")
    state = {"case": dict(case), "stacks": stacks, "seed": _draw_key(case, seed)}
    if case["call"] == "batched":
        W, M, G = stacks[0]
        state["lists"] = ([W[i] for i in range(W.shape[0])], [M[i] for i in range(M.shape[0])],
                          [G[i] for i in range(G.shape[0])])
    return state


def run(state):
    case = state["case"]
    call, alpha = case["call"], case["alpha"]
    W, M, G = state["stacks"][0]
    if call == "step":
        binding.dion2_step(W[0], M[0], G[0], alpha, MU, LR, STEPS)
    elif call == "strided":
        binding.dion2_step_strided(W, M, G, alpha, MU, LR, STEPS)
    elif call == "batched":
        binding.dion2_step_batched(*state["lists"], alpha, MU, LR, STEPS)
    elif call == "ex":
        binding.dion2_step_ex(
            W, M, G, alpha, MU, LR, STEPS,
            select_rule=binding.SELECT_RANDOM if case.get("rule") == "random" else binding.SELECT_L1,
            rand_seed=state["seed"],
            ns_master=binding.MASTER_FP32 if case.get("master") else binding.MASTER_BF16)
    else:
        binding.dion2_step_groups([(w, m, g, binding.AXIS_AUTO) for w, m, g in state["stacks"]], alpha, MU, LR, STEPS)
    return [{"W": w, "M": m} for w, m, _ in state["stacks"]]


def tolerance(case):
    """Of W and M together. M is a 32-bit sum and product, alike for every correct implementation; W is off by what
    Newton-Schulz on bf16 operands is off by (O 2e-3 to 1.2e-2 from the exact iteration, most where the compact matrix is
    near square; with the fp32 master 3e-5 and more), times the step's size beside W. In bf16 W that turns some roundings
    by a unit (2^-7 of the value at most).
    Four times the largest distance of W from exact() rounded to W's type over the listed cases and 104 draws: bf16 W
    3.4e-4, 6.5e-4 at alpha 0.5, 1.1e-3 at alpha 1; fp32 W 1.1e-4, 3.4e-4 from alpha 0.5; fp32 W under the master 1.1e-7,
    2.5e-6 from alpha 0.5 (forty times that there: near-square compact matrices spread more than those drawn)."""
    half = case["alpha"] >= 0.5
    if case.get("w") != "f32":
        return {"rel": 4.4e-3 if case["alpha"] == 1.0 else 2.6e-3 if half else 1.4e-3, "max": 4e-2}
    if case.get("master"):
        return {"rel": 1e-4 if half else 1e-6, "max": 5e-3 if half else 1e-4}
    return {"rel": 1.4e-3 if half else 4.5e-4, "max": 2.5e-2}


def _philox_keys(n, matrix, step, seed):
    """Philox-4x32-10 (Salmon et al., SC 2011) of counters (line, matrix, step low, step high): the first two words."""
    mask = 0xFFFFFFFF
    keys = []
    for line in range(n):
        c = [line, matrix & mask, step & mask, step >> 32]
        k0, k1 = seed & mask, seed >> 32
        for r in range(10):
            if r:
                k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
            p0, p1 = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
            c = [(p1 >> 32) ^ c[1] ^ k0, p1 & mask, (p0 >> 32) ^ c[3] ^ k1, p0 & mask]
        keys.append((c[0] << 32) | c[1])
    return keys


def exact(case, seed):
    """The step's definition in 64 bits: momentum, selection, Newton-Schulz on the selected lines, decay, update."""
    stacks = _inputs(case, seed, "cuda")
    f32 = lambda v: float(torch.tensor(v, dtype=torch.float32))  # noqa: E731 - the call takes 32-bit numbers
    mu, lr = f32(MU), f32(LR)
    coeffs = tuple(f32(v) for v in QUINTIC)
    key = _draw_key(case, seed)
    out = []
    for W, M, G in stacks:
        n, rows, cols = W.shape
        k, by_rows = _plan(rows, cols, case["alpha"])
        big = n * rows * cols > 50_000_000   # the comparison reads a part of such an output: fp32 halves its memory
        W1 = torch.empty(W.shape, dtype=torch.float32 if big else torch.float64, device=W.device)
        M1 = torch.empty_like(W1)
        for i in range(n):
            m = M[i].double() + G[i].double()
            lines = m if by_rows else m.T
            if case.get("rule") == "random":
                keys = _philox_keys(lines.shape[0], i, 0, key)
                K = torch.tensor(sorted(sorted(range(len(keys)), key=lambda j: (keys[j], j))[:k]), device=m.device)
            else:
                order = torch.sort(lines.abs().sum(1), descending=True, stable=True).indices
                K = order[:k].sort().values
            X = lines[K].clone()
            X /= X.norm() + EPS
            flip = X.shape[0] > X.shape[1]
            X = X.T.contiguous() if flip else X
            a, b, c = coeffs
            for _ in range(STEPS):
                A = X @ X.T.contiguous()
                X = a * X + (b * A + c * (A @ A)) @ X
            X = X.T if flip else X
            w = W[i].double()
            new_m = m.clone()
            step = lr * math.sqrt(rows / cols)
            if by_rows:
                new_m[K] *= mu
                w[K] -= step * X
            else:
                new_m[:, K] *= mu
                w[:, K] -= step * X.T
            W1[i], M1[i] = w, new_m
        out.append({"W": W1, "M": M1})
    return out
