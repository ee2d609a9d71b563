"""What is timed of this library: calls of its public entry points, at the sizes and options they are used with.

A case is a dict of plain values.  `kind` says which call it stands for:

  forward4 / forward8   one layer's forward on bf16 activations (rotate, quantise, GEMM, dequantise), the weight
                        prepared beforehand and the workspace kept, as a model that runs layer after layer does
  shared4               one rotated and quantised activation that feeds several layers (query, key and value
                        projections of the same tokens): convrot_rotquant_act once, then one GEMM per layer
  prepare4 / prepare8   the offline pass over a weight, once per layer of a model that is loaded

M is the number of tokens, K the layer's input width, N its output width, g the rotation group.
"""
import math

import torch

from paper_2512_03673_amd import binding as cr

GROUPS = (4, 16, 64, 256, 1024)
FORWARDS = ("forward4", "forward8")
M_MAX, K_MAX, N_MAX = 16896, 15360, 12288
MOST_PRODUCTS = 16896 * 12288 * 3072       # multiply-adds of the largest listed case
MOST_PREPARED = 12288 * 15360              # weights of the largest layer
PAD = 0                                    # value of the code bytes past a matrix's last row, which no call writes


def listed():
    return [
        # A conditioning vector's layer: one row, all time goes to launches and to reading the weight.
        {"name": "one_row", "kind": "forward4", "M": 1, "K": 3072, "N": 9216, "g": 16, "x": "normal", "bias": True},
        # The small configuration of the benchmark.
        {"name": "tiny", "kind": "forward4", "M": 256, "K": 1024, "N": 1024, "g": 16, "x": "normal", "bias": False},
        # A small layer with no size a multiple of any tile, as the random-shape tests draw them.
        {"name": "ragged", "kind": "forward4", "M": 389, "K": 1056, "N": 437, "g": 4, "x": "normal", "bias": True},
        # The 512 text tokens alone, at the paper's default group.
        {"name": "text_up", "kind": "forward4", "M": 512, "K": 3072, "N": 12288, "g": 256, "x": "normal", "bias": True},
        # The headline layer of the benchmark: 4096 image and 512 text tokens.
        {"name": "mlp_up", "kind": "forward4", "M": 4608, "K": 3072, "N": 12288, "g": 16, "x": "normal", "bias": False},
        {"name": "mlp_down", "kind": "forward4", "M": 4608, "K": 12288, "N": 3072, "g": 16, "x": "halfnormal", "bias": False},
        # Query, key and value of the same tokens.
        {"name": "qkv_shared", "kind": "shared4", "M": 4608, "K": 3072, "N": 3072, "layers": 3, "g": 64, "x": "normal", "bias": True},
        # The fused-width output layer at the group the paper uses for its high-outlier layers.
        {"name": "fused_out", "kind": "forward4", "M": 4608, "K": 15360, "N": 3072, "g": 1024, "x": "halfnormal", "bias": True},
        # High-resolution tokens: the largest.
        {"name": "hires_down", "kind": "forward4", "M": 16896, "K": 12288, "N": 3072, "g": 16, "x": "halfnormal", "bias": False},
        # The 8-bit layers of a mixed-precision model: a small one and the headline layer.
        {"name": "small8", "kind": "forward8", "M": 77, "K": 3072, "N": 3072, "g": 64, "x": "normal", "bias": True},
        {"name": "mlp_up8", "kind": "forward8", "M": 4608, "K": 3072, "N": 12288, "g": 256, "x": "normal", "bias": True},
        # A layer's weight as a model is loaded.
        {"name": "prepare", "kind": "prepare4", "N": 12288, "K": 3072, "g": 256},
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges: any group, sizes over their logarithm, odd ones among them."""
    kind = rng.choice(("forward4",) * 5 + ("forward8",) * 2 + ("shared4", "prepare4", "prepare8"))
    g = rng.choice(GROUPS)
    step = max(g, 32)                       # K is a multiple of the group and of 32
    case = {"kind": kind, "g": g}
    while True:
        M, N = _spread(rng, 1, M_MAX), _spread(rng, 64, N_MAX)
        K = max(1, round(_spread(rng, 64, K_MAX) / step)) * step
        if rng.random() < 0.5:              # widths of real layers are round numbers; token counts need not be
            N = max(1, round(N / 64)) * 64
        if kind.startswith("prepare"):
            if 2 ** 16 <= N * K <= MOST_PREPARED:
                case.update(N=N, K=K)
                return case
            continue
        layers = rng.choice((2, 3)) if kind == "shared4" else 1
        # an 8-bit multiply-add costs about two 4-bit ones
        if M * N * K * layers * (2 if kind == "forward8" else 1) > MOST_PRODUCTS:
            continue
        case.update(M=M, K=K, N=N, x=rng.choice(("normal", "halfnormal")), bias=rng.random() < 0.5)
        if kind == "shared4":
            case["layers"] = layers
        return case


def _log_uniform(gen, lo, hi, n):
    u = torch.rand(n, generator=gen, device="cuda")
    return torch.exp(math.log(lo) + u * math.log(hi / lo))


def _activation(case, gen):
    """Tokens with outlier channels and outlier tokens (the recipe of workloads.py, drawn on the GPU)."""
    M, K = case["M"], case["K"]
    x = torch.randn(M, K, generator=gen, device="cuda")
    if case["x"] == "halfnormal":           # behind a GELU
        x.abs_()
    cols, rows = round(0.01 * K), round(0.005 * M)
    if cols:
        x[:, torch.randperm(K, generator=gen, device="cuda")[:cols]] *= _log_uniform(gen, 20.0, 100.0, cols)
    if rows:
        x[torch.randperm(M, generator=gen, device="cuda")[:rows]] *= _log_uniform(gen, 10.0, 40.0, rows)[:, None]
    return x.to(torch.bfloat16)


def _weight(case, gen):
    return (torch.randn(case["N"], case["K"], generator=gen, device="cuda") * 0.02).to(torch.bfloat16)


def _bias(case, gen):
    return (torch.randn(case["N"], generator=gen, device="cuda") * 0.1).to(torch.bfloat16) if case["bias"] else None


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind, K, N, g = case["kind"], case["K"], case["N"], case["g"]
    state = {"kind": kind, "g": g}
    if kind.startswith("prepare"):
        size = cr.packed_bytes if kind == "prepare4" else cr.packed_bytes8
        state.update(W=_weight(case, gen), Wq=torch.full((size(N, K),), PAD, dtype=torch.uint8, device="cuda"))
        return state
    prep = cr.convrot_prepare_weight8 if kind == "forward8" else cr.convrot_prepare_weight
    space = cr.workspace_bytes8 if kind == "forward8" else cr.workspace_bytes
    state["layers"] = [(*prep(_weight(case, gen), g), _bias(case, gen)) for _ in range(case.get("layers", 1))]
    state["X"] = _activation(case, gen)
    if kind == "shared4":
        state["Xq"] = torch.full((cr.packed_bytes(case["M"], K),), PAD, dtype=torch.uint8, device="cuda")
    else:
        state["workspace"] = torch.empty(space(case["M"], K), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    kind, g = state["kind"], state["g"]
    if kind == "prepare4":
        return cr.convrot_prepare_weight(state["W"], g, Wq=state["Wq"])
    if kind == "prepare8":
        return cr.convrot_prepare_weight8(state["W"], g, Wq=state["Wq"])
    X = state["X"]
    if kind == "shared4":
        Xq, x_scale = cr.convrot_rotquant_act(X, g, Xq=state["Xq"])
        return [Xq, x_scale] + [cr.convrot_w4a4_gemm_dequant(Xq, x_scale, Wq, w_scale, X.shape[1], bias=bias)
                                for Wq, w_scale, bias in state["layers"]]
    forward = cr.convlinear8bit_forward if kind == "forward8" else cr.convlinear4bit_forward
    (Wq, w_scale, bias), = state["layers"]
    return forward(X, Wq, w_scale, g, workspace=state["workspace"], bias=bias)


def work(case):
    """Inputs read once, outputs written once; a 4-bit code matrix takes 0.75 bytes a code, an 8-bit one 1."""
    kind, K, N, g = case["kind"], case["K"], case["N"], case["g"]
    code = 1.0 if kind.endswith("8") else 0.75
    rotate = 2 * math.log(g, 4)             # a radix-4 step takes two operations an element and digit (7 for 4)
    if kind.startswith("prepare"):
        return {"bytes": N * K * (2 + code) + 4 * N, "flops": N * K * rotate}
    M, layers = case["M"], case.get("layers", 1)
    nbytes = 2 * M * K + layers * (code * N * K + 4 * N + (2 * N if case["bias"] else 0) + 2 * M * N)
    if kind == "shared4":
        nbytes += code * M * K + 4 * M      # the codes are an output of the shared call
    return {"bytes": nbytes, "flops": 2 * M * N * K * layers + M * K * rotate}


def tolerance(case):
    """About four times what 192 rows of each listed case (and of drawn ones) differ by from the same path in 64 bits
    (the double-precision oracle).

    Codes and sums of products are whole numbers, so a difference comes from the rotation's 32-bit sums: a scale one
    or two steps off, which moves some bf16 results by one step (relative to the whole 2e-6 to 3e-5 at 4 bits, 8e-5 at
    8, 3.5e-4 at g = 1024), and, from the largest groups' sums on, a code on a tie that falls the other way (11 in
    118 million at g = 1024, none seen below; it moves a result by up to 0.035 of the results' root mean square).
    """
    g = case["g"]
    differ = 0.0 if g <= 16 else 1e-6 if g <= 256 else 2e-5
    if case["kind"].startswith("prepare"):
        return {"rel": 5e-7, "max": 1e-6, "differ": differ}        # the scales: two steps of fp32
    return {"rel": 1.4e-3 if g == 1024 else 3e-4, "max": 0.14 if g == 1024 else 0.03, "differ": differ}
