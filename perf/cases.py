"""The work whose speed counts: calls of libpisa as a program that replaces its attention by it makes them.

`listed()` holds the cases, `draw()` further ones of the same ranges.  A case names an entry point
and its sizes:

    forward    pisa_forward, statistics -> selection -> attention in one call, with the output, the
               log-sum-exp (where asked for) and the workspace held by the caller, as a layer that runs
               once per denoising step keeps them
    steps      the same path as separate library calls (forward_in_steps), which is how the
               covariance-aware score, its norms and the ablation variants are reached
    dense      dense_attention: the layers and denoising steps that stay dense

Inputs follow the recipe of the repository's workloads, made on the device: q, k = N(0,1) plus a smooth
field shared by q and k over the latent grid (sinusoids per channel), v = N(0,1); a sequence without a
grid gets an offset per 64-token block shared by q and k instead.
"""
import math

import torch

import paper_2602_01077_amd as pisa

_DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}
_NORMS = {"spectral": pisa.PISA_NORM_SPECTRAL, "frobenius": pisa.PISA_NORM_FROBENIUS,
          "frobenius-fast": pisa.PISA_NORM_FROBENIUS_FAST}


def _case(name, entry, batch, heads, length, d, dtype="bf16", block=64, sparsity=0.85, grid="", text=0, lse=False,
          norm="", variant="hybrid"):
    """grid: "t,h,w" or "h,w" of the latent tokens ("" = none); text: plain tokens ahead of it.
    norm: of the covariance-aware score ("" = plain score).  variant: hybrid | zeroth | sparse."""
    return {"name": name, "entry": entry, "batch": batch, "heads": heads, "length": length, "d": d, "dtype": dtype,
            "block": block, "sparsity": sparsity, "grid": grid, "text": text, "lse": lse, "norm": norm,
            "variant": variant}


def listed():
    return [
        # the smallest call: 16 blocks of 64, two heads, where launches and latency are all there is
        _case("tiny-fp32", "forward", 1, 2, 1024, 64, dtype="fp32", sparsity=0.75),
        # a short ragged bf16 sequence (last block 40 rows)
        _case("short-ragged", "forward", 1, 2, 1000, 128, sparsity=0.8, lse=True),
        # the fp32 build on an image-sized sequence of odd length (a debugging or reference run of a layer)
        _case("image-fp32", "forward", 1, 8, 4500, 128, dtype="fp32", lse=True),
        # one image layer: 512 text tokens, then a 64 x 64 latent grid
        _case("flux", "forward", 1, 24, 4608, 128, grid="64,64", text=512),
        # the same layer with the covariance-aware score of the image setting: the operator norm (the default) ...
        _case("flux-cov-spectral", "steps", 1, 24, 4608, 128, grid="64,64", text=512, norm="spectral"),
        # ... and the fast Frobenius kind, the one that pays at this size
        _case("flux-cov-fast", "steps", 1, 24, 4608, 128, grid="64,64", text=512, norm="frobenius-fast"),
        # the layers of an image model that stay dense
        _case("flux-dense", "dense", 1, 24, 4608, 128, grid="64,64", text=512, lse=True),
        # a dense layer or denoising step of a 480p video model (21 x 30 x 52 latents, 12 heads)
        _case("video-480p-dense", "dense", 1, 12, 32760, 128, grid="21,30,52"),
        # 64-channel heads at a long sequence
        _case("head-dim-64", "forward", 1, 40, 32768, 64, grid="11,45,80"),
        # the headline layer: 720p video, 21 x 45 x 80 latents, last block 16 rows
        _case("wan", "forward", 1, 40, 75600, 128, grid="21,45,80"),
        # the same layer at block 128 (the block-size axis of the sweep)
        _case("wan-block128", "forward", 1, 40, 75600, 128, block=128, grid="21,45,80"),
        # the longest: 33 x 45 x 80 latents and 256 text tokens behind them, 90 % sparsity, separate calls
        _case("hunyuan-steps", "steps", 1, 24, 119056, 128, sparsity=0.9, grid="33,45,80"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["forward", "forward", "forward", "forward", "steps", "cov", "dense", "fp32"])
    d = rng.choice([128, 128, 128, 64])
    block = rng.choice([64, 64, 64, 128])
    sparsity = rng.choice([0.5, 0.75, 0.8, 0.85, 0.85, 0.875, 0.9, 0.95])
    lse = rng.random() < 0.3
    kw = dict(d=d, block=block, sparsity=sparsity, lse=lse)
    if family == "fp32":                      # both directions of the path in fp32: sparse and dense
        entry = rng.choice(["forward", "forward", "steps", "dense"])
        case = _case("", entry, rng.choice([1, 2]), rng.randint(1, 8), _log_int(rng, 200, 4608), dtype="fp32", **kw)
    elif family == "cov":                     # image layers with the covariance-aware score
        norm = rng.choice(["spectral", "frobenius", "frobenius-fast"])
        case = _case("", "steps", rng.choice([1, 2]), rng.randint(4, 24), _log_int(rng, 1000, 4608), norm=norm, **kw)
    elif family == "dense":
        length = _log_int(rng, 500, 32768)
        case = _case("", "dense", rng.choice([1, 2]), rng.randint(2, 24), length, **kw)
    else:
        length = _log_int(rng, 500, 120000)
        case = _case("", family, rng.choice([1, 1, 2]), rng.randint(2, 40), length,
                     variant=rng.choice(["hybrid", "zeroth", "sparse"]) if family == "steps" else "hybrid", **kw)
    if case["dtype"] == "bf16" and rng.random() < 0.6 and case["length"] > 4000:
        frame = 45 * 80 if case["length"] > 12000 else 32 * 32
        case["grid"] = "%d,%s" % (max(1, case["length"] // frame), "45,80" if frame == 3600 else "32,32")
        case["text"] = 0 if frame == 3600 else case["length"] % frame
    limit = work(listed()[9])                 # the headline layer; fp32 has an eighth of the bf16 rate at most
    if case["dtype"] == "fp32" or case["norm"]:
        limit = work(listed()[4])             # kept to the size of an image layer
    while True:
        w = work(case)
        over = max(w["bytes"] / limit["bytes"], w["flops"] / limit["flops"])
        if over <= 1.0 or case["heads"] * case["batch"] == 1:
            return case
        if case["batch"] > 1:
            case["batch"] = 1
        else:
            case["heads"] = max(1, min(case["heads"] - 1, int(case["heads"] / over)))


def _field(case, gen, device):
    """[length, d] smooth field of one head (fp32), zero outside the grid."""
    dims = [int(x) for x in case["grid"].split(",")]
    L, d = case["length"], case["d"]
    n = min(math.prod(dims), L - case["text"])
    t = torch.arange(n, device=device)
    coords = []
    for g in reversed(dims):
        coords.append((t % g).float())
        t = t // g
    freq = torch.rand(4, len(dims), d, generator=gen, device=device) * (0.2 * 2.0 * math.pi)
    phase = torch.rand(4, d, generator=gen, device=device) * (2.0 * math.pi)
    out = torch.zeros(L, d, device=device)
    part = out[case["text"]:case["text"] + n]
    for m in range(4):
        arg = phase[m].expand(n, d).clone()
        for a, x in enumerate(reversed(coords)):
            arg.addcmul_(x[:, None], freq[m, a][None, :])
        part += arg.sin_()
    return out


def _inputs(case, seed, device):
    gen = torch.Generator(device=device).manual_seed(seed)
    b, h, L, d = case["batch"], case["heads"], case["length"], case["d"]
    q, k, v = (torch.empty(b, h, L, d, dtype=_DTYPES[case["dtype"]], device=device) for _ in range(3))
    for i in range(b * h):
        if case["grid"]:
            shared = _field(case, gen, device)
        else:
            off = 0.5 * torch.randn(-(-L // 64), d, generator=gen, device=device)
            shared = off.repeat_interleave(64, dim=0)[:L]
        for dst in (q, k):
            dst.view(b * h, L, d)[i] = torch.randn(L, d, generator=gen, device=device) + shared
        v.view(b * h, L, d)[i] = torch.randn(L, d, generator=gen, device=device)
    return q, k, v


def prepare(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    q, k, v = _inputs(case, seed, device)
    state = {"case": case, "q": q, "k": k, "v": v}
    if case["entry"] != "steps":
        state["out"] = torch.empty_like(q)
        state["lse"] = torch.empty(q.shape[:3], dtype=torch.float32, device=device) if case["lse"] else None
    if case["entry"] == "forward":
        shape = pisa.make_shape(q, case["block"])
        k_top = pisa.topk_count(pisa.num_blocks(case["length"], case["block"]), case["sparsity"])
        state["shape"], state["k_top"] = shape, k_top
        state["workspace"] = torch.empty(pisa.forward_workspace_bytes(shape, k_top), dtype=torch.uint8, device=device)
    return state


def run(state):
    case, q, k, v = state["case"], state["q"], state["k"], state["v"]
    if case["entry"] == "forward":
        out, lse = pisa.forward(state["shape"], q, k, v, state["k_top"], out=state["out"], lse=state["lse"],
                                workspace=state["workspace"])
        return {"out": out} if lse is None else {"out": out, "lse": lse}
    if case["entry"] == "dense":
        out, lse = pisa.dense_attention(q, k, v, case["block"], out=state["out"], lse=state["lse"])
        return {"out": out} if lse is None else {"out": out, "lse": lse}
    res = pisa.forward_in_steps(q, k, v, case["block"], case["sparsity"], first_order=case["variant"] == "hybrid",
                                approximate=case["variant"] != "sparse", want_lse=case["lse"],
                                covariance_aware=bool(case["norm"]),
                                norm=_NORMS[case["norm"] or "spectral"], hbar_from_stats=case["norm"] == "frobenius-fast")
    out = {"out": res["out"], "idx": res["idx"], "hsum": res["stats"]["hsum"]}
    if case["lse"]:
        out["lse"] = res["lse"]
    if case["norm"]:
        out["log_m"] = res["log_m"]
    return out


def work(case):
    """Compulsory bytes (q, k, v in, output out) and operations (4 d per query-key pair attended exactly or
    through a centroid, 2 d^2 per token for the block moments and for the first-order term, the pooled
    scores; the spectral norm: one product with D and one with its transpose)."""
    L, d, B = case["length"], case["d"], case["block"]
    heads = case["batch"] * case["heads"]
    size = 4 if case["dtype"] == "fp32" else 2
    n = -(-L // B)
    k_top = n if case["entry"] == "dense" else n - math.floor(case["sparsity"] * n + 1e-9)
    out_bytes = L * d * size + (4 * L if case["lse"] else 0)
    if case["entry"] == "dense":
        return {"bytes": heads * (3 * L * d * size + out_bytes), "flops": heads * 4 * L * L * d}
    flops = 4 * L * d * min(k_top * B, L) + 2 * n * n * d + 2 * L * d * d
    if case["variant"] != "sparse":
        flops += 4 * L * d * n
    if case["variant"] == "hybrid":
        flops += 2 * L * d * d
    if case["entry"] == "steps":              # outputs beside the attention: index rows, hsum (and log M)
        out_bytes += 4 * n * k_top + 4 * d * d
    if case["norm"]:
        out_bytes += 8 * n
        flops += 2 * n * d * d + (4 * n * d * d if case["norm"] == "spectral" else 0)
    return {"bytes": heads * (3 * L * d * size + out_bytes), "flops": heads * flops}


def tolerance(case):
    # About four times the distance to a 64-bit evaluation of the same formulas: bf16 (output and
    # probabilities rounded once each) 2.3e-3 at the flux sizes, fp32 1.1e-6 at the image-fp32 sizes.
    # Whole values: the index rows, which may differ only where two pooled scores agree to rounding.
    return {"rel": 5e-6 if case["dtype"] == "fp32" else 1e-2, "differ": 1e-4}
