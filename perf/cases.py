"""The calls whose speed this library is judged by, as a program that serves or produces CCQ weights makes them.

Four kinds of case, all through the public functions of `paper_2507_07145_amd.binding`:

  gemm      y = x W_dq^T for M activation rows: decode steps (M = 1 .. a few dozen), batched decode, prefill (hundreds to
            thousands of rows), in every weight format and both scale modes.  `call` says how the program calls it:
            "new" lets the call make its own output and workspace, "kept" passes buffers that a serving loop holds,
            "static" is the entry point that needs no workspace.
  grouped   the product of a mixture-of-experts layer: T tokens, each routed to `topk` of E experts; `host` says whether
            the program has the expert offsets on the host too.
  quantize  an fp32 matrix to packed weights on the GPU.
  load      packed weights in the paper's order on the host (a checkpoint) to device-resident weights.
"""
import math

import numpy as np
import torch

from paper_2507_07145_amd import binding as ccq

FORMATS = ("narrow", "wide", "mix", "h16")
GROUP = 64
CODE_BYTES = {"narrow": 16, "wide": 22, "h16": 20}     # of a 64-weight group
WIDE_SHARE = 0.25                                      # of the groups of a mix

# the largest of each kind: what draw() stays below
MAX_GEMM_MKN = 2048 * 7168 * 18432
MAX_GEMM_KN = 8192 * 28672
MAX_GROUPED_EKN = 64 * 7168 * 2048
MAX_QUANTIZE_KN = 8192 * 8192
MAX_LOAD_KN = 4096 * 11008


def listed():
    return [
        # the smallest layer of the test configurations, one token: launch and call overhead
        {"name": "gemv-1024", "kind": "gemm", "fmt": "narrow", "mode": 0, "M": 1, "K": 1024, "N": 1024, "call": "new"},
        # one token through a square projection of a large model: the benchmark line
        {"name": "gemv-8192", "kind": "gemm", "fmt": "narrow", "mode": 0, "M": 1, "K": 8192, "N": 8192, "call": "kept"},
        # a few sequences through a down projection whose K has no equal split, at 2.06 bits per weight
        {"name": "rows4-11008", "kind": "gemm", "fmt": "narrow", "mode": 1, "M": 4, "K": 11008, "N": 4096, "call": "new"},
        # a decode batch from a loop that may not allocate
        {"name": "rows16-8192", "kind": "gemm", "fmt": "narrow", "mode": 0, "M": 16, "K": 8192, "N": 8192, "call": "static"},
        # one token on weights that mix the 2-bit and the 2.75-bit format group by group
        {"name": "gemv-mix-28672", "kind": "gemm", "fmt": "mix", "mode": 0, "M": 1, "K": 8192, "N": 28672, "call": "kept"},
        # a large decode batch (or a short prompt) on 2.75-bit weights
        {"name": "rows64-wide-28672", "kind": "gemm", "fmt": "wide", "mode": 0, "M": 64, "K": 8192, "N": 28672, "call": "new"},
        # a prompt of odd length on hybrid-word weights, every dimension ragged
        {"name": "prompt-h16-ragged", "kind": "gemm", "fmt": "h16", "mode": 1, "M": 777, "K": 7232, "N": 5001, "call": "new"},
        # a full prefill chunk through an up projection
        {"name": "prefill-2048", "kind": "gemm", "fmt": "narrow", "mode": 0, "M": 2048, "K": 7168, "N": 18432, "call": "new"},
        # a decode batch through the up projections of a mixture-of-experts layer
        {"name": "moe-decode-64", "kind": "grouped", "fmt": "narrow", "mode": 0, "E": 64, "topk": 8, "T": 64, "K": 7168, "N": 2048, "host": True},
        # a prompt through the down projections of the same layer
        {"name": "moe-prompt-512", "kind": "grouped", "fmt": "narrow", "mode": 0, "E": 64, "topk": 8, "T": 512, "K": 2048, "N": 7168, "host": True},
        # making the weights of one large projection
        {"name": "quantize-8192", "kind": "quantize", "fmt": "narrow", "mode": 0, "K": 8192, "N": 8192},
        # a projection's weights from a checkpoint
        {"name": "load-11008", "kind": "load", "fmt": "narrow", "mode": 0, "K": 4096, "N": 11008},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, k_hi, n_lo, n_hi, most):
    """K a multiple of the group, N any number (every other one a multiple of 16, as most layers have it)."""
    while True:
        K, N = GROUP * _log(rng, 8, k_hi // GROUP), _log(rng, n_lo, n_hi)
        if rng.random() < 0.5:
            N = max(16, N // 16 * 16)
        if K * N <= most:
            return K, N


def draw(rng):
    kind = rng.choice(["gemm"] * 6 + ["grouped"] * 3 + ["quantize"] * 2 + ["load"])
    case = {"kind": kind, "fmt": rng.choice(FORMATS + ("narrow",)), "mode": rng.choice((0, 1))}
    if kind == "gemm":
        while True:
            K, N = _shape(rng, 28672, 1000, 28672, MAX_GEMM_KN)
            M = _log(rng, 1, 2048)
            if M * K * N <= MAX_GEMM_MKN:
                break
        calls = ["new", "kept"] + (["static"] if M <= 16 else [])
        case.update(M=M, K=K, N=N, call=rng.choice(calls))
    elif kind == "grouped":
        E = _log(rng, 8, 256)
        K, N = _shape(rng, 7168, 512, 7168, MAX_GROUPED_EKN // E)
        case.update(E=E, topk=8, T=_log(rng, 1, 512), K=K, N=N, host=rng.random() < 0.75)
    else:
        K, N = _shape(rng, 8192, 1000, 11008, MAX_QUANTIZE_KN if kind == "quantize" else MAX_LOAD_KN)
        case.update(K=K, N=N)
    return case


def _gen(seed, stream, device="cuda"):
    return torch.Generator(device=device).manual_seed((int(seed) * 16 + stream) & (2 ** 62 - 1))


def _formats(fmt):
    return {"narrow": [ccq.NARROW], "wide": [ccq.WIDE], "mix": [ccq.NARROW, ccq.WIDE], "h16": ccq.H16}[fmt]


def _wide_groups(G):
    return max(1, int(round(G * WIDE_SHARE)))


def _group_map(case, seed):
    if case["fmt"] != "mix":
        return None
    G = case["K"] // GROUP
    m = np.zeros(G, dtype=np.uint8)
    m[np.random.default_rng([seed, 7]).choice(G, size=_wide_groups(G), replace=False)] = 1
    return m


def _dense_weights(case, seed):
    """fp32 weights as a model has them, N(0, 0.02)."""
    return torch.randn(case["N"], case["K"], generator=_gen(seed, 0), device="cuda") * 0.02


def _canonical(case, seed, E=None):
    """Host arrays in the paper's order: random code bits (every pattern decodes), scales and Code Cluster parameters in
    the ranges that quantized weights have.  With E, a leading expert axis."""
    K, N, fmt, mode = case["K"], case["N"], case["fmt"], case["mode"]
    G, lead, g = K // GROUP, () if E is None else (E,), _gen(seed, 1)
    gf = _group_map(case, seed)
    wide = int(gf.sum()) if gf is not None else 0
    row = (G - wide) * 16 + wide * 22 if fmt == "mix" else G * CODE_BYTES[fmt]

    def uniform(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(lead + shape, generator=g, device="cuda")

    def fp16_bits(t):
        return t.half().view(torch.int16).cpu().numpy().view(np.uint16)

    a = {"codes": torch.randint(0, 256, lead + (N, row), generator=g, device="cuda", dtype=torch.uint8).cpu().numpy(), "group_fmt": gf}
    if mode == 0:
        a["scales"] = fp16_bits(torch.exp(uniform(math.log(1e-3), math.log(1e-1), N, G)))
    else:
        narrow = G - wide if fmt in ("narrow", "mix") else 0
        a["fields"] = torch.randint(0, 256, lead + (N, (narrow + 1) // 2), generator=g, device="cuda", dtype=torch.uint8).cpu().numpy() if narrow else None
        top = 1e-3 if fmt == "h16" else 1e-2
        a["super"] = fp16_bits(torch.exp(uniform(math.log(top / 100), math.log(top), N)))
    a["alpha"] = a["beta"] = None
    if fmt in ("narrow", "mix"):
        alpha = uniform(64.0, 128.0, N)
        beta = torch.floor(uniform(0.0, 1.0, N) * (32766.0 - 255.0 * alpha).clamp_min(0.0))
        a["alpha"], a["beta"] = alpha.cpu().numpy(), beta.cpu().numpy()
    return a


def _from_host(case, a, E=None):
    K, N, fmts = case["K"], case["N"], _formats(case["fmt"])
    if case["mode"] == 0:
        return ccq.Weight.from_canonical(K, N, fmts, a["codes"], a["scales"], a["alpha"], a["beta"], a["group_fmt"], experts=E)
    return ccq.Weight.from_canonical_compressed(K, N, fmts, a["codes"], a["fields"], a["super"], a["alpha"], a["beta"], a["group_fmt"], experts=E)


def _activations(rows, K, seed):
    return torch.randn(rows, K, generator=_gen(seed, 2), device="cuda").to(torch.bfloat16)


def _routing(T, E, topk, seed):
    """Every token to `topk` distinct experts; rows sorted by expert."""
    choice = np.argsort(np.random.default_rng([seed, 9]).random((T, E)), axis=1)[:, :topk].reshape(-1)
    order = np.argsort(choice, kind="stable")
    rows = (order // topk).astype(np.int32)
    offsets = np.zeros(E + 1, dtype=np.int32)
    np.cumsum(np.bincount(choice, minlength=E), out=offsets[1:])
    return rows, offsets


def prepare(case, seed):
    s = {"case": case}
    kind = case["kind"]
    if kind == "gemm":
        w = ccq.quantize(_dense_weights(case, seed), _formats(case["fmt"]), scale_mode=case["mode"], group_fmt=_group_map(case, seed))
        s.update(w=w, x=_activations(case["M"], case["K"], seed))
        if case["call"] != "new":
            s["out"] = torch.empty(case["M"], (case["N"] + 7) // 8 * 8, dtype=torch.bfloat16, device="cuda")[:, :case["N"]]
        if case["call"] == "kept":
            s["workspace"] = torch.empty(max(16, ccq.gemm_workspace_bytes(w.desc, case["M"])), dtype=torch.uint8, device="cuda")
        if case["call"] == "static" and ccq.gemm_workspace_bytes(w.desc, case["M"]) > ccq.load().ccq_gemm_static_max_workspace():
            s["case"] = dict(case, call="new")      # what a program does where the static entry point says no
    elif kind == "grouped":
        rows, offsets = _routing(case["T"], case["E"], case["topk"], seed)
        s.update(w=_from_host(case, _canonical(case, seed, case["E"]), case["E"]), x=_activations(case["T"], case["K"], seed),
                 rows=torch.from_numpy(rows).cuda(), offsets=torch.from_numpy(offsets).cuda(), offsets_host=offsets if case["host"] else None)
    elif kind == "quantize":
        s.update(W=_dense_weights(case, seed), group_fmt=_group_map(case, seed))
    else:
        s.update(arrays=_canonical(case, seed))
    return s


def _weight_arrays(w):
    named = {"codes": w.codes, "scales": w.scales, "alpha": w.alpha, "beta": w.beta, "super": w.ssup, "meta": w.meta}
    return {k: v for k, v in named.items() if v is not None}


def run(s):
    c = s["case"]
    if c["kind"] == "gemm":
        if c["call"] == "static":
            return ccq.gemm_static(s["w"], s["x"], s["out"])
        if c["call"] == "kept":
            return ccq.gemm(s["w"], s["x"], out=s["out"], workspace=s["workspace"])
        return ccq.gemm(s["w"], s["x"])
    if c["kind"] == "grouped":
        return ccq.grouped_gemm(s["w"], s["x"], s["rows"], s["offsets"], s["offsets_host"])
    if c["kind"] == "quantize":
        return _weight_arrays(ccq.quantize(s["W"], _formats(c["fmt"]), scale_mode=c["mode"], group_fmt=s["group_fmt"]))
    return _weight_arrays(_from_host(c, s["arrays"]))


def _stored_bytes(case):
    """Codes, scales and per-row parameters of one matrix."""
    K, N, fmt, mode = case["K"], case["N"], case["fmt"], case["mode"]
    G = K // GROUP
    wide = _wide_groups(G) if fmt == "mix" else 0
    row = (G - wide) * 16 + wide * 22 if fmt == "mix" else G * CODE_BYTES[fmt]
    narrow = G - wide if fmt in ("narrow", "mix") else 0
    row += 2 * G if mode == 0 else (narrow + 1) // 2 + 2
    return N * (row + (8 if narrow else 0))


def work(case):
    K, N, stored = case["K"], case["N"], _stored_bytes(case)
    if case["kind"] == "gemm":
        M = case["M"]
        return {"bytes": stored + 2 * M * (K + N), "flops": 2 * M * K * N}
    if case["kind"] == "grouped":
        E, T, P = case["E"], case["T"], case["T"] * case["topk"]
        busy = E * (1.0 - (1.0 - case["topk"] / E) ** T)    # experts that some token goes to, on average
        return {"bytes": busy * stored + 2 * T * K + 2 * P * N, "flops": 2 * P * K * N}
    if case["kind"] == "quantize":
        return {"bytes": 4 * K * N + stored, "flops": 0}
    return {"bytes": 2 * stored, "flops": 0}


def tolerance(case):
    # quantized and loaded weights are whole numbers and stored bits; products are bf16 (half a unit in the last place is
    # 2^-9), from bf16 activations and weights that a kernel may round to bf16, summed in fp32
    return "exact" if case["kind"] in ("quantize", "load") else {"rel": 5e-3, "max": 3e-2}
