"""The calls that a program built on this library makes, as cases to be timed and compared.

A case is one pass through the public entry points of ``paper_2412_14363_amd.binding``: a quantized linear layer
at a serving size (one token, a handful, a batch of generating sequences, a prefill chunk, a full prefill), the
gated MLP block, the cache-side kernels, and the offline preparation of a layer's weights and of a head's basis.
Sizes are layer shapes of ``paper_2412_14363_amd.workloads`` (Llama-3-8B, Llama-3-70B, Qwen2.5-72B) and generic
ragged ones.  ``draw`` gives more cases of the same kinds over the same ranges.
"""
import math

import torch

from paper_2412_14363_amd import binding as rq

DEV = "cuda"


# ---- the cases ---------------------------------------------------------------------------------

def _layer(name, M, K, N, r, path="two_calls", act="outliers", block=0):
    """path: "one_call" (quantizer inside the GEMM), "two_calls", "asym" (asymmetric activations),
    "hadamard" (block Walsh-Hadamard transform of the low group fused with the quantizer)."""
    return {"name": name, "kind": "layer", "path": path, "M": M, "K": K, "N": N, "r": r, "act": act, "block": block}


def listed():
    return [
        # one sequence generating on an 8B model: the smallest call there is, o_proj for a single token
        _layer("o_proj_m1_one_call", 1, 4096, 4096, 512, path="one_call"),
        # a few sequences generating on a 70B model: the up projection, 133 MB of weights for 4 tokens
        _layer("up_70b_m4", 4, 8192, 28672, 1024),
        # batched generation, 64 sequences, same layer
        _layer("up_70b_m64", 64, 8192, 28672, 1024),
        # a 512-token prefill chunk through the 8B down projection, with its online transform
        _layer("down_8b_chunk_m512", 512, 14336, 4096, 1792, path="hadamard", act="student_t3"),
        # a prompt of ragged length on a layer whose sizes divide nothing, asymmetric activations
        # (the setting of the paper's own experiments)
        _layer("ragged_asym_m777", 777, 5000, 3001, 624, path="asym", act="student_t3"),
        # a 2048-token prefill through the 8B o_proj
        _layer("o_proj_8b_m2048", 2048, 4096, 4096, 512),
        # the whole MLP block of an 8B model on 4096 tokens: gate/up with the gated activation, transform, down
        {"name": "mlp_block_8b_m4096", "kind": "mlp", "M": 4096, "K": 4096, "F": 14336, "r": 512, "r2": 1792, "block": 256},
        # the largest prefill: 8192 tokens through the gate/up shape of Qwen2.5-72B
        _layer("mlp_72b_m8192", 8192, 8192, 29568, 1024, act="student_t3"),
        # K and V entries of 2048 new tokens (8 heads each) into compact cache rows, and back for attention
        {"name": "kv_cache_2048_tokens", "kind": "kv", "rows": 32768, "d": 128, "r": 16},
        # queries and keys of 2048 tokens (32 + 8 heads) onto the cache basis
        {"name": "heads_2048_tokens", "kind": "heads", "rows": 81920, "d": 128},
        # offline: the basis folded into the weights of an o_proj (W U), which are then quantized and packed
        {"name": "fold_and_pack_4096", "kind": "fold", "N": 4096, "K": 4096, "r": 512},
        # offline: the principal axes of one head's calibration covariance
        {"name": "head_basis_128", "kind": "eig", "K": 128, "sweeps": 12},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rank(rng, K, unit):
    """Width of the 8-bit group: mostly an eighth of K, now and then none, a quarter, or something between."""
    r = rng.choice([K // 8, K // 8, K // 8, K // 4, 0, rng.randint(0, K // 4)])
    return r // unit * unit


def draw(rng):
    kind = rng.choice(["layer"] * 8 + ["mlp", "kv", "heads", "fold", "eig"])
    act = rng.choice(["normal", "outliers", "student_t3"])
    if kind == "layer":
        path = rng.choice(["one_call", "two_calls", "two_calls", "asym", "hadamard"])
        while True:
            M = rng.randint(1, 4) if path == "one_call" else _log_int(rng, 1, 8192)
            K = _log_int(rng, 1024, 28672)
            N = _log_int(rng, 256, 29568)
            if 2 * M * K * N <= 2 * 8192 * 8192 * 29568 and K * N <= 8192 * 29568:
                break
        block = 0
        if path == "hadamard":
            block = rng.choice([64, 128, 256, 256])
            K = min(K, 28672 if block == 256 else 16384)
            K = max(1024, K // block * block)
            r = _rank(rng, K, block)
            if block == 256 and K > 16384:
                r = max(K - 26624, min(r, 4096))
        elif path == "one_call":  # this entry point wants whole 16-byte pieces
            K = K // 8 * 8
            r = _rank(rng, K, 8)
        else:
            unit = rng.choice([64, 8, 8, 2])
            K = K // unit * unit
            r = _rank(rng, K, unit)
        return dict(_layer("", M, K, N, r, path, act, block), name="%s_%dx%dx%d" % (path, M, K, N))
    if kind == "mlp":
        M, K, F = _log_int(rng, 16, 4096), _log_int(rng, 1024, 4096) // 64 * 64, rng.randint(2, 7) * 2048
        c = {"kind": "mlp", "M": M, "K": K, "F": F, "r": K // 8 // 8 * 8, "r2": F // 8, "block": 256}
    elif kind == "kv":
        d = rng.choice([64, 128, 128, 256])
        c = {"kind": "kv", "rows": _log_int(rng, 64, 262144), "d": d, "r": d // 8}
    elif kind == "heads":
        c = {"kind": "heads", "rows": _log_int(rng, 40, 327680), "d": rng.choice([64, 128, 128])}
    elif kind == "fold":
        K = _log_int(rng, 512, 4096) // 8 * 8
        c = {"kind": "fold", "N": _log_int(rng, 256, 8192), "K": K, "r": _rank(rng, K, 8)}
    else:
        c = {"kind": "eig", "K": rng.choice([64, 128, rng.randrange(32, 129, 2)]), "sweeps": 12}
    return dict(c, name=c["kind"] + "".join("_%s%d" % (k, v) for k, v in c.items() if k != "kind"))


# ---- inputs ------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _activations(M, K, r, act, g):
    """Projected activations: close to Gaussian, or heavy-tailed, or with 1 % of the columns twenty times as large
    (columns that the projection has moved into the 8-bit group, where there is one)."""
    x = torch.randn(M, K, generator=g, device=DEV)
    if act == "student_t3":
        chi = torch.zeros_like(x)
        for _ in range(3):
            chi += torch.randn(M, K, generator=g, device=DEV).square_()
        x /= chi.div_(3.0).sqrt_()
    elif act == "outliers":
        width = r if r > 0 else K
        at = torch.randperm(width, generator=g, device=DEV)[:min(width, -(-K // 100))]
        x[:, at] *= 20.0
    return x.to(torch.bfloat16)


def _weights(N, K, g):
    return (torch.randn(N, K, generator=g, device=DEV) * 0.02).to(torch.bfloat16)


def _orthogonal(n, g):
    return torch.linalg.qr(torch.randn(n, n, generator=g, device=DEV, dtype=torch.float32))[0].contiguous()


def _covariance(K, g):
    """Covariance of a head's calibration rows: a decaying spectrum in a random basis, distinct eigenvalues."""
    q = torch.linalg.qr(torch.randn(K, K, generator=g, device=DEV, dtype=torch.float64))[0]
    lam = torch.exp(-6.0 * torch.arange(K, device=DEV, dtype=torch.float64) / K)
    lam *= 1.0 + 0.02 * torch.rand(K, generator=g, device=DEV, dtype=torch.float64)
    c = (q * lam) @ q.t()
    return (0.5 * (c + c.t())).float().contiguous()


def _inputs(case, seed):
    """The tensors that a case starts from; also what exact() starts from."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "layer":
        return {"w": _weights(case["N"], case["K"], g),
                "x": _activations(case["M"], case["K"], case["r"], case["act"], g)}
    if kind == "mlp":
        return {"w1": _weights(2 * case["F"], case["K"], g),  # gate and up rows interleaved
                "w2": _weights(case["K"], case["F"], g),
                "x": _activations(case["M"], case["K"], case["r"], "outliers", g)}
    if kind == "kv":
        return {"x": _activations(case["rows"], case["d"], case["r"], "student_t3", g)}
    if kind == "heads":
        d = case["d"]
        return {"w": _orthogonal(d, g).t().contiguous().to(torch.bfloat16),
                "x": _activations(case["rows"], d, d, "normal", g)}
    if kind == "fold":
        return {"w": _weights(case["N"], case["K"], g), "u": _orthogonal(case["K"], g)}
    return {"c": _covariance(case["K"], g)}


def prepare(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    s = {"case": case}
    if kind == "layer":
        M, K, N, r = case["M"], case["K"], case["N"], case["r"]
        s["packed"] = rq.resq_pack_weights(t["w"], r)
        s["x"] = t["x"]
        s["y"] = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
        if case["path"] != "one_call":
            s["act"] = rq.ActCodes(M, K, r, DEV)
    elif kind == "mlp":
        M, K, F = case["M"], case["K"], case["F"]
        s["p1"] = rq.resq_pack_weights(t["w1"], case["r"])
        s["p2"] = rq.resq_pack_weights(t["w2"], case["r2"])
        s["x"] = t["x"]
        s["act1"], s["act2"] = rq.ActCodes(M, K, case["r"], DEV), rq.ActCodes(M, F, case["r2"], DEV)
        s["h"] = torch.empty((M, F), dtype=torch.bfloat16, device=DEV)
        s["y"] = torch.empty((M, K), dtype=torch.bfloat16, device=DEV)
    elif kind == "kv":
        s["x"] = t["x"]
        s["cache"] = torch.empty((case["rows"], rq.resq_kv_cache_row_bytes(case["d"], case["r"])), dtype=torch.uint8, device=DEV)
        s["out"] = torch.empty_like(t["x"])
    elif kind == "heads":
        s["packed"] = rq.resq_pack_weights(t["w"], case["d"])
        s["x"] = t["x"]
        s["y"] = torch.empty_like(t["x"])
    elif kind == "fold":
        s.update(t)
        s["wu"] = torch.empty_like(t["w"])
        s["packed"] = rq.alloc_packed(case["N"], case["K"], case["r"], DEV)
    else:
        s.update(t)
        K = case["K"]
        s["lam"] = torch.empty(K, dtype=torch.float32, device=DEV)
        s["p"] = torch.empty((K, K), dtype=torch.float32, device=DEV)
    return s


# ---- one pass ----------------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "layer":
        path, r, N = case["path"], case["r"], case["N"]
        if path == "one_call":
            return {"y": rq.resq_quantize_gemm_mixed(s["x"], s["packed"], N, r, y=s["y"])}
        if path == "asym":
            rq.resq_quantize_act_asym(s["x"], r, out=s["act"])
            return {"y": rq.resq_gemm_mixed_asym(s["act"], s["packed"], N, y=s["y"])}
        if path == "hadamard":
            rq.resq_hadamard_quantize_act(s["x"], r, case["block"], out=s["act"])
        else:
            rq.resq_quantize_act(s["x"], r, out=s["act"])
        return {"y": rq.resq_gemm_mixed(s["act"], s["packed"], N, y=s["y"])}
    if kind == "mlp":
        rq.resq_quantize_act(s["x"], case["r"], out=s["act1"])
        rq.resq_gemm_mixed_swiglu(s["act1"], s["p1"], 2 * case["F"], y=s["h"])
        rq.resq_hadamard_quantize_act(s["h"], case["r2"], case["block"], out=s["act2"])
        rq.resq_gemm_mixed(s["act2"], s["p2"], case["K"], y=s["y"])
        return {"h": s["h"], "y": s["y"]}
    if kind == "kv":
        rq.resq_quantize_kv_cache(s["x"], case["r"], cache=s["cache"])
        rq.resq_dequantize_kv_cache(s["cache"], case["d"], case["r"], out=s["out"])
        return {"cache": s["cache"], "x": s["out"]}
    if kind == "heads":
        return {"y": rq.resq_project_heads(s["x"], s["packed"], y=s["y"])}
    if kind == "fold":
        rq.resq_project_rows(s["w"], s["u"], out=s["wu"])
        rq.resq_pack_weights(s["wu"], case["r"], packed=s["packed"])
        return {"wu": s["wu"], "packed": s["packed"]}
    lam, p = rq.resq_sym_eig_static(s["c"], s["lam"], s["p"], sweeps=case["sweeps"])
    return {"lam": lam, "p": p}


# ---- what a pass cannot do without ---------------------------------------------------------------

def _weight_bytes(N, K, r):
    return N * (r + (K - r) / 2 + 4)  # codes and two fp16 scales per channel


def work(case):
    kind = case["kind"]
    if kind == "layer":
        M, K, N, r = case["M"], case["K"], case["N"], case["r"]
        return {"bytes": 2 * M * K + _weight_bytes(N, K, r) + 2 * M * N, "flops": 2 * M * N * K}
    if kind == "mlp":
        M, K, F = case["M"], case["K"], case["F"]
        return {"bytes": 4 * M * K + 2 * M * F + _weight_bytes(2 * F, K, case["r"]) + _weight_bytes(K, F, case["r2"]),
                "flops": 6 * M * K * F}
    if kind == "kv":
        return {"bytes": case["rows"] * (4 * case["d"] + case["r"] + (case["d"] - case["r"]) / 2 + 16), "flops": 0}
    if kind == "heads":
        return {"bytes": case["rows"] * 4 * case["d"] + case["d"] ** 2, "flops": 2 * case["rows"] * case["d"] ** 2}
    if kind == "fold":
        N, K = case["N"], case["K"]
        return {"bytes": 4 * N * K + 4 * K * K + _weight_bytes(N, K, case["r"]), "flops": 2 * N * K * K}
    K = case["K"]
    return {"bytes": 8 * K * K + 4 * K, "flops": 9 * K ** 3}  # reduction, values and vectors of a direct method


def tolerance(case):
    """bf16 outputs of exact integer sums: two correct implementations differ where the last fp32 rounding of the
    scaling moves a value over a bf16 boundary (one bf16 step of the value, on few values).  Behind the online
    transform a rotated value can be the neighbouring bf16 and move a 4-bit code by one step, which the sum over K
    averages out."""
    kind = case["kind"]
    if kind == "kv":  # codes at exact ties aside, cache bytes are defined bit by bit
        return {"rel": 1e-3, "max": 1e-2, "differ": 1e-4}
    if kind == "fold":  # a weight next to a bf16 boundary moves, and with it a code now and then
        return {"rel": 2e-3, "max": 1e-2, "differ": 5e-3}
    if kind == "eig":
        return {"rel": 1e-5, "max": 1e-4}
    if kind == "mlp" or case.get("path") == "hadamard":
        return {"rel": 5e-3, "max": 0.1}
    return {"rel": 2e-3, "max": 1e-2}


# ---- the same in 64 bits ---------------------------------------------------------------------------

def _scale(top, qmax):
    s = (top.double() / qmax).float()
    return torch.where(s > 0, s, torch.ones_like(s))


def _symmetric(v, qmax):
    """v quantized to [-qmax, qmax] per row and put back, in float64; codes are those of fp32 quotients."""
    if v.shape[1] == 0:
        return v.double()
    s = _scale(v.abs().amax(1, keepdim=True).float(), qmax).double()
    q = (v.double() / s).float().double().round().clamp(-qmax, qmax)
    return q * s


def _asymmetric(v, levels):
    """(codes 0..levels, scale, zero-point) of each row, float64."""
    lo, hi = v.amin(1, keepdim=True).float(), v.amax(1, keepdim=True).float()
    s = ((hi - lo).double() / levels).float()
    s = torch.where(s > 0, s, torch.ones_like(s)).double()
    q = ((v.float() - lo).double() / s).float().double().round().clamp(0, levels)
    return q, s, lo.double()


def _act(x, r, asym=False):
    if not asym:
        return torch.cat([_symmetric(x[:, :r], 127), _symmetric(x[:, r:], 7)], 1)
    parts = []
    for v, levels in ((x[:, :r], 255), (x[:, r:], 15)):
        if v.shape[1]:
            q, s, z = _asymmetric(v, levels)
            parts.append(q * s + z)
    return torch.cat(parts, 1)


def _weight_group(w, qmax):
    if w.shape[1] == 0:
        return w.double()
    s = (w.abs().amax(1, keepdim=True).double() / qmax).float()
    h = s.half()
    up = torch.nextafter(h.cpu(), torch.tensor(float("inf"), dtype=torch.float16)).to(h.device)
    h = torch.where(h.float() < s, up, h).float().clamp(2.0 ** -14, 65504.0).double()
    q = (w.double() / h).float().double().round().clamp(-qmax, qmax)
    return q * h


def _weight(w, r):
    return torch.cat([_weight_group(w[:, :r], 127), _weight_group(w[:, r:], 7)], 1)


def _hadamard(x, r, block):
    """Columns [r, K) through the block transform in float64, rounded to bf16."""
    n = x.shape[1] - r
    if block == 0:
        block = 1
        while n % (2 * block) == 0 and block < 8192:
            block *= 2
    v = x[:, r:].double().reshape(x.shape[0], n // block, block)
    h = 1
    while h < block:
        v = v.reshape(x.shape[0], n // block, block // (2 * h), 2, h)
        a, b = v[..., 0, :], v[..., 1, :]
        v = torch.stack([a + b, a - b], -2)
        h *= 2
    v = v.reshape(x.shape[0], n) / math.sqrt(block)
    return torch.cat([x[:, :r], v.to(torch.bfloat16)], 1)


def exact(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "layer":
        x, r = t["x"], case["r"]
        if case["path"] == "hadamard":
            x = _hadamard(x, r, case["block"])
        return {"y": _act(x, r, case["path"] == "asym") @ _weight(t["w"], r).t().contiguous()}
    if kind == "mlp":
        z = _act(t["x"], case["r"]) @ _weight(t["w1"], case["r"]).t().contiguous()
        gate, up = z[:, 0::2], z[:, 1::2]
        h = gate / (1 + torch.exp(-gate)) * up
        x2 = _hadamard(h.to(torch.bfloat16), case["r2"], case["block"])
        return {"h": h, "y": _act(x2, case["r2"]) @ _weight(t["w2"], case["r2"]).t().contiguous()}
    if kind == "kv":
        return {"cache": None, "x": _act(t["x"], case["r"], asym=True)}
    if kind == "heads":
        return {"y": _symmetric(t["x"], 127) @ _weight_group(t["w"], 127).t().contiguous()}
    if kind == "fold":
        return {"wu": t["w"].double() @ t["u"].double(), "packed": None}
    lam = torch.linalg.eigvalsh(t["c"].double().cpu()).flip(0)
    return {"lam": lam.to(DEV), "p": None}  # eigenvectors are defined up to their signs
