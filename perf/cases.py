"""The performance cases of this library: the work a user has it do, through its public entry points.

A case names what is called ("kind"), the matrices (a Llama 3.1 layer, or N and K), the precision (bits, group size
along K; 0 = one scale per output channel) and the rows M of the activations.  The kinds:

  linear    rtn_linear on one matrix, output and workspace kept by the caller: one projection of a decode step
  layer     rtn_layer_forward on the four linear modules of a Transformer layer: a decode step, a speculative or
            batched step, or the prefill of M prompt tokens, depending on M
  grouped   rtn_grouped_forward on the active experts of a mixture-of-experts layer, each with its own rows
  asym      rtn_linear_asym (per-group zero points) on the four modules of a layer
  dense     rtn_linear_dense on one matrix: dequantise, then the 16-bit GEMM, for long prompts
  quantize  rtn_quantize / rtn_quantize_asym on the four matrices of a layer: loading a model
"""
import math

import torch

import paper_2505_15909_amd as rtn
from paper_2505_15909_amd import synth

LAYERS = {"8b": synth.LLAMA_8B, "70b": synth.LLAMA_70B, "405b": synth.LLAMA_405B}
DEV = "cuda:0"

# What a drawn case may cost at most: the largest listed layers (405B selective layer at 16 rows, 70B dense path).
MOST_FLOPS = 1.9e12
MOST_BYTES = 2.3e9


def _layer(name, model, M, bits=4, group=128, bits8="", kind="layer"):
    """bits8: the modules kept at 8 bit with one scale per channel (selective precision), comma-separated."""
    return {"name": name, "kind": kind, "model": model, "M": M, "bits": bits, "group": group, "bits8": bits8}


def listed():
    return [
        # the smallest call: one 4096 x 4096 projection, one token
        {"name": "linear_w4_m1", "kind": "linear", "N": 4096, "K": 4096, "M": 1, "bits": 4, "group": 128},
        # token generation, one sequence and a batch of sixteen, 4 bit
        _layer("decode_8b_w4_m1", "8b", 1),
        _layer("decode_8b_w4_m16", "8b", 16),
        # token generation at 8 bit with per-channel scales
        _layer("decode_8b_w8_m4", "8b", 4, bits=8, group=0),
        # selective precision: the attention output and down projections of a large model kept at 8 bit
        _layer("decode_405b_selective_m16", "405b", 16, bits8="o,down"),
        # a batch of 32 sequences on a large model
        _layer("batch_70b_w4_m32", "70b", 32),
        # a ragged batch of prompt pieces and decode rows in one step
        _layer("mixed_8b_w4_m200", "8b", 200),
        # prefill of a prompt
        _layer("prefill_8b_w4_m2048", "8b", 2048),
        # zero points at the finer group size, a short prompt
        _layer("prefill_8b_asym_g64_m256", "8b", 256, group=64, kind="asym"),
        # a long prompt on the dual path of large inputs
        {"name": "dense_70b_down_m4096", "kind": "dense", "N": 8192, "K": 28672, "M": 4096, "bits": 4, "group": 128},
        # eight active experts with a few tokens each
        {"name": "experts_w4", "kind": "grouped", "N": 2048, "K": 7168, "experts": 8, "rows": 4, "bits": 4, "group": 128},
        # loading: quantise and pack the four matrices of a layer
        {"name": "quantize_70b_w4", "kind": "quantize", "model": "70b", "bits": 4, "group": 128, "asym": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_rows(rng, hi):
    """Rows from 1 to hi, spread over their logarithm; now and then a power of two."""
    m = _log_int(rng, 1, hi)
    return min(hi, 1 << m.bit_length() - 1) if rng.random() < 0.25 else m


def _draw_matrix(rng):
    """A matrix of one of the layers, or one of other sizes (N in sixteens, K in 512s)."""
    if rng.random() < 0.4:
        K, N = rng.choice([s for d in LAYERS.values() for s in d.values()])
        return N, K
    K = 512 * _log_int(rng, 2, 48)
    return 16 * max(32, min(3584, _log_int(rng, 64, 3584), (1 << 29) // (16 * K))), K


def _draw_format(rng):
    """bits and group size: mostly those of the paper, sometimes the other ones."""
    return rng.choice([(4, 128), (4, 128), (4, 128), (8, 0), (8, 0), (8, 128), (4, 0), (4, 64), (4, 32), (4, 256)])


def draw(rng):
    while True:
        kind = rng.choice(["linear", "linear", "layer", "layer", "layer", "layer", "asym", "dense", "grouped", "quantize"])
        bits, group = _draw_format(rng)
        c = {"kind": kind, "bits": bits, "group": group}
        if kind == "linear":
            c["N"], c["K"] = _draw_matrix(rng)
            c["M"] = _draw_rows(rng, 2048)
        elif kind == "layer":
            c["model"] = rng.choice(["8b", "8b", "70b", "405b"])
            c["bits8"] = rng.choice(["", "", "o,down", "qkv,gate_up,down"]) if bits == 4 else ""
            c["M"] = _draw_rows(rng, 4096)
        elif kind == "asym":
            c["model"], c["bits8"] = rng.choice(["8b", "8b", "70b"]), ""
            c["M"] = _draw_rows(rng, 512)
        elif kind == "dense":
            c["N"], c["K"] = _draw_matrix(rng)
            c["M"] = _log_int(rng, 1024, 8192)
        elif kind == "grouped":
            c["K"] = rng.choice([2048, 4096, 6144, 7168])
            c["N"] = 16 * _log_int(rng, 64, 512)
            c["experts"] = rng.randint(2, 16)
            c["rows"] = _log_int(rng, 1, 16)
        else:
            c["model"] = rng.choice(["8b", "70b", "70b"])
            c["asym"] = rng.random() < 0.3
        w = work(c)
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES:
            return c


def _weight(model, N, K, seed):
    """Weights as in the models: normal, with heavy tails and 1 % of outlier columns in the 70B ones.  Drawn in row blocks."""
    W = torch.empty((N, K), dtype=torch.float16, device=DEV)
    rows = max(16, (1 << 26) // K)
    for b, r in enumerate(range(0, N, rows)):
        n = min(rows, N - r)
        if model == "70b":
            W[r:r + n] = synth.heavy_tail_weight(n, K, 0.02, seed * 1009 + b, DEV, outlier_gain=1.0)
        else:
            W[r:r + n] = synth.normal_weight(n, K, 0.01 if model == "405b" else 0.02, seed * 1009 + b, DEV)
    if model == "70b":
        g = torch.Generator(device=DEV)
        g.manual_seed(seed * 1009 + 997)
        W[:, torch.randperm(K, generator=g, device=DEV)[:K // 100]] *= 10.0
    return W


def _modules(case):
    """(name, N, K, bits, group, M) of the matrices of a case."""
    if "model" in case:
        out = []
        for name, (K, N) in LAYERS[case["model"]].items():
            eight = name in (case.get("bits8") or "").split(",")
            out.append((name, N, K, 8 if eight else case["bits"], 0 if eight else case["group"], case.get("M", 0)))
        return out
    if case["kind"] == "grouped":
        # ragged rows per expert, 1 .. twice the typical number (at most 16, what one decode step routes to an expert)
        return [("e%d" % e, case["N"], case["K"], case["bits"], case["group"],
                 max(1, min(16, (case["rows"] * (1 + e * 5 % 8)) // 4))) for e in range(case["experts"])]
    return [("w", case["N"], case["K"], case["bits"], case["group"], case["M"])]


def prepare(case, seed):
    model = case.get("model", "")
    mods = []
    for i, (name, N, K, bits, group, M) in enumerate(_modules(case)):
        W = _weight(model, N, K, seed * 64 + i)
        if case["kind"] == "quantize":
            mods.append({"W": W})
            continue
        m = {"A": synth.activation(M, K, seed * 64 + 32 + i, DEV), "bits": bits, "group_size": group,
             "C": torch.empty((M, N), dtype=torch.float16, device=DEV)}
        if case["kind"] == "asym":
            m["qweight"], m["scales"], m["zeros"] = rtn.rtn_quantize_asym(W, bits, group)
        else:
            m["qweight"], m["scales"] = rtn.rtn_quantize(W, bits, group)
        del W
        mods.append(m)
    state = {"case": case, "mods": mods}
    if case["kind"] in ("layer", "grouped"):
        state["plan"] = rtn.LayerPlan(mods)
    elif case["kind"] != "quantize":
        need = max(rtn.rtn_workspace_nbytes(m["A"].shape[0], m["C"].shape[1], m["A"].shape[1], m["bits"], m["group_size"])
                   for m in mods)
        state["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
        if case["kind"] == "dense":
            state["w_tmp"] = torch.empty(rtn.rtn_dense_weight_nbytes(case["N"], case["K"]), dtype=torch.uint8, device=DEV)
    else:
        for m in mods:                                     # the model's packed tensors, allocated once as a loader does
            N, K = m["W"].shape
            g = case["group"] or K
            m["out"] = (torch.empty(rtn.rtn_qweight_nbytes(N, K, case["bits"]), dtype=torch.uint8, device=DEV),
                        torch.empty((N, K // g), dtype=torch.float16, device=DEV))
    return state


def run(state):
    case, mods, kind = state["case"], state["mods"], state["case"]["kind"]
    if kind == "layer":
        state["plan"].run()
    elif kind == "grouped":
        state["plan"].run_grouped()
    elif kind == "linear":
        m = mods[0]
        return rtn.rtn_linear(m["A"], m["qweight"], m["scales"], m["bits"], m["group_size"], out=m["C"],
                              workspace=state["workspace"])
    elif kind == "asym":
        for m in mods:
            rtn.rtn_linear_asym(m["A"], m["qweight"], m["scales"], m["zeros"], m["bits"], m["group_size"], out=m["C"],
                                workspace=state["workspace"])
    elif kind == "dense":
        m = mods[0]
        return rtn.rtn_linear_dense(m["A"], m["qweight"], m["scales"], m["bits"], m["group_size"], state["w_tmp"],
                                    out=m["C"], workspace=state["workspace"])
    elif case["asym"]:
        return [rtn.rtn_quantize_asym(m["W"], case["bits"], case["group"]) for m in mods]
    else:
        return [rtn.rtn_quantize(m["W"], case["bits"], case["group"], out=m["out"]) for m in mods]
    return [m["C"] for m in mods]


def work(case):
    """Every weight, scale, activation and output moved once; the products of the matrices as asked for (no padding)."""
    nbytes = flops = 0
    for name, N, K, bits, group, M in _modules(case):
        packed = N * K * bits / 8 + N * (K // (group or K)) * 2 * (2 if case["kind"] == "asym" or case.get("asym") else 1)
        if case["kind"] == "quantize":
            nbytes += 2 * N * K + packed
        else:
            nbytes += packed + 2 * M * K + 2 * M * N
            flops += 2 * M * N * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Packing is exact by definition.  A linear layer rounds its result to fp16 and, where weights are scaled in fp16
    before the product, each weight once more: against a float64 product of the dequantised weights the listed cases are
    off by 2.0e-4 .. 2.7e-4 of the norm, and single outputs by 4.5e-4 .. 1.1e-3.  Four to five times that."""
    if case["kind"] == "quantize":
        return "exact"
    return {"rel": 1.1e-3, "max": 6e-3}
