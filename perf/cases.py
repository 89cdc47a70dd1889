"""What this framework's speed is measured on: the work that its users have it do, through the calls of
paper_2505_06653_amd.binding, from a cache-resident tensor to a Llama-70B-shaped layer.

A case is a dict of plain values; its "op" says which call (or chain of calls) a pass is:

  step        one step of the data-driven codebook design with the quantised tensor as its by-product: bof4_quantize_lloyd,
              bof4_codebook_update, bof4_dequantize (what bench.py times)
  roundtrip   bof4_quantize, then bof4_dequantize of what it wrote: encode and decode of a tensor
  lloyd       bof4_lloyd_step and bof4_codebook_update: one iteration of the codebook design alone (MSE criterion)
  mae         bof4_lloyd_step_mae and bof4_codebook_update_mae: the same under the MAE criterion
  error       bof4_quant_error: the MSE / MAE figures of a tensor
  gemv        one or a few tokens through the quantised matrices of a model's block (generation)
  gemm        many tokens through them (a batch in generation, or the processing of a prompt)

Weights are what inputs.py makes for the workloads of the tests and of bench.py: Student-t or Gaussian values, with a
scale per row, with or without planted outliers; activations are normal, bfloat16.  Buffers, workspaces and the tables
of the products are allocated and filled once, as a program that calls in a loop keeps them.
"""
import math

import torch

from paper_2505_06653_amd import binding, codebooks, inputs

# The projections of a block as matrices of one input each, [rows x cols]: q, k, v together, o, gate and up together,
# down.
LLAMA7B = "12288x4096 4096x4096 22016x4096 4096x11008"
LLAMA70B = "10240x8192 8192x8192 57344x8192 8192x28672"


def listed():
    return [
        # A tensor of a small model (1024 x 1024, Gaussian): everything fits the caches, launches and host work count.
        {"name": "step_1m", "op": "step", "shapes": "1024x1024", "block": 64, "signed": 1, "opq": 0, "dist": "gauss"},
        # Encode and decode of a Llama-7B-shaped block with the plain method: absolute maxima, no outlier list.
        {"name": "roundtrip_7b", "op": "roundtrip", "shapes": LLAMA7B, "block": 64, "signed": 0, "opq": 0, "dist": "t5"},
        # The same with the finest blocks, signed maxima and outliers that pile up in a few columns.
        {"name": "roundtrip_7b_opq_i32", "op": "roundtrip", "shapes": LLAMA7B, "block": 32, "signed": 1, "opq": 1,
         "dist": "planted"},
        # The flagship step: one Llama-70B-shaped layer, outliers kept apart.
        {"name": "step_70b_opq", "op": "step", "shapes": LLAMA70B, "block": 64, "signed": 1, "opq": 1, "dist": "t4"},
        # Codebook design over the weights of several Llama-7B-shaped blocks at once (the largest stream).
        {"name": "lloyd_7b_x8", "op": "lloyd", "shapes": " ".join([LLAMA7B] * 8), "block": 64, "signed": 1, "opq": 0,
         "dist": "t5"},
        # Codebook design for the MAE criterion over one Llama-70B-shaped layer.
        {"name": "mae_70b", "op": "mae", "shapes": LLAMA70B, "block": 64, "signed": 1, "opq": 0, "dist": "t4"},
        # Quality figures of one odd-sized matrix.
        {"name": "error_ragged_opq_i128", "op": "error", "shapes": "10001x4224", "block": 128, "signed": 1, "opq": 1,
         "dist": "t5"},
        # Generation: three sequences through a small odd-sized projection, and one through a whole block.
        {"name": "gemv_small_3tok", "op": "gemv", "shapes": "1001x1504", "block": 32, "signed": 0, "opq": 0,
         "dist": "t5", "tokens": 3},
        {"name": "gemv_7b_opq", "op": "gemv", "shapes": LLAMA7B, "block": 64, "signed": 1, "opq": 1, "dist": "t5",
         "tokens": 1},
        # A batch of sequences in generation, without and with outliers.
        {"name": "gemm_7b_32tok", "op": "gemm", "shapes": LLAMA7B, "block": 64, "signed": 0, "opq": 0, "dist": "t5",
         "tokens": 32},
        {"name": "gemm_70b_128tok_opq", "op": "gemm", "shapes": LLAMA70B, "block": 64, "signed": 1, "opq": 1,
         "dist": "t4", "tokens": 128},
        # A prompt of 2000 tokens through a block.
        {"name": "gemm_7b_2000tok_opq", "op": "gemm", "shapes": LLAMA7B, "block": 64, "signed": 1, "opq": 1,
         "dist": "t5", "tokens": 2000},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "roundtrip", "roundtrip", "lloyd", "mae", "error", "gemv", "gemv", "gemm", "gemm", "gemm"])
    block = rng.choice([32, 64, 64, 128, 256])
    case = {"op": op, "block": block, "signed": rng.choice([0, 1, 1]), "opq": rng.choice([0, 1]),
            "dist": rng.choice(["gauss", "t5", "t4", "planted"])}
    if op in ("gemv", "gemm"):
        rows = _log_uniform(rng, 500, 28672)
        cols = max(1, _log_uniform(rng, 512, 28672) // block) * block
        tokens = rng.choice([1, 1, 1, 2, 3, 4]) if op == "gemv" else _log_uniform(rng, 8, 2500)
        while rows * cols * tokens > 202_375_168 * 2000:
            tokens //= 2
        case.update(shapes=f"{rows}x{cols}", tokens=tokens)
    else:
        n = _log_uniform(rng, 1 << 18, 1_500_000_000 if op == "lloyd" else 600_000_000)
        cols = max(1, _log_uniform(rng, 512, 12000) // block) * block
        case["shapes"] = f"{max(1, n // cols)}x{cols}"
    return case


def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split()]


def _n(case):
    return sum(r * c for r, c in _shapes(case))


def _weights(case, seed):
    mats = []
    for k, (r, c) in enumerate(_shapes(case)):
        s = seed * 64 + k
        if case["dist"] == "gauss":
            m = inputs.gaussian_matrix(r, c, 0.02, s, "cuda")
        elif case["dist"] == "t4":
            m = inputs.student_t_matrix(r, c, 4.0, 0.015, 0.0, s, "cuda")
        else:
            m = inputs.student_t_matrix(r, c, 5.0, 0.02, 0.3, s, "cuda")
        if case["dist"] == "planted":
            inputs.plant_outliers(m, s + 32)
        mats.append(m)
    return mats


def _codebook(case):
    if case["op"] == "mae":
        return codebooks.array(codebooks.BOF4S_MAE_64 if case["signed"] else codebooks.BOF4_MAE_64)
    return codebooks.array(codebooks.BOF4S_MSE[case["block"]] if case["signed"] else codebooks.BOF4_MSE_64)


def _quantized(w, case, cb, T):
    n, block = w.numel(), case["block"]
    cap = n // 16 + 64 if T > 0 else 0
    codes, scales, idx, val, k = binding.bof4_quantize(w, block, cb, case["signed"], opq_T=T, out_capacity=cap)
    return codes, scales, idx.clone() if k else None, val.clone() if k else None, k


def prepare(case, seed):
    block, dev = case["block"], "cuda"
    cb = _codebook(case)
    T = binding.bof4_opq_threshold(0.95, block) if case["opq"] else 0.0
    st = {"case": case, "cb": cb, "T": T, "pin": codebooks.PIN_BOF4S if case["signed"] else codebooks.PIN_BOF4}
    mats = _weights(case, seed)
    if case["op"] in ("gemv", "gemm"):
        g = torch.Generator(device=dev)
        g.manual_seed(seed + 7)
        layers = []
        for m in mats:
            r, c = m.shape
            codes, scales, idx, val, k = _quantized(m.reshape(-1), case, cb, T)
            x = torch.randn((case["tokens"], c), generator=g, device=dev, dtype=torch.float32).to(torch.bfloat16)
            y = torch.empty((case["tokens"], r), dtype=torch.float32, device=dev)
            if case["op"] == "gemv":
                tab = binding.bof4_gemv_outlier_table(codes, scales, r, c, block, cb, idx, val) if k else None
                layers.append((r, c, codes, scales, tab, k, x, y, None))
            else:
                tab = binding.bof4_gemm_outlier_table(codes, scales, r, c, block, cb, idx, val) if k else None
                packed = binding.bof4_gemm_pack(codes, scales, r, c, block)
                ws = torch.empty(binding.bof4_gemm_workspace_bytes(r, c, case["tokens"]), dtype=torch.uint8, device=dev)
                layers.append((r, c, packed, None, tab, k, x, y, ws))
        st["layers"] = layers
        return st
    w = torch.cat([m.reshape(-1) for m in mats]) if len(mats) > 1 else mats[0].reshape(-1)
    del mats
    n = w.numel()
    st["w"] = w
    cap = n // 16 + 64 if T > 0 and case["op"] in ("step", "roundtrip") else 0
    st["cap"] = cap
    st["ws"] = binding.alloc_workspace(n, block, cap, dev)
    if case["op"] in ("step", "roundtrip"):
        st["codes"] = torch.empty(n // 2, dtype=torch.uint8, device=dev)
        st["scales"] = torch.empty(n // block, dtype=torch.float16, device=dev)
        # (cleared once: the list's buffers are returned whole, and nothing is written behind its end)
        st["idx"] = torch.zeros(cap, dtype=torch.int64, device=dev) if cap else None
        st["val"] = torch.zeros(cap, dtype=torch.float16, device=dev) if cap else None
        st["out"] = torch.empty(n, dtype=torch.bfloat16, device=dev)
        st["counter"] = binding.pinned_counter()
    if case["op"] in ("step", "lloyd"):
        st["rec"] = binding.pinned_lloyd_stats()
    elif case["op"] == "mae":
        st["rec"] = binding.pinned_mae_stats()
    elif case["op"] == "error":
        st["rec"] = binding.pinned_error_stats()
    return st


def run(st):
    case, cb, T = st["case"], st["cb"], st["T"]
    block, signed, op = case["block"], case["signed"], case["op"]
    if op == "gemv":
        for r, c, codes, scales, tab, k, x, y, _ in st["layers"]:
            binding.bof4_gemv(codes, scales, r, c, block, cb, x, tab, k, out=y)
        return [layer[7] for layer in st["layers"]]
    if op == "gemm":
        for r, c, packed, _, tab, k, x, y, ws in st["layers"]:
            binding.bof4_gemm(packed, r, c, cb, x, tab, k, out=y, ws=ws)
        return [layer[7] for layer in st["layers"]]
    w, ws = st["w"], st["ws"]
    if op == "lloyd":
        rec = binding.bof4_lloyd_step(w, block, cb, signed, opq_T=T, ws=ws, out=st["rec"][0], raw=True)
        return rec.as_dict(), binding.bof4_codebook_update(rec, st["pin"], cb)
    if op == "mae":
        rec = binding.bof4_lloyd_step_mae(w, block, cb, signed, opq_T=T, skip_mask=st["pin"], ws=ws, out=st["rec"][0],
                                          raw=True)
        return rec.as_dict(), binding.bof4_codebook_update_mae(rec, st["pin"], cb)
    if op == "error":
        return binding.bof4_quant_error(w, block, cb, signed, opq_T=T, ws=ws, out=st["rec"][0])
    buffers = dict(codes=st["codes"], scales=st["scales"], out_idx=st["idx"], out_val=st["val"], ws=ws,
                   counter=st["counter"][0], trim=False)
    if op == "step":
        codes, scales, idx, val, k, rec = binding.bof4_quantize_lloyd(
            w, block, cb, signed, opq_T=T, out_capacity=st["cap"], stats=st["rec"][0], raw=True, **buffers)
        new_cb = binding.bof4_codebook_update(rec, st["pin"], cb)
        stats = rec.as_dict()
    else:
        codes, scales, idx, val, k = binding.bof4_quantize(w, block, cb, signed, opq_T=T, out_capacity=st["cap"], **buffers)
        new_cb = stats = None
    out = binding.bof4_dequantize(codes, scales, w.numel(), block, cb, idx, val, out=st["out"], n_outliers=k)
    return codes, scales, idx, val, k, stats, new_cb, out


# Share of the weights that the outlier rule stores (q = 0.95; heavy-tailed weights): for the bytes of the list.
_RHO = {"gauss": 0.0012, "t5": 0.0066, "t4": 0.0087, "planted": 0.0075}


def work(case):
    n, I, op = _n(case), case["block"], case["op"]
    rho = _RHO[case["dist"]] if case["opq"] else 0.0
    stored = 0.5 + 2.0 / I
    if op in ("lloyd", "mae", "error"):
        return {"bytes": 2.0 * n, "flops": 0.0}
    if op in ("step", "roundtrip"):  # weights in, quantised tensor out and in again, decoded weights out
        return {"bytes": n * (4.0 + 2.0 * (stored + 10.0 * rho)), "flops": 0.0}
    t = case["tokens"]
    io = sum(t * (2.0 * c + 4.0 * r) for r, c in _shapes(case))
    return {"bytes": n * (stored + 8.0 * rho) + io, "flops": 2.0 * n * t}


def tolerance(case):
    # Codes, constants, lists, counts, decoded weights and medians are exact whatever the tolerance of the sums says
    # (whole numbers compare as such; the rest comes out bit-equal).
    if case["op"] == "roundtrip":
        return "exact"
    if case["op"] in ("gemv", "gemm"):
        # binary32 sums over up to 28672 columns in any order: a product in binary32 that adds in one chain lies 1e-6 (largest
        # 2.6e-5) from binary64, the present kernels 1.4e-7
        return {"rel": 4e-6, "max": 1e-4}
    # binary64 sums in any order, x in fixed point of 2^-40: 6e-14 between the calls and from plain binary64 at 2^25
    # weights, where sse cancels two to three digits
    return {"rel": 1e-12, "max": 1e-12}
