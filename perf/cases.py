"""The work a user of this library has it do, as a list of timed cases.

Every case goes through the public entry points of `paper_2511_13061_amd` as the README uses them: products with
one vector (single, grouped by a decoder layer's dependences, a whole stack at once), products with a small batch of
vectors, conversion of a pruned dense matrix to the format and back.  Matrices are synthetic: N(0, 0.02) fp16
weights (times 32 and rounded to E4M3 for 8-bit values), either exactly the same number kept in every row, at random
places (what a per-output pruner such as Wanda leaves; `"mask": "rows"`), or every element kept independently
(`"mask": "iid"`).  They are drawn on the GPU from the seed.

  op      spmv    one product y = W x
          layer   the seven products of a decoder layer in the four launches its dependences allow
          stack   all products of several layers, independent of each other, in one call
          spmm    `batch` products with one matrix
          encode  dense -> format on the GPU, and back (the round trip that checks a conversion)
          decode  format -> dense on the GPU
          group   `n` independent products of one shape in one launch
  codes   bits per column code; vals: bits per stored value (16: fp16, 8: E4M3)
"""
import math

import torch

import paper_2511_13061_amd as M

SIGMA = 0.02
CELLS_MAX = 36864 * 12288            # the largest matrix
CELLS_SMALL = 11008 * 4096           # the largest matrix of the batch and conversion cases


def listed():
    def case(name, op, rows, cols, sparsity, mask="rows", codes=4, vals=16, **more):
        return dict(name=name, op=op, rows=rows, cols=cols, sparsity=sparsity, mask=mask, codes=codes, vals=vals, **more)

    return [
        # the smallest product: all of its time is latency (call, launch, the kernel's start)
        case("spmv_512x512_s50", "spmv", 512, 512, 0.5),
        # an attention projection of a 7B-shaped decoder layer, one token
        case("spmv_4096x4096_s50", "spmv", 4096, 4096, 0.5),
        # one decoding step's products of a Llama2-7B-shaped layer: {q,k,v} {o} {gate,up} {down}
        case("layer_7b_s50", "layer", 11008, 4096, 0.5),
        # the sweep matrix, the largest single product
        case("spmv_36864x12288_s50", "spmv", 36864, 12288, 0.5, mask="iid"),
        # high sparsity: short rows, a third of the stored entries is padding
        case("spmv_12288x12288_s95", "spmv", 12288, 12288, 0.95, mask="iid"),
        # nothing divides anything: odd row and column counts (a pruned or reshaped layer)
        case("spmv_11007x4093_s60", "spmv", 11007, 4093, 0.6, mask="iid"),
        # 8-bit values: an up / gate projection
        case("spmv_11008x4096_s50_e4m3", "spmv", 11008, 4096, 0.5, vals=8),
        # two Llama2-13B-shaped layers with 2-bit codes, 14 independent products in one call
        case("stack_13b_2layers_2bit", "stack", 13824, 5120, 0.5, mask="iid", codes=2, layers=2),
        # eight sequences decoded together: a down projection
        case("spmm_4096x11008_b8", "spmm", 4096, 11008, 0.5, batch=8),
        # the largest batch the library takes (a short prompt): an up / gate projection
        case("spmm_11008x4096_b64", "spmm", 11008, 4096, 0.5, batch=64),
        # converting a pruned weight when a model is loaded, and checking that it comes back
        case("encode_11008x4096_s50", "encode", 11008, 4096, 0.5),
        # the dense weight back for a compute-bound phase
        case("decode_4096x11008_s50", "decode", 4096, 11008, 0.5),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def size(lo, hi):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return n if rng.random() < 0.4 else max(8, n // 8 * 8)

    op = rng.choice(["spmv"] * 6 + ["group"] * 2 + ["spmm"] * 5 + ["encode"] * 2 + ["decode"] * 2)
    sparsity = round(rng.uniform(0.3, 0.97), 3)
    vals = 8 if rng.random() < 0.15 else 16
    # the code width that suits the sparsity (8-bit values come with 4-bit codes)
    codes = 4 if vals == 8 else rng.choice([1, 2, 4] if sparsity < 0.35 else [2, 4, 4] if sparsity < 0.55
                                           else [4] if sparsity < 0.9 else [4, 8])
    case = dict(op=op, sparsity=sparsity, mask=rng.choice(["rows", "iid"]), codes=codes, vals=vals)
    n = 1
    if op == "group":
        n = case["n"] = rng.randint(2, 4)
    if op == "spmm":
        case["batch"] = int(round(math.exp(rng.uniform(math.log(2), math.log(64)))))
    cap = (CELLS_MAX if op in ("spmv", "group") else CELLS_SMALL) // n
    hi = 36864 if op in ("spmv", "group") else 14336
    while True:
        rows, cols = size(256, hi), size(256, 14336)
        if rows * cols <= cap:
            return dict(case, rows=rows, cols=cols)


# ---- inputs -----------------------------------------------------------------

def _shapes(case):
    r, c = case["rows"], case["cols"]
    layer = [(c, c)] * 4 + [(r, c)] * 2 + [(c, r)]             # q k v o gate up down
    return {"layer": layer, "stack": layer * case.get("layers", 1), "group": [(r, c)] * case.get("n", 1)}.get(case["op"], [(r, c)])


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _dense(gen, case, rows, cols):
    """A pruned dense matrix on the GPU: fp16, or uint8 E4M3 bit patterns."""
    sparsity = case["sparsity"]
    u = torch.rand((rows, cols), generator=gen, device="cuda")
    if case["mask"] == "rows":
        keep = max(1, int(round(cols * (1.0 - sparsity))))
        kept = u <= u.kthvalue(keep, dim=1, keepdim=True).values
    else:
        kept = u >= sparsity
    w = torch.empty((rows, cols), dtype=torch.float16, device="cuda").normal_(0.0, SIGMA, generator=gen)
    w.mul_(kept)
    if case["vals"] == 8:
        return (w.float() * 32.0).to(torch.float8_e4m3fn).view(torch.uint8)
    return w


def _vectors(gen, n, cols):
    return torch.empty((n, cols), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=gen)


def _problem(case, seed):
    """(dense matrix, its x vectors) of every product, one after the other."""
    gen = _generator(seed)
    for i, (rows, cols) in enumerate(_shapes(case)):
        w = _dense(gen, case, rows, cols)
        yield w, _vectors(gen, case.get("batch", 1), cols)


def _encode(case, w):
    return M.encode_device_fp8(w) if case["vals"] == 8 else M.encode_device(w, b_delta=case["codes"])


def prepare(case, seed):
    op = case["op"]
    mats, xs = [], []
    for w, x in _problem(case, seed):
        mats.append(w if op == "encode" else _encode(case, w))
        xs.append(x)
    if op == "encode":
        return {"op": op, "case": case, "w": mats[0]}
    if op == "decode":
        return {"op": op, "m": mats[0]}
    if op == "spmm":
        return {"op": op, "m": mats[0], "x": xs[0]}
    xs = [x[0] for x in xs]
    if op == "spmv":
        return {"op": op, "m": mats[0], "x": xs[0]}
    if op == "layer":
        xs[1] = xs[2] = xs[0]                                  # q, k, v read the same vector, so do gate and up
        xs[5] = xs[4]
    ys = [torch.empty(m.rows, dtype=torch.float16, device="cuda") for m in mats]
    if op == "stack":
        return {"op": op, "calls": [M.SpmvMany(mats, xs, ys)], "y": ys}
    cuts = [(0, 3), (3, 4), (4, 6), (6, 7)] if op == "layer" else [(0, len(mats))]
    return {"op": op, "calls": [M.SpmvGroup(mats[a:b], xs[a:b], ys[a:b]) for a, b in cuts], "y": ys}


def run(state):
    op = state["op"]
    if op == "spmv":
        return state["m"].spmv(state["x"])
    if op == "spmm":
        return state["m"].spmm(state["x"])
    if op == "decode":
        return state["m"].decode_device()
    if op == "encode":
        m = _encode(state["case"], state["w"])
        r = m.report
        return {"dense": m.decode_device(), "nnz": r.nnz, "pad_nnz": r.pad_nnz, "alloc_nnz": r.alloc_nnz,
                "empty_rows": r.empty_rows, "max_row_entries": r.max_row_entries, "total_bytes": r.total_bytes}
    for call in state["calls"]:
        call.launch()
    return state["y"]


# ---- what a pass cannot do without -------------------------------------------

def _format_bytes(case, rows, cols):
    """Bytes of the three arrays: kept elements and the expected padding entries (a gap longer than the largest
    delta is bridged by entries of value zero)."""
    q = case["sparsity"]
    gap = q ** (2 ** case["codes"])
    entries = rows * cols * (1.0 - q) * (1.0 + gap / (1.0 - gap))
    return entries * (case["vals"] + case["codes"]) / 8.0 + 4.0 * (rows + 1)


def work(case):
    op, batch = case["op"], case.get("batch", 1)
    moved = flops = 0.0
    for rows, cols in _shapes(case):
        encoded, dense = _format_bytes(case, rows, cols), rows * cols * case["vals"] / 8.0
        if op == "encode":
            moved += dense + encoded + encoded + dense       # written once, and read once by the way back
        elif op == "decode":
            moved += encoded + dense
        else:
            moved += encoded + 2.0 * batch * (rows + cols)
            flops += 2.0 * batch * rows * cols * (1.0 - case["sparsity"])
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    if case["op"] in ("encode", "decode"):
        return "exact"                                         # the format is lossless
    # 32-bit sums rounded once to fp16: measured 2.1e-4 from 64 bits over all products, most of it that rounding
    return {"rel": 8e-4, "max": 4e-3}


# ---- the same in 64 bits -------------------------------------------------------

def _exact_product(case, w, x):
    out = torch.empty((x.shape[0], w.shape[0]), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 26) // w.shape[1])                     # 512 MB of doubles at a time
    xt = x.double().t().contiguous()
    for a in range(0, w.shape[0], step):
        piece = w[a:a + step]
        piece = piece.view(torch.float8_e4m3fn).float().double() if case["vals"] == 8 else piece.double()
        out[:, a:a + step] = (piece @ xt).t()
    return out


def exact(case, seed):
    op = case["op"]
    if op in ("encode", "decode"):
        w = next(iter(_problem(case, seed)))[0]
        if case["vals"] == 8:
            dense = torch.where((w & 0x7F) == 0, torch.zeros_like(w), w)     # bit patterns; -0 comes back as +0
        else:
            dense = w.double() + 0.0                           # -0 + 0 is +0
        return {"dense": dense, "nnz": None, "pad_nnz": None, "alloc_nnz": None, "empty_rows": None,
                "max_row_entries": None, "total_bytes": None} if op == "encode" else dense
    ys, first = [], {}
    for i, (w, x) in enumerate(_problem(case, seed)):
        if op == "layer":
            x = first.setdefault({1: 0, 2: 0, 5: 4}.get(i, i), x)
        ys.append(_exact_product(case, w, x))
    if op == "spmm":
        return ys[0]
    ys = [y[0] for y in ys]
    return ys[0] if op == "spmv" else ys
