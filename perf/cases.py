"""The work that a program using this library has it do, as a list of cases that can be timed.

The matrices are those of the LLaMA-3.2 shapes that inputs/synth.py and bench.py name (1B: hidden 2048, key/value 512,
feed-forward 8192; 3B: 3072, 1024, 8192), filled with the same kinds of values: 0.02 * N(0, 1) or 0.02 * t(4), quantized per
row and dictionary-coded by the library's own encoder, one dictionary over the sequence of matrices, as bench.py does.

Kinds of case:
  linear   one product, tq_matvec: a single projection, the smallest call there is
  layer    the seven projections of one layer, tq_matvec_multi
  pairs    gate/up pairs with silu(gate) * up fused in, tq_matvec_gate_up_multi
  step     all products of several layers as one prepared step (a decode step of the model)
  staged   the same products in the order a layer's dependencies allow, one prepared step
  expand   the un-fused form: whole int8 matrices, a prepared expansion
  listing  a parameter in the stream format of the paper's section 4 listings, expanded on the device
  encode   the host encoder: fp32 matrix -> container bytes
"""
import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2509_22951_amd as tq

WORKERS = 8      # encoder threads side by side, as many as bench.py takes
CHAIN = 7        # matrices after which a dictionary that has not filled up is taken as it is (one layer, as in bench.py)


def listed():
    return [
        # a single projection at batch 1: launch, staging and tail count more than bandwidth
        {"name": "linear_2048_b1", "kind": "linear", "rows": 2048, "cols": 2048, "bits": 8, "dist": "normal", "batch": 1},
        # a model with widths that are no multiple of anything (odd rows, odd columns), a few sequences side by side
        {"name": "linear_odd_b5", "kind": "linear", "rows": 4099, "cols": 2999, "bits": 8, "dist": "normal", "batch": 5},
        # one LLaMA-3.2-1B layer, one token
        {"name": "layer_1b_b1", "kind": "layer", "hidden": 2048, "kv": 512, "inter": 8192, "bits": 8, "dist": "normal", "batch": 1},
        # one LLaMA-3.2-3B layer, eight sequences: what a server that runs layer by layer launches
        {"name": "layer_3b_b8", "kind": "layer", "hidden": 3072, "kv": 1024, "inter": 8192, "bits": 8, "dist": "normal", "batch": 8},
        # the gated pairs of eight 3B feed-forward blocks, heavy-tailed weights, the largest batch
        {"name": "pairs_3b_t4_b16", "kind": "pairs", "layers": 8, "hidden": 3072, "inter": 8192, "bits": 8, "dist": "student_t4", "batch": 16},
        # one token through the whole of LLaMA-3.2-1B: 16 layers and the output projection, 113 matrices, 1.24 G weights
        {"name": "step_1b_b1", "kind": "step", "layers": 16, "hidden": 2048, "kv": 512, "inter": 8192, "vocab": 128256, "bits": 8, "dist": "normal",
         "batch": 1},
        # eight layers of LLaMA-3.2-3B, eight sequences
        {"name": "step_3b_b8", "kind": "step", "layers": 8, "hidden": 3072, "kv": 1024, "inter": 8192, "vocab": 0, "bits": 8, "dist": "normal", "batch": 8},
        # the same layers with 4-bit weights, two to a byte, one token
        {"name": "step_3b_4bit_b1", "kind": "step", "layers": 8, "hidden": 3072, "kv": 1024, "inter": 8192, "vocab": 0, "bits": 4, "dist": "normal",
         "batch": 1},
        # one token through four 3B layers with the dependencies of a real layer: q,k,v | o | gate,up | down, 16 stages
        {"name": "staged_3b_b1", "kind": "staged", "layers": 4, "hidden": 3072, "kv": 1024, "inter": 8192, "bits": 8, "dist": "normal", "batch": 1},
        # four 3B layers expanded to int8 matrices
        {"name": "expand_3b", "kind": "expand", "layers": 4, "hidden": 3072, "kv": 1024, "inter": 8192, "bits": 8, "dist": "normal"},
        # a 3B gate projection in the paper's printed format
        {"name": "listing_gate_3b", "kind": "listing", "values": 8192 * 3072, "table_values": 1 << 20, "bits": 8, "dist": "normal"},
        # encoding one 2048 x 2048 matrix with a dictionary of its own
        {"name": "encode_2048", "kind": "encode", "rows": 2048, "cols": 2048, "bits": 8, "dist": "normal"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A matrix dimension: a multiple of 256 or 64, or any number."""
    v = _log_uniform(rng, lo, hi)
    step = rng.choice([256, 64, 1])
    return max(step, v // step * step)


def draw(rng):
    kind = rng.choice(["linear", "linear", "layer", "pairs", "step", "step", "staged", "expand", "listing", "encode"])
    dist = rng.choice(["normal", "normal", "student_t4"])
    bits = rng.choice([8, 8, 4])
    batch = rng.choice([1, 1, 2, 3, 4, 5, 8, 12, 16])
    if kind in ("linear", "encode"):
        cols = _width(rng, 256, 8192 if kind == "linear" else 4096)
        case = {"kind": kind, "rows": _width(rng, 256, 16384 if kind == "linear" else 4096), "cols": cols + cols % 2 if bits == 4 else cols,
                "bits": bits, "dist": dist}
        return dict(case, batch=batch) if kind == "linear" else case
    if kind == "listing":
        return {"kind": kind, "values": _log_uniform(rng, 1 << 16, 8192 * 3072), "table_values": 1 << rng.randint(14, 20),
                "bits": rng.choice([8, 4, 2]), "dist": dist}
    hidden = _width(rng, 1024, 3072)
    inter = _width(rng, 2 * hidden, 8192)
    if bits == 4:      # two columns to a byte: an even number of them
        hidden, inter = hidden + hidden % 2, inter + inter % 2
    case = {"kind": kind, "hidden": hidden, "inter": inter, "bits": bits, "dist": dist}
    if kind != "pairs":
        case["kv"] = max(64, hidden // rng.choice([3, 4]) // 64 * 64)
    if kind == "layer":
        return dict(case, batch=batch)
    if kind == "pairs":
        return dict(case, layers=rng.randint(1, 8), batch=batch)
    if kind == "staged":
        return dict(case, layers=rng.randint(1, 4), batch=rng.choice([1, 1, 1, 2]))
    if kind == "expand":
        return dict(case, layers=rng.randint(1, 4))
    return dict(case, layers=rng.randint(2, 8), vocab=rng.choice([0, 32000]), batch=batch)


# ---- matrices of a case --------------------------------------------------------------------------------------------

def _shapes(case):
    """(rows, cols) of the matrices, in order."""
    kind = case["kind"]
    if kind in ("linear", "encode"):
        return [(case["rows"], case["cols"])]
    h, inter = case["hidden"], case["inter"]
    if kind == "pairs":
        return [(inter, h)] * (2 * case["layers"])
    one = [(h, h), (case["kv"], h), (case["kv"], h), (h, h), (inter, h), (inter, h), (h, inter)]
    return one * case.get("layers", 1) + ([(case["vocab"], h)] if case.get("vocab") else [])


def _stages(case):
    one = [0, 0, 0, 1, 2, 2, 3]      # q, k, v | o | gate, up | down
    return [4 * layer + s for layer in range(case["layers"]) for s in one]


def _weights(case, seed, index, rows, cols):
    """fp32 weights of one matrix, on the GPU, a function of (seed, index) alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * seed + index)
    w = torch.randn((rows, cols), generator=g, device="cuda", dtype=torch.float32)
    if case["dist"] == "student_t4":      # z / sqrt(chi2_4 / 4), chi2_4 = -2 ln(u1 u2)
        for _ in range(2):
            u = 1.0 - torch.rand((rows, cols), generator=g, device="cuda", dtype=torch.float32)
            chi = u if _ == 0 else chi * u
        w /= torch.sqrt(-0.5 * torch.log(chi))
    return w * 0.02


def _activations(seed, index, batch, cols):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * seed + 500_000 + index)
    return torch.randn((batch, cols), generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)


def _quantized(w, bits):
    """The library's quantizer in plain torch: per row, symmetric, round half to even -> (int8 values, fp32 scales)."""
    qmax = float(2 ** (bits - 1) - 1)
    scale = w.abs().amax(dim=1)
    scale = scale / torch.full_like(scale, qmax)      # (a division by a number would be a product with its inverse)
    safe = torch.where(scale > 0, scale, torch.ones_like(scale))
    return torch.clamp(torch.round(w / safe[:, None]), -qmax, qmax).to(torch.int8), scale


def _encoded(case, seed, n, encode_one):
    """n containers as resident matrices, one dictionary over the sequence: one after the other until the dictionary is
    full (or a layer is through), the others from that dictionary side by side."""
    opts = {"bits": case["bits"], "pack": case["bits"] == 4}
    mats, prev = [], None
    while len(mats) < min(n, CHAIN):
        prev = encode_one(len(mats), dict(opts, dict_from=prev))
        mats.append(tq.Matrix(prev))
        if mats[-1].info["n_entries"] == tq.TQ_MAX_ENTRIES_DEVICE:
            break
    if len(mats) < n:
        opts = dict(opts, dict_from=prev, max_entries=mats[-1].info["n_entries"], n_threads=2)
        with ThreadPoolExecutor(WORKERS) as pool:
            mats += [tq.Matrix(blob) for blob in pool.map(lambda i: encode_one(i, opts), range(len(mats), n))]
    return mats


def _outputs(batch, rows, dtype, values=None):
    """Output matrices [batch, rows], seven to a buffer (a layer's), each on a 256-byte boundary -> (buffers, matrices).
    Elements between two matrices are zero."""
    buffers, views = [], []
    for first in range(0, len(rows), 7):
        part = rows[first:first + 7]
        starts = [0]
        for r in part:
            starts.append(starts[-1] + -(-batch * r // 64) * 64)
        buffers.append(torch.zeros(starts[-1], dtype=dtype, device="cuda"))
        views += [buffers[-1][s:s + batch * r].view(batch, r) for s, r in zip(starts, part)]
    if values is not None:
        for view, v in zip(views, values):
            view.copy_(v)
    return buffers, views


def _stream():
    return torch.cuda.current_stream().cuda_stream


def prepare(case, seed):
    kind = case["kind"]
    if kind == "listing":
        values, table = _listing_inputs(case, seed)
        h = tq.Listing(tq.tq_listing_compress(values, table), table)
        return {"case": case, "listing": h, "out": torch.empty(values.size, dtype=torch.uint8, device="cuda")}
    shapes = _shapes(case)

    def host_weights(i):
        return _weights(case, seed, i, *shapes[i]).cpu().numpy()

    if kind == "encode":
        # room for any container of this shape: a code per weight, padding, dictionary, offsets and scales
        return {"case": case, "w": host_weights(0), "out": np.zeros(int(2.5 * case["rows"] * (case["cols"] + 1024)) + (1 << 18), dtype=np.uint8)}
    if kind == "pairs":
        mats = _encoded(case, seed, len(shapes) // 2, lambda i, o: tq.tq_encode_gate_up(host_weights(2 * i), host_weights(2 * i + 1), **o))
        shapes = shapes[::2]
    else:
        mats = _encoded(case, seed, len(shapes), lambda i, o: tq.tq_encode(host_weights(i), **o))
    state = {"case": case, "mats": mats}
    handles = [m.handle for m in mats]
    if kind == "expand":
        state["out"] = [torch.empty(s, dtype=torch.int8, device="cuda") for s in shapes]
        state["step"] = tq.Step(handles, None, [o.data_ptr() for o in state["out"]], decompress=True)
        return state
    batch = case["batch"]
    state["x"] = [_activations(seed, i, batch, c) for i, (_, c) in enumerate(shapes)]
    state["out"], ys = _outputs(batch, [r for r, _ in shapes], torch.float32)
    xs, ys = [x.data_ptr() for x in state["x"]], [y.data_ptr() for y in ys]
    if kind == "layer":
        state["call"] = tq.MultiCall(handles, xs, ys, batch)
    elif kind == "pairs":
        state["args"] = (handles, xs, ys, batch)
    elif kind == "step":
        state["step"] = tq.Step(handles, xs, ys, batch)
    elif kind == "staged":
        state["step"] = tq.Step(handles, xs, ys, batch, stages=_stages(case))
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "linear":
        state["mats"][0].matvec(state["x"][0].data_ptr(), state["out"][0].data_ptr(), case["batch"], _stream())
    elif kind == "layer":
        state["call"].launch(_stream())
    elif kind == "pairs":
        tq.tq_matvec_gate_up_multi(*state["args"], _stream())
    elif kind in ("step", "staged", "expand"):
        state["step"].launch(_stream())
    elif kind == "listing":
        state["listing"].decompress(state["out"].data_ptr(), _stream())
    else:
        blob = tq.tq_encode(state["w"], bits=case["bits"], pack=case["bits"] == 4)
        state["out"][:len(blob)] = np.frombuffer(blob, dtype=np.uint8)
    return state["out"]


def _listing_inputs(case, seed):
    """Quantized values of one parameter as bytes, and a table made over the start of another one."""
    rows = -(-case["values"] // 3072)
    values = _quantized(_weights(case, seed, 0, rows, 3072), case["bits"])[0].cpu().numpy().view(np.uint8).reshape(-1)[:case["values"]]
    rows = -(-case["table_values"] // 3072)
    other = _quantized(_weights(case, seed, 1, rows, 3072), case["bits"])[0].cpu().numpy().view(np.uint8).reshape(-1)[:case["table_values"]]
    return values, tq.tq_listing_build_table([other])


# Bytes per weight of the coded matrices without padding: two-weight codes but for the singles among them (8 bits,
# Gaussian: 1.958 weights per code, Student-t: 1.999); packed 4 bits: two codes' worth of weights in two bytes.
_BYTES_PER_WEIGHT = {(8, "normal"): 2 / 1.958, (8, "student_t4"): 2 / 1.999, (4, "normal"): 0.5016, (4, "student_t4"): 0.5016}
# Words per value of a listing stream: 8 bits nearly all escaped (5 words for 4 values), 2 and 4 bits nearly all codewords
_WORDS_PER_VALUE = {8: 1.25, 4: 0.3, 2: 0.25}


def work(case):
    kind, n = case["kind"], 0
    if kind == "listing":
        return {"bytes": case["values"] * (2 * _WORDS_PER_VALUE[case["bits"]] + 1), "flops": 0}
    shapes = _shapes(case)
    n = sum(r * c for r, c in shapes)
    coded = n * _BYTES_PER_WEIGHT[case["bits"], case["dist"]] + sum(4 * r for r, _ in shapes)
    if kind == "encode":
        return {"bytes": 4 * n + coded, "flops": 0}
    if kind == "expand":
        return {"bytes": coded + n, "flops": 0}
    b = case["batch"]
    if kind == "pairs":
        io = sum(b * (2 * c + 4 * r) for r, c in shapes[::2])
    else:
        io = sum(b * (2 * c + 4 * r) for r, c in shapes)
    return {"bytes": coded + io, "flops": 2 * n * b}


def tolerance(case):
    if case["kind"] in ("expand", "listing", "encode"):
        return "exact"
    # fp32 sums of products that are themselves exact in fp32 (8-bit weight times bf16), in any order.  Measured against
    # 64 bits: 0.6e-7 .. 1.2e-7 with sums split over lanes as the kernels do it; one single chain over 8192 columns
    # shows 2.8e-7, its worst output 1.15e-6.
    return {"rel": 1e-6, "max": 5e-6}


def exact(case, seed):
    kind = case["kind"]
    if kind == "encode":
        return None
    if kind == "listing":
        return torch.from_numpy(_listing_inputs(case, seed)[0].copy())
    shapes = _shapes(case)
    if kind == "expand":
        return [_quantized(_weights(case, seed, i, *s), case["bits"])[0] for i, s in enumerate(shapes)]

    def product(i, x):
        q, scale = _quantized(_weights(case, seed, i, *shapes[i]), case["bits"])
        return (x @ q.to(torch.float64).T.contiguous()) * scale.to(torch.float64)

    out = []
    if kind == "pairs":
        for i in range(len(shapes) // 2):
            x = _activations(seed, i, case["batch"], shapes[2 * i][1]).to(torch.float64)
            gate, up = product(2 * i, x), product(2 * i + 1, x)
            out.append(gate / (1.0 + torch.exp(-gate)) * up)
    else:
        for i, (_, c) in enumerate(shapes):
            out.append(product(i, _activations(seed, i, case["batch"], c).to(torch.float64)))
    return _outputs(case["batch"], [y.shape[1] for y in out], torch.float64, out)[0]
