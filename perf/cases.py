"""Measured workloads of the library: what a program that rearranges data on one
MI355X has it do, through the package's public entry points.

Every case is one call of one operation on tensors that already lie in device
memory.  ``listed`` names twelve of them, from a latency-bound transpose of
192 KiB to the 4096-job batch of 7.5 GB per side; ``draw`` gives more of the same
ranges, odd extents among them.  Moved bytes are opaque to the library, so
inputs are random bits held in integer tensors of the element's size; the
stencil, the one operation that computes, gets uniform values in [-1, 1).
"""
from __future__ import annotations

import math

import torch

import paper_1011_3583_amd as rr
import rr_synth

DEVICE = "cuda"
_DTYPE = {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}


def listed() -> list:
    return [
        # a matrix turned inside a larger program: launch and host latency
        {"name": "transpose_small", "kind": "permute", "dims": "256x192", "perm": "10", "esize": 4},
        # a batch of fp16 activations from channels-last to channels-first
        {"name": "nhwc_to_nchw_f16", "kind": "permute", "dims": "64x128x128x64", "perm": "0312", "esize": 2},
        # a volume read along its slowest axis (the reversed order of Table 1), fp32
        {"name": "reverse_3d_f32", "kind": "permute", "dims": "512x512x256", "perm": "210", "esize": 4},
        # the large out-of-cache matrix transpose, fp64 / complex64
        {"name": "transpose_16k_f64", "kind": "permute", "dims": "16384x16384", "perm": "10", "esize": 8},
        # a data cube with no round extent (records x steps x channels), fp16
        {"name": "cube_odd_f16", "kind": "permute", "dims": "4325x1001x31", "perm": "201", "esize": 2},
        # image preprocessing: the centre crop of a batch of RGB images, to planes
        {"name": "crop_hwc_to_chw_u8", "kind": "reorder", "dims": "256x256x256x3", "base": "0x16x16x0",
         "range": "256x224x224x3", "order": "0312", "esize": 1},
        # a point cloud's x, y, z arrays joined into records, an arbitrary number of points
        {"name": "interlace_xyz_f32", "kind": "interlace", "n": 3, "count": 10000019, "esize": 4},
        # nine interlaced fields split into arrays (the widest row of Table 3)
        {"name": "deinterlace_9_f32", "kind": "deinterlace", "n": 9, "count": 1 << 22, "esize": 4},
        # a random index set over a 1 GiB table
        {"name": "gather_random_f32", "kind": "gather", "src_count": 1 << 28, "count": 1 << 26, "esize": 4,
         "sorted": False},
        # the order-IV finite-difference Laplacian on Table 4's grid
        {"name": "stencil_fd4_4096", "kind": "stencil", "rows": 4096, "cols": 4096, "radius": 4, "shape": "star"},
        # a few hundred small jobs kept as a handle and replayed every step
        {"name": "batch_handle_256", "kind": "batch", "njobs": 256, "max_elements": 1000000, "mix": 256,
         "handle": True},
        # thousands of uneven jobs in one call: validated, planned, uploaded and run
        {"name": "batch_call_4096", "kind": "batch", "njobs": 4096, "max_elements": 10000000, "mix": 40960001,
         "handle": False},
    ]


# ----------------------------------------------------------------- drawing
def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _extents(rng, total, rank):
    """`rank` extents whose product is about `total`: round ones and odd ones."""
    shares = [rng.uniform(0.4, 1.6) for _ in range(rank)]
    s = sum(shares)
    dims = [max(2, round(total ** (x / s))) for x in shares]
    if rng.random() < 0.4:   # multiples of 16 where the extent allows it
        dims = [max(16, d // 16 * 16) if d >= 16 else d for d in dims]
    return dims


def _text(values):
    return "x".join(str(v) for v in values)


def draw(rng) -> dict:
    kind = rng.choice(["permute", "permute", "permute", "reorder", "interlace", "deinterlace", "gather", "stencil",
                       "batch"])
    if kind == "permute":   # 64 KiB to 1 GiB per side, ranks 2 to 5
        esize = rng.choice([1, 2, 4, 8, 16])
        rank = rng.randint(2, 5)
        dims = _extents(rng, _log_uniform(rng, 1 << 16, 1 << 30) / esize, rank)
        perm = list(range(rank))
        while perm[-1] == rank - 1 and perm == list(range(rank)):
            rng.shuffle(perm)
        return {"kind": kind, "dims": _text(dims), "perm": "".join(map(str, perm)), "esize": esize}
    if kind == "reorder":   # crops of image batches of 1, 3 or 4 channels, to planes
        h, w = rng.randint(64, 700), rng.randint(64, 700)
        c = rng.choice([1, 3, 3, 4])
        n = max(1, round(_log_uniform(rng, 1 << 18, 1 << 28) / (h * w * c)))
        rh, rw = rng.randint(h // 2, h), rng.randint(w // 2, w)
        return {"kind": kind, "dims": _text((n, h, w, c)), "base": _text((0, (h - rh) // 2, (w - rw) // 2, 0)),
                "range": _text((n, rh, rw, c)), "order": "0312", "esize": rng.choice([1, 1, 2, 4])}
    if kind in ("interlace", "deinterlace"):   # 2 to 16 sets, 1 MiB to 1 GiB in all
        n, esize = rng.randint(2, 16), rng.choice([1, 2, 4, 8])
        count = max(1, round(_log_uniform(rng, 1 << 20, 1 << 30) / (n * esize)))
        if rng.random() < 0.5:
            count = max(16, count // 16 * 16)
        return {"kind": kind, "n": n, "count": count, "esize": esize}
    if kind == "gather":   # index sets over tables of 1 MiB to 1 GiB
        esize = rng.choice([2, 4, 8, 16])
        src_count = round(_log_uniform(rng, 1 << 20, 1 << 30) / esize)
        return {"kind": kind, "src_count": src_count, "count": round(_log_uniform(rng, 1 << 12, 1 << 26)),
                "esize": esize, "sorted": rng.random() < 0.5}
    if kind == "stencil":   # grids from 256^2 to 16384^2
        shape = rng.choice(["star", "star", "box"])
        return {"kind": kind, "rows": round(_log_uniform(rng, 256, 16384)),
                "cols": round(_log_uniform(rng, 256, 16384)),
                "radius": rng.randint(1, 4) if shape == "star" else rng.randint(1, 2), "shape": shape}
    return {"kind": "batch", "njobs": round(_log_uniform(rng, 16, 2500)),
            "max_elements": round(_log_uniform(rng, 1e4, 5e6)), "mix": rng.randrange(1 << 30),
            "handle": rng.random() < 0.5}


# ----------------------------------------------------------------- inputs
def _ints(text):
    return tuple(int(v) for v in text.split("x"))


def _axes(text):
    return tuple(int(v) for v in text)


def _product(values):
    n = 1
    for v in values:
        n *= v
    return n


def _random(gen, count, esize):
    """`count` elements of `esize` random bytes (16-byte elements as pairs of int64)."""
    if esize == 16:
        return _random(gen, 2 * count, 8)
    words = torch.empty((count * esize + 7) // 8, dtype=torch.int64, device=DEVICE)
    words.random_(-(1 << 63), (1 << 63) - 1, generator=gen)
    return words.view(_DTYPE[esize])[:count]


def _zeros(count, esize):
    return _zeros(2 * count, 8) if esize == 16 else torch.zeros(count, dtype=_DTYPE[esize], device=DEVICE)


def _batch_specs(case):
    return rr_synth.sample_jobs(case["mix"], njobs=case["njobs"], total_range=(1e3, case["max_elements"]))


def _weights(case):
    r = case["radius"]
    if case["shape"] == "star":
        return [float(w) for w in rr_synth.FD_LAPLACIAN[r]]
    return [float(w) for w in rr_synth.rng(r).uniform(-1, 1, (2 * r + 1) ** 2).astype("float32")]


def _grid(case, gen):
    x = torch.rand(case["rows"], case["cols"], generator=gen, device=DEVICE, dtype=torch.float32)
    return x.mul_(2).sub_(1)


def _generator(seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    return gen


def prepare(case, seed):
    """The case's buffers (and, for a kept batch, its handle), inputs from the seed."""
    gen = _generator(seed)
    kind, s = case["kind"], {"case": case}
    if kind in ("permute", "reorder"):
        dims, e = _ints(case["dims"]), case["esize"]
        s.update(dims=dims, src=_random(gen, _product(dims), e))
        if kind == "permute":
            s["perm"] = _axes(case["perm"])
            s["dst"] = _zeros(_product(dims), e)
            if e != 16:
                s["src"] = s["src"].view(dims)
                s["dst"] = s["dst"].view([dims[p] for p in s["perm"]])
        else:
            s.update(base=_ints(case["base"]), range=_ints(case["range"]), order=_axes(case["order"]))
            s["dst"] = _zeros(_product(s["range"]), e).view([s["range"][a] for a in s["order"]])
    elif kind == "interlace":
        s["planes"] = [_random(gen, case["count"], case["esize"]) for _ in range(case["n"])]
        s["dst"] = _zeros(case["count"] * case["n"], case["esize"]).view(case["count"], case["n"])
    elif kind == "deinterlace":
        s["src"] = _random(gen, case["count"] * case["n"], case["esize"])
        s["planes"] = [_zeros(case["count"], case["esize"]) for _ in range(case["n"])]
    elif kind == "gather":
        s["src"] = _random(gen, case["src_count"], case["esize"])
        idx = torch.randint(0, case["src_count"], (case["count"],), generator=gen, device=DEVICE, dtype=torch.int64)
        s["idx"] = torch.sort(idx).values if case["sorted"] else idx
        s["dst"] = _zeros(case["count"], case["esize"])
        s["bad"] = torch.zeros(1, dtype=torch.int64, device=DEVICE)
    elif kind == "stencil":
        s["src"] = _grid(case, gen)
        s["dst"] = torch.zeros_like(s["src"])
        s["weights"] = _weights(case)
    else:
        specs = _batch_specs(case)
        offs, total = [], 0
        for j in specs:   # every job's buffers on 256-byte boundaries of two pools
            offs.append(total)
            total += -(-_product(j["dims"]) * j["esize"] // 256) * 256
        s["src"], s["dst"] = _random(gen, total // 8, 8), _zeros(total // 8, 8)
        s["jobs"] = rr.make_jobs([(s["dst"].data_ptr() + o, s["src"].data_ptr() + o, j["dims"], j["perm"], j["esize"])
                                  for o, j in zip(offs, specs)])
        if case["handle"]:
            s["batch"] = rr.Batch(s["jobs"], rr.RR_BATCH_GRAPH)
    return s


# ----------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    kind, e = case["kind"], case.get("esize")
    if kind == "permute":
        if e != 16:
            return rr.permute(s["src"], s["perm"], out=s["dst"])
        rr.check(rr.permute_raw(s["dst"].data_ptr(), s["src"].data_ptr(), s["dims"], s["perm"], 16, None))
        return s["dst"]
    if kind == "reorder":
        rr.check(rr.reorder_raw(s["dst"].data_ptr(), s["src"].data_ptr(), s["dims"], s["base"], s["range"],
                                s["order"], e, None))
        return s["dst"]
    if kind == "interlace":
        return rr.interlace(s["planes"], out=s["dst"])
    if kind == "deinterlace":
        return rr.deinterlace(s["src"], case["n"], outs=s["planes"])
    if kind == "gather":
        rr.check(rr.gather_raw(s["dst"].data_ptr(), s["src"].data_ptr(), case["src_count"], s["idx"].data_ptr(),
                               case["count"], e, s["bad"].data_ptr(), None))
        return [s["dst"], s["bad"]]
    if kind == "stencil":
        shape = rr.STENCIL_STAR if case["shape"] == "star" else rr.STENCIL_BOX
        rr.check(rr.stencil2d_raw(s["dst"].data_ptr(), s["src"].data_ptr(), case["rows"], case["cols"],
                                  case["radius"], s["weights"], shape, None))
        return s["dst"]
    if case["handle"]:
        s["batch"].launch()
    else:
        rr.check(rr.permute_batched_raw(s["jobs"], stream=None))
    return s["dst"]


# ----------------------------------------------------------------- what it cannot do without
def work(case):
    kind, e = case["kind"], case.get("esize")
    if kind == "permute":
        return {"bytes": 2 * e * _product(_ints(case["dims"])), "flops": 0}
    if kind == "reorder":
        return {"bytes": 2 * e * _product(_ints(case["range"])), "flops": 0}
    if kind in ("interlace", "deinterlace"):
        return {"bytes": 2 * e * case["n"] * case["count"], "flops": 0}
    if kind == "gather":
        return {"bytes": case["count"] * (8 + 2 * e), "flops": 0}
    if kind == "stencil":
        r, points = case["radius"], case["rows"] * case["cols"]
        per_point = 6 * r + 1 if case["shape"] == "star" else 2 * (2 * r + 1) ** 2
        return {"bytes": 8 * points, "flops": per_point * points}
    return {"bytes": 2 * sum(_product(j["dims"]) * j["esize"] for j in _batch_specs(case)), "flops": 0}


# ----------------------------------------------------------------- in 64 bits
def exact(case, seed):
    """The stencil's sums in fp64 (the library's fp32 weights and inputs, widened); the
    other operations compute nothing: their outputs are bytes moved unchanged."""
    if case["kind"] != "stencil":
        return None
    x = _grid(case, _generator(seed)).double()
    w = torch.tensor(_weights(case), dtype=torch.float32).double().tolist()
    r, (rows, cols) = case["radius"], x.shape
    out = x.clone()
    if rows <= 2 * r or cols <= 2 * r:
        return out

    def shifted(dy, dx):
        return x[r + dy:rows - r + dy, r + dx:cols - r + dx]

    if case["shape"] == "star":
        acc = w[0] * shifted(0, 0)
        for k in range(1, r + 1):
            acc += w[k] * (shifted(-k, 0) + shifted(k, 0) + shifted(0, -k) + shifted(0, k))
    else:
        acc = torch.zeros_like(shifted(0, 0))
        for i in range(2 * r + 1):
            for j in range(2 * r + 1):
                acc += w[i * (2 * r + 1) + j] * shifted(i - r, j - r)
    out[r:rows - r, r:cols - r] = acc
    return out
