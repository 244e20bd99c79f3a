"""The work that users of this package have it do, as cases that can be timed.

A case is one call (or one training step) through the public entry points:
decoding a material's queries, many materials at once, unpacking raw blocks,
and a training forward and backward. listed() covers the range from a handful
of picked points to a 4K frame and a 2^20-sample training batch; draw() gives
more of the same ranges. exact() evaluates a case in binary64 with plain torch.

Materials follow the shapes of the paper's Table 1 and of this repository's
benchmark: power-of-two pyramids of three channels with full mip chains or
chains that end at one 4x4 block, blocks of all 14 BC6H modes with endpoints
bounded so that texels stay of order one, MLP weights N(0, 1/fan_in).
"""
import math
import random
import re

import torch

import paper_2311_16121_amd as bcf

DEVICE = "cuda"
POOL = 1 << 14          # distinct blocks that a material's textures draw from


def listed():
    return [
        # a few picked points (a material picker, one shading probe): latency of one call
        {"name": "probe_fp32", "kind": "decode", "call": "decode", "sizes": "256,256,256,256", "chain": "full",
         "bias": "zero", "dims": "12-16-16-9", "precision": "FP32", "signed": False, "queries": "uniform", "n": 501,
         "grid": 0},
        # the smallest workload of the benchmark through the call that allocates nothing
        {"name": "tiny_noalloc_fp16", "kind": "decode", "call": "decode_noalloc", "sizes": "256,256,256,256",
         "chain": "full", "bias": "zero", "dims": "12-16-16-9", "precision": "FP16", "signed": False,
         "queries": "uniform", "n": 65536, "grid": 0},
        # a whole 4K frame, textures unpacked and decoded: the headline benchmark
        {"name": "frame4k_fp16", "kind": "decode", "call": "decode", "sizes": "2048,2048,2048,2048", "chain": "full",
         "bias": "zero", "dims": "12-32-32-10", "precision": "FP16", "signed": False, "queries": "frame",
         "n": 3840 * 2160, "grid": 3840},
        # a 1080p frame of a material that stays unpacked, at the default precision
        {"name": "frame1080_fp32", "kind": "decode", "call": "decode_unpacked", "sizes": "1024,1024,1024,1024",
         "chain": "full", "bias": "zero", "dims": "12-32-32-10", "precision": "FP32", "signed": False,
         "queries": "frame", "n": 1920 * 1080, "grid": 1920},
        # unordered points (ray hits, texture-space baking) through the precision sweep's wide decoder, in fp8
        {"name": "points_fp8", "kind": "decode", "call": "decode_unpacked", "sizes": "256,256,256,256",
         "chain": "full", "bias": "zero", "dims": "12-64-64-10", "precision": "FP8", "signed": False,
         "queries": "uniform", "n": (1 << 22) + 1, "grid": 0},
        # the paper's 2K configuration (pyramids of four sizes, eq. (10) biases) at an odd screen size, signed
        {"name": "mixed2k_bf16", "kind": "decode", "call": "decode", "sizes": "2048,1024,512,256", "chain": "blocks",
         "bias": "auto", "dims": "12-32-32-8", "precision": "BF16", "signed": True, "queries": "frame",
         "n": 1366 * 768, "grid": 1366},
        # three pyramids of one size, one hidden layer, exact weights on the matrix cores, a ragged point count
        {"name": "three_fp32_mfma", "kind": "decode", "call": "decode_unpacked", "sizes": "1024,1024,1024",
         "chain": "full", "bias": "zero", "dims": "9-32-10", "precision": "FP32_MFMA", "signed": False,
         "queries": "uniform", "n": 999983, "grid": 0},
        # a scene's materials in one go, only the touched blocks unpacked
        {"name": "batch_touched_fp16", "kind": "batch", "unpack": "touched", "materials": 24, "mix": 5,
         "res_min": 256, "res_max": 2048, "mixed": False, "dims": "12-32-32-10", "precision": "FP16",
         "log2_lo": 12.0, "log2_hi": 20.0},
        # fewer materials of the paper's mixed sizes, all unpacked, at full precision
        {"name": "batch_mixed_fp32", "kind": "batch", "unpack": "all", "materials": 6, "mix": 3, "res_min": 512,
         "res_max": 2048, "mixed": True, "dims": "12-16-16-10", "precision": "FP32", "log2_lo": 12.0,
         "log2_hi": 18.0},
        # one training step of the benchmark: 2^20 random samples, straight-through rounding
        {"name": "train_step", "kind": "train", "sizes": "1024,1024,1024,1024", "chain": "full", "bias": "minus1",
         "dims": "12-32-32-10", "straight": True, "n": 1 << 20, "uv": "random"},
        # an iteration as the paper samples it: a 512 x 512 uv grid, its 0.5K configuration, continuous parameters
        {"name": "train_grid_small", "kind": "train", "sizes": "512,256,128,64", "chain": "blocks", "bias": "auto",
         "dims": "12-16-16-8", "straight": False, "n": 512 * 512, "uv": "grid"},
        # raw blocks to halves, for export checks and for tools that want texels
        {"name": "blocks", "kind": "blocks", "n": 1000003, "signed": False},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["batch"] * 2 + ["train"] * 2 + ["blocks"])
    if kind == "blocks":
        return {"kind": kind, "n": _log_int(rng, 1000, 1000000), "signed": rng.random() < 0.5}
    if kind == "batch":
        lo = rng.choice([256, 512])
        return {"kind": kind, "unpack": rng.choice(["touched", "all"]), "materials": rng.randint(2, 20),
                "mix": rng.randint(0, 1 << 20), "res_min": lo, "res_max": rng.choice([1024, 2048]),
                "mixed": rng.random() < 0.4, "dims": rng.choice(["12-16-16-9", "12-32-32-10", "12-64-16"]),
                "precision": rng.choice(["FP16", "FP16", "FP32"]), "log2_lo": 11.0, "log2_hi": rng.uniform(13.0, 19.0)}
    n_tex = rng.choice([4, 4, 4, 3, 2, 1])
    shared = rng.random() < 0.6
    if kind == "train":
        top = rng.choice([256, 512, 1024])
        sizes = [top if shared else max(top >> t, 32) for t in range(n_tex)]
        h = rng.choice([16, 32])
        dims = [3 * n_tex] + [h] * rng.randint(1, 3) + [rng.randint(1, 12)]
        uv = rng.choice(["random", "grid"])
        n = rng.randint(64, 900) ** 2 if uv == "grid" else _log_int(rng, 2000, 900000)
        return {"kind": kind, "sizes": ",".join(map(str, sizes)), "chain": rng.choice(["full", "blocks"]),
                "bias": "zero" if shared else "auto", "dims": "-".join(map(str, dims)),
                "straight": rng.random() < 0.5, "n": n, "uv": uv}
    top = rng.choice([256, 512, 1024, 2048])
    sizes = [top if shared else max(top >> t, 64) for t in range(n_tex)]
    hidden = [rng.choice([16, 24, 32, 32, 64])] * rng.randint(1, 3)
    dims = [3 * n_tex] + hidden + [rng.choice([3, 7, 8, 9, 10, 10, 16])]
    call = rng.choice(["decode", "decode_unpacked", "decode_unpacked", "decode_noalloc"])
    if call == "decode_noalloc" and top == 2048:
        call = "decode"
    queries = rng.choice(["uniform", "frame"])
    if queries == "frame":
        grid = rng.randint(160, 1920)
        n = grid * rng.randint(90, 1080) - rng.choice([0, 0, rng.randint(1, grid - 1)])
    else:
        grid, n = 0, _log_int(rng, 1, 1 << 21)
    precision = rng.choice(["FP16", "FP16", "FP32", "FP32", "BF16", "FP8", "FP32_MFMA"])
    return {"kind": kind, "call": call, "sizes": ",".join(map(str, sizes)), "chain": rng.choice(["full", "blocks"]),
            "bias": "zero" if shared else "auto", "dims": "-".join(map(str, dims)), "precision": precision,
            "signed": precision != "FP8" and rng.random() < 0.25, "queries": queries, "n": n, "grid": grid}


# ---------------------------------------------------------------------------
# shapes

def _ints(text, sep):
    return [int(x) for x in text.split(sep)]


def _levels(size, chain):
    full = size.bit_length()                       # down to 1x1
    return full if chain == "full" else max(full - 2, 1)


def _biases(sizes, rule):
    if rule == "zero":
        return [0.0] * len(sizes)
    if rule == "minus1":                           # features at half the reference's resolution
        return [-1.0] * len(sizes)
    return [float(math.log2(s / sizes[0])) for s in sizes]


def _level_blocks(size, level):
    b = (max(size >> level, 1) + 3) // 4
    return b * b


def _chain_blocks(size, levels):
    return sum(_level_blocks(size, l) for l in range(levels))


def _batch_shapes(case):
    """[(sizes, query count)] of a batch's materials: the scene's, the same for every seed."""
    r = random.Random(case["mix"])
    tops = [1 << k for k in range(6, 16) if case["res_min"] <= 1 << k <= case["res_max"]]
    out = []
    for _ in range(case["materials"]):
        top = r.choice(tops)
        mixed = case["mixed"] and r.random() < 0.5
        out.append(([max(top >> t, 64) if mixed else top for t in range(4)],
                    int(2 ** r.uniform(case["log2_lo"], case["log2_hi"]))))
    return out


def _mlp_flops(dims):
    return 2 * sum(a * b for a, b in zip(dims[:-1], dims[1:]))


def work(case):
    """Every input read once and every output written once; the filter's 8
    taps per pyramid and channel and the MLP's products."""
    if case["kind"] == "blocks":
        return {"bytes": case["n"] * (16 + 96), "flops": 0}
    dims = _ints(case["dims"], "-")

    def decode(sizes, chain, n, unpacked):
        # the textures, but no more of them than the queries can touch
        taps = n * len(sizes) * 8
        blocks = sum(_chain_blocks(s, _levels(s, chain)) for s in sizes)
        tex = min(blocks * 16 * 6, taps * 6) if unpacked else 16 * min(blocks, taps)
        return tex + n * 12 + n * 4 * dims[-1], n * (_mlp_flops(dims) + len(sizes) * 3 * 8 * 2)

    if case["kind"] == "decode":
        b, f = decode(_ints(case["sizes"], ","), case["chain"], case["n"], case["call"] == "decode_unpacked")
        return {"bytes": b, "flops": f}
    if case["kind"] == "batch":
        parts = [decode(sizes, "full", n, False) for sizes, n in _batch_shapes(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    sizes, n = _ints(case["sizes"], ","), case["n"]
    blocks = sum(_chain_blocks(s, _levels(s, case["chain"])) for s in sizes)
    # parameters read and their gradients written, queries, targets, outputs and the loss's gradient
    return {"bytes": blocks * (2 * 4 * (12 + 16) + 1) + n * 12 + n * 4 * dims[-1] * 3,
            "flops": 3 * n * (_mlp_flops(dims) + len(sizes) * 3 * 8 * 2)}


# ---------------------------------------------------------------------------
# BC6H blocks (the format's layout strings), packed and unpacked with torch

_LAYOUT = {
    1: "m[1:0] gy[4] by[4] bz[4] rw[9:0] gw[9:0] bw[9:0] rx[4:0] gz[4] gy[3:0] gx[4:0] bz[0] "
       "gz[3:0] bx[4:0] bz[1] by[3:0] ry[4:0] bz[2] rz[4:0] bz[3] d[4:0]",
    2: "m[1:0] gy[5] gz[4] gz[5] rw[6:0] bz[0] bz[1] by[4] gw[6:0] by[5] bz[2] gy[4] bw[6:0] "
       "bz[3] bz[5] bz[4] rx[5:0] gy[3:0] gx[5:0] gz[3:0] bx[5:0] by[3:0] ry[5:0] rz[5:0] d[4:0]",
    3: "m[4:0] rw[9:0] gw[9:0] bw[9:0] rx[4:0] rw[10] gy[3:0] gx[3:0] gw[10] bz[0] gz[3:0] "
       "bx[3:0] bw[10] bz[1] by[3:0] ry[4:0] bz[2] rz[4:0] bz[3] d[4:0]",
    4: "m[4:0] rw[9:0] gw[9:0] bw[9:0] rx[3:0] rw[10] gz[4] gy[3:0] gx[4:0] gw[10] gz[3:0] "
       "bx[3:0] bw[10] bz[1] by[3:0] ry[3:0] bz[0] bz[2] rz[3:0] gy[4] bz[3] d[4:0]",
    5: "m[4:0] rw[9:0] gw[9:0] bw[9:0] rx[3:0] rw[10] by[4] gy[3:0] gx[3:0] gw[10] bz[0] "
       "gz[3:0] bx[4:0] bw[10] by[3:0] ry[3:0] bz[1] bz[2] rz[3:0] bz[4] bz[3] d[4:0]",
    6: "m[4:0] rw[8:0] by[4] gw[8:0] gy[4] bw[8:0] bz[4] rx[4:0] gz[4] gy[3:0] gx[4:0] bz[0] "
       "gz[3:0] bx[4:0] bz[1] by[3:0] ry[4:0] bz[2] rz[4:0] bz[3] d[4:0]",
    7: "m[4:0] rw[7:0] gz[4] by[4] gw[7:0] bz[2] gy[4] bw[7:0] bz[3] bz[4] rx[5:0] gy[3:0] "
       "gx[4:0] bz[0] gz[3:0] bx[4:0] bz[1] by[3:0] ry[5:0] rz[5:0] d[4:0]",
    8: "m[4:0] rw[7:0] bz[0] by[4] gw[7:0] gy[5] gy[4] bw[7:0] gz[5] bz[4] rx[4:0] gz[4] "
       "gy[3:0] gx[5:0] gz[3:0] bx[4:0] bz[1] by[3:0] ry[4:0] bz[2] rz[4:0] bz[3] d[4:0]",
    9: "m[4:0] rw[7:0] bz[1] by[4] gw[7:0] by[5] gy[4] bw[7:0] bz[5] bz[4] rx[4:0] gz[4] "
       "gy[3:0] gx[4:0] bz[0] gz[3:0] bx[5:0] by[3:0] ry[4:0] bz[2] rz[4:0] bz[3] d[4:0]",
    10: "m[4:0] rw[5:0] gz[4] bz[0] bz[1] by[4] gw[5:0] gy[5] by[5] bz[2] gy[4] bw[5:0] gz[5] "
        "bz[3] bz[5] bz[4] rx[5:0] gy[3:0] gx[5:0] gz[3:0] bx[5:0] by[3:0] ry[5:0] rz[5:0] d[4:0]",
    11: "m[4:0] rw[9:0] gw[9:0] bw[9:0] rx[9:0] gx[9:0] bx[9:0]",
    12: "m[4:0] rw[9:0] gw[9:0] bw[9:0] rx[8:0] rw[10] gx[8:0] gw[10] bx[8:0] bw[10]",
    13: "m[4:0] rw[9:0] gw[9:0] bw[9:0] rx[7:0] rw[10:11] gx[7:0] gw[10:11] bx[7:0] bw[10:11]",
    14: "m[4:0] rw[9:0] gw[9:0] bw[9:0] rx[3:0] rw[10:15] gx[3:0] gw[10:15] bx[3:0] bw[10:15]",
}
_CODE = {1: 0x00, 2: 0x01, 3: 0x02, 4: 0x06, 5: 0x0A, 6: 0x0E, 7: 0x12, 8: 0x16, 9: 0x1A, 10: 0x1E, 11: 0x03,
         12: 0x07, 13: 0x0B, 14: 0x0F}
# endpoint bits, stored widths of x/y/z per channel, transformed, subsets
_SHAPE = {1: (10, (5, 5, 5), 1, 2), 2: (7, (6, 6, 6), 1, 2), 3: (11, (5, 4, 4), 1, 2), 4: (11, (4, 5, 4), 1, 2),
          5: (11, (4, 4, 5), 1, 2), 6: (9, (5, 5, 5), 1, 2), 7: (8, (6, 5, 5), 1, 2), 8: (8, (5, 6, 5), 1, 2),
          9: (8, (5, 5, 6), 1, 2), 10: (6, (6, 6, 6), 0, 2), 11: (10, (10, 10, 10), 0, 1), 12: (11, (9, 9, 9), 1, 1),
          13: (12, (8, 8, 8), 1, 1), 14: (16, (4, 4, 4), 1, 1)}
_ANCHOR = (15,) * 17 + (2, 8, 2, 2, 8, 8, 15, 2, 8, 2, 2, 8, 8, 2, 2)
_MASK = (0xCCCC, 0x8888, 0xEEEE, 0xECC8, 0xC880, 0xFEEC, 0xFEC8, 0xEC80, 0xC800, 0xFFEC, 0xFE80, 0xE800, 0xFFE8,
         0xFF00, 0xFFF0, 0xF000, 0xF710, 0x008E, 0x7100, 0x08CE, 0x008C, 0x7310, 0x3100, 0x8CCE, 0x088C, 0x3110,
         0x6666, 0x366C, 0x17E8, 0x0FF0, 0x718E, 0x399C)


def _positions(mode):
    """[(field, bit of the field)] of header bits 0, 1, 2, ..."""
    out = []
    for name, a, b in re.findall(r"([a-z]+)\[(\d+)(?::(\d+))?\]", _LAYOUT[mode]):
        a, b = int(a), int(b) if b else int(a)
        step = 1 if a >= b else -1
        out += [(name, k) for k in range(b, a + step, step)]
    return out


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed) * 2654435761 % (1 << 31) + 11)


def _randint(g, lo, hi, shape):
    return torch.randint(lo, hi, shape, generator=g, device=DEVICE)


def _rand(g, shape, dtype=torch.float32):
    return torch.rand(shape, generator=g, device=DEVICE, dtype=dtype)


def _index_widths(subsets, part):
    """Stored index bits per texel [n, 16]: texel 0 and the second subset's anchor have one fewer."""
    n = part.shape[0]
    nb = torch.full((n, 16), 3 if subsets == 2 else 4, device=DEVICE)
    nb[:, 0] -= 1
    if subsets == 2:
        anchor = torch.tensor(_ANCHOR, device=DEVICE)[part]
        nb[torch.arange(n, device=DEVICE), anchor] -= 1
    return nb


def _pool(g, signed):
    """POOL blocks, their modes in turn: uint8 [POOL, 16] and the texels that
    the format decodes them to, half bit patterns as int64 [POOL, 16, 3]."""
    blocks = torch.empty((POOL, 16), dtype=torch.uint8, device=DEVICE)
    halves = torch.empty((POOL, 16, 3), dtype=torch.int64, device=DEVICE)
    for m in _LAYOUT:
        rows = torch.arange(m - 1, POOL, 14, device=DEVICE)
        n = rows.numel()
        bits, widths, transformed, subsets = _SHAPE[m]
        cap = int(0.48 * (1 << (bits - 1 if signed else bits)))
        low = -cap + 1 if signed else 0
        n_ep = 2 * subsets
        ends = torch.zeros((n, 4, 3), dtype=torch.int64, device=DEVICE)
        fields = {"m": torch.full((n,), _CODE[m], device=DEVICE)}
        for c, ch in enumerate("rgb"):
            base = _randint(g, low, cap, (n,))
            ends[:, 0, c] = base
            fields[ch + "w"] = base
            for j, name in enumerate("xyz"[:n_ep - 1]):
                if transformed:
                    half = 1 << (widths[c] - 1)
                    lo, hi = (base - half).clamp(min=low), (base + half - 1).clamp(max=cap - 1)
                    e = (lo + (_rand(g, (n,), torch.float64) * (hi - lo + 1)).long()).minimum(hi)
                    fields[ch + name] = e - base
                else:
                    e = _randint(g, low, cap, (n,))
                    fields[ch + name] = e
                ends[:, j + 1, c] = e
        part = _randint(g, 0, 32, (n,)) if subsets == 2 else torch.zeros(n, dtype=torch.int64, device=DEVICE)
        fields["d"] = part
        width = 3 if subsets == 2 else 4
        nb = _index_widths(subsets, part)
        idx = _randint(g, 0, 1 << width, (n, 16)) & ((1 << nb) - 1)
        # placed bit by bit (negative values as two's complement)
        out = torch.zeros((n, 129), dtype=torch.int64, device=DEVICE)     # 128: bits that are not stored
        head = _positions(m)
        for pos, (name, k) in enumerate(head):
            out[:, pos] = (fields[name] >> k) & 1
        first = len(head) + nb.cumsum(1) - nb
        for k in range(width):
            out.scatter_(1, torch.where(k < nb, first + k, torch.full_like(first, 128)), (idx >> k) & 1)
        weights = 1 << torch.arange(8, device=DEVICE)
        blocks[rows] = (out[:, :128].view(n, 16, 8) * weights).sum(-1).to(torch.uint8)
        # and decoded as the format says
        if signed:
            mag = ends.abs()
            top = (1 << (bits - 1)) - 1
            u = ((mag << 15) + 0x4000) >> (bits - 1)
            u = torch.where(mag == 0, 0, torch.where(mag >= top, 0x7FFF, u))
            u = ends if bits >= 16 else u * ends.sign()
        else:
            u = ((ends << 16) + 0x8000) >> bits
            u = torch.where(ends == 0, 0, torch.where(ends == (1 << bits) - 1, 0xFFFF, u))
            u = ends if bits >= 16 else u
        sub = ((torch.tensor(_MASK, device=DEVICE)[part][:, None] >> torch.arange(16, device=DEVICE)) & 1) * (subsets - 1)
        a = torch.gather(u, 1, (2 * sub)[:, :, None].expand(-1, -1, 3))
        b = torch.gather(u, 1, (2 * sub + 1)[:, :, None].expand(-1, -1, 3))
        wt = ((idx * (64 * 2) + (1 << width) - 1) // (2 * ((1 << width) - 1)))[:, :, None]
        v = ((64 - wt) * a + wt * b + 32) >> 6
        halves[rows] = (((v.abs() * 31) >> 5) | torch.where(v < 0, 0x8000, 0)) if signed else (v * 31) >> 6
    return blocks, halves


def _half_values(halves):
    """Half bit patterns to binary64, by the format's definition (finite ones)."""
    e, m = (halves >> 10) & 31, (halves & 1023).double()
    v = torch.where(e == 0, m * 2.0 ** -24, torch.ldexp(1.0 + m / 1024.0, (e - 15).double()))
    return torch.where(halves >= 0x8000, -v, v)


# ---------------------------------------------------------------------------
# inputs

def _params(g, dims):
    parts = []
    for a, b in zip(dims[:-1], dims[1:]):
        parts += [torch.randn(a * b, generator=g, device=DEVICE) / math.sqrt(a),
                  torch.randn(b, generator=g, device=DEVICE) / math.sqrt(a)]
    return torch.cat(parts)


def _uniform(g, n, s_max):
    q = _rand(g, (n, 3))
    q[:, 2] *= s_max
    return q


def _frame(g, n, grid, res, s_max):
    """A perspective view of a textured ground plane in scanline order, the
    scale from the uv derivatives; the camera's pitch and place drawn."""
    rows = (n + grid - 1) // grid
    pitch, u0, v0 = (float(x) for x in _rand(g, (3,), torch.float64))
    p = math.radians(39.0 + 2.0 * pitch)
    t = math.tan(math.radians(30.0))
    aspect = grid / rows
    px = torch.arange(grid, device=DEVICE, dtype=torch.float64) + 0.5
    py = torch.arange(rows, device=DEVICE, dtype=torch.float64) + 0.5
    a, b = (2 * px / grid - 1) * t * aspect, (1 - 2 * py / rows) * t
    depth = math.sin(p) - b * math.cos(p)
    dx = 2 * t * aspect / grid / depth
    dy = 2 * t / rows / depth ** 2
    tau = res * max(float(dx[-1]), float(dy[-1]))
    x = a[None, :] / depth[:, None]
    y = ((b * math.sin(p) + math.cos(p)) / depth)[:, None].expand_as(x)
    skew = a[None, :] * math.cos(p) * (2 * t / rows) / depth[:, None] ** 2
    scale = torch.maximum(dx[:, None].expand_as(x), (skew ** 2 + dy[:, None] ** 2).sqrt())
    q = torch.stack([x / tau + u0, y / tau + v0, torch.log2(scale * res / tau).clamp(0.0, s_max)], -1)
    q[..., :2] -= q[..., :2].floor()
    return q.reshape(-1, 3)[:n].float().contiguous()


def _textures(g, pool, sizes, levels):
    """Per pyramid the pool's rows that its blocks are, and the blocks."""
    rows = [_randint(g, 0, POOL, (_chain_blocks(s, l),)) for s, l in zip(sizes, levels)]
    return rows, [pool[r].reshape(-1) for r in rows]


def _decode_inputs(case, seed):
    g = _generator(seed)
    sizes, dims = _ints(case["sizes"], ","), _ints(case["dims"], "-")
    levels = [_levels(s, case["chain"]) for s in sizes]
    pool, halves = _pool(g, case["signed"])
    rows, blocks = _textures(g, pool, sizes, levels)
    params = _params(g, dims)
    s_max = float(levels[0] - 1)
    if case["queries"] == "frame":
        q = _frame(g, case["n"], case["grid"], sizes[0], s_max)
    else:
        q = _uniform(g, case["n"], s_max)
    return {"sizes": sizes, "levels": levels, "bias": _biases(sizes, case["bias"]), "dims": dims, "halves": halves,
            "rows": rows, "blocks": blocks, "params": params, "queries": q, "generator": g}


def _batch_inputs(case, seed):
    g = _generator(seed)
    dims = _ints(case["dims"], "-")
    pool, halves = _pool(g, False)
    mats, queries, counts = [], [], []
    for sizes, n in _batch_shapes(case):
        levels = [_levels(s, "full") for s in sizes]
        rows, blocks = _textures(g, pool, sizes, levels)
        mats.append({"sizes": sizes, "levels": levels, "bias": _biases(sizes, "auto"), "dims": dims, "rows": rows,
                     "blocks": blocks, "params": _params(g, dims), "halves": halves})
        queries.append(_uniform(g, n, float(levels[0] - 1)))
        counts.append(n)
    return mats, queries, counts


def _train_inputs(case, seed):
    g = _generator(seed)
    sizes, dims, n = _ints(case["sizes"], ","), _ints(case["dims"], "-"), case["n"]
    levels = [_levels(s, case["chain"]) for s in sizes]
    blocks = [_chain_blocks(s, l) for s, l in zip(sizes, levels)]
    q = _uniform(g, n, float(levels[0] - 1))
    if case["uv"] == "grid":                       # a jittered square grid, row by row
        side = math.isqrt(n)
        i = torch.arange(n, device=DEVICE)
        q[:, 0] = ((i % side) + q[:, 0]) / side
        q[:, 1] = ((i // side) + q[:, 1]) / side
    return {"sizes": sizes, "levels": levels, "bias": _biases(sizes, case["bias"]), "dims": dims,
            "ends": [31.0 * _rand(g, (b, 4, 3)) for b in blocks], "idxs": [_rand(g, (b, 16)) for b in blocks],
            "parts": [_randint(g, 0, 32, (b,)).to(torch.uint8) for b in blocks],
            "params": _params(g, dims), "queries": q, "target": _rand(g, (n, dims[-1]))}


# ---------------------------------------------------------------------------
# the calls

def prepare(case, seed):
    if case["kind"] == "blocks":
        g = _generator(seed)
        pool, _ = _pool(g, case["signed"])
        return {"case": case, "blocks": pool[_randint(g, 0, POOL, (case["n"],))]}
    if case["kind"] == "batch":
        mats, queries, counts = _batch_inputs(case, seed)
        batch = bcf.Batch([bcf.Material(m["blocks"], m["sizes"], m["levels"], m["dims"], m["params"], m["bias"])
                           for m in mats], bcf.Precision[case["precision"]])
        ends = torch.tensor([0] + counts).cumsum(0).to(torch.int32).to(DEVICE)
        return {"case": case, "batch": batch, "queries": torch.cat(queries), "offsets": ends}
    if case["kind"] == "train":
        x = _train_inputs(case, seed)
        geo = bcf.TrainGeometry(x["sizes"], x["levels"], x["parts"], x["dims"], x["bias"], case["straight"])
        leaves = [t.requires_grad_(True) for t in x["ends"] + x["idxs"] + [x["params"]]]
        return {"case": case, "geo": geo, "leaves": leaves, "queries": x["queries"], "target": x["target"]}
    x = _decode_inputs(case, seed)
    precision = bcf.Precision[case["precision"]]
    mat = bcf.Material(x["blocks"], x["sizes"], x["levels"], x["dims"], x["params"], x["bias"], case["signed"])
    if precision == bcf.Precision.FP8:
        mat.set_act_absmax(bcf.calibrate(mat, _uniform(x["generator"], 1 << 14, float(x["levels"][0] - 1))))
    state = {"case": case, "mat": mat, "precision": precision, "queries": x["queries"]}
    if case["call"] != "decode_noalloc":
        state["ws"] = bcf.prepare(mat, precision)
        if case["call"] == "decode_unpacked":
            bcf.unpack(mat, state["ws"])
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "blocks":
        return bcf.decode_blocks(state["blocks"], case["signed"])
    if case["kind"] == "batch":
        batch, q, offsets = state["batch"], state["queries"], state["offsets"]
        if case["unpack"] == "touched":
            batch.unpack_touched(q, offsets)
        else:
            batch.unpack()
        return batch.decode(q, offsets)
    if case["kind"] == "train":
        leaves, n = state["leaves"], len(state["geo"].sizes)
        out = bcf.train_decode(state["geo"], leaves[:n], leaves[n:2 * n], leaves[2 * n], state["queries"])
        loss = torch.nn.functional.mse_loss(out, state["target"])
        return {"out": out.detach(), "grads": list(torch.autograd.grad(loss, leaves))}
    if case["call"] == "decode_noalloc":
        return bcf.decode_noalloc(state["mat"], state["queries"], state["precision"], case["grid"])
    call = bcf.decode if case["call"] == "decode" else bcf.decode_unpacked
    return call(state["mat"], state["ws"], state["queries"], state["precision"], case["grid"])


# ---------------------------------------------------------------------------
# the same in binary64, with plain torch

def _level_tables(sizes, levels):
    """Per pyramid the (block, texel) of every level's texels, row-major, as
    block * 16 + texel, and each level's first entry and size."""
    out = []
    for s, n in zip(sizes, levels):
        first_block, parts, first, dims = 0, [], [0], []
        for l in range(n):
            w = max(s >> l, 1)
            bx = (w + 3) // 4
            y, x = torch.arange(w, device=DEVICE)[:, None], torch.arange(w, device=DEVICE)[None, :]
            parts.append(((first_block + (y >> 2) * bx + (x >> 2)) * 16 + (y & 3) * 4 + (x & 3)).reshape(-1))
            first.append(first[-1] + w * w)
            dims.append(w)
            first_block += bx * bx
        out.append((torch.cat(parts), torch.tensor(first[:-1], device=DEVICE), torch.tensor(dims, device=DEVICE)))
    return out


def _filter(texels, table, levels, bias, q):
    """Trilinear taps (eqs. (9), (10)) of one pyramid: [n, 3]."""
    _, first, dims = table
    u, v = q[:, 0] - q[:, 0].floor(), q[:, 1] - q[:, 1].floor()
    s = (q[:, 2] + bias).clamp(0.0, levels - 1)
    l0 = s.floor().long()
    lam = s - l0
    out = 0.0
    for l, lw in ((l0, 1.0 - lam), ((l0 + 1).clamp(max=levels - 1), lam)):
        w = dims[l]
        x, y = u * w - 0.5, v * w - 0.5
        x0, y0 = x.floor(), y.floor()
        fx, fy = x - x0, y - y0
        x0, y0 = x0.long(), y0.long()
        for dy, wy in ((0, 1.0 - fy), (1, fy)):
            for dx, wx in ((0, 1.0 - fx), (1, fx)):
                at = first[l] + ((y0 + dy) % w) * w + (x0 + dx) % w
                out = out + (lw * wx * wy)[:, None] * texels.index_select(0, at)
    return out


def _mlp(params, dims, z):
    at = 0
    for k, (a, b) in enumerate(zip(dims[:-1], dims[1:])):
        w, c = params[at:at + a * b].view(b, a), params[at + a * b:at + a * b + b]
        at += a * b + b
        z = torch.nn.functional.linear(z, w, c)
        z = torch.relu(z) if k < len(dims) - 2 else z
    return z


def _exact_decode(x, q):
    tables = _level_tables(x["sizes"], x["levels"])
    pool = _half_values(x["halves"])
    texels = [pool[r].reshape(-1, 3)[t[0]] for r, t in zip(x["rows"], tables)]
    params, out = x["params"].double(), []
    for part in q.double().split(1 << 20):
        z = [_filter(f, t, l, b, part) for f, t, l, b in zip(texels, tables, x["levels"], x["bias"])]
        out.append(_mlp(params, x["dims"], torch.cat(z, 1)))
    return torch.cat(out)


def _half_of(y):
    """eq. (8) of y, its step held constant, and its slope."""
    h = (((y.detach() - 1.0) / 1024.0).floor() - 1.0).clamp(min=0.0)
    return torch.exp2(h - 14.0) * (y / 1024.0 - h), torch.exp2(h - 24.0)


def _train_texels(ends, idxs, parts, straight):
    """Block parameters to texels [blocks * 16, 3]: eqs. (6)-(8), continuous
    or straight-through (the exported block's value, the continuous slopes at
    its rounded parameters)."""
    sub = (torch.tensor(_MASK, device=DEVICE)[parts.long()][:, None] >> torch.arange(16, device=DEVICE)) & 1
    at = (2 * sub)[:, :, None].expand(-1, -1, 3)
    scale = 31.0 / 64.0

    def blend(a, b, x):
        return scale * (1024.0 * a + 512.0 + x * 1024.0 * (b - a))

    if not straight:
        e, x = ends.double(), idxs.double()[:, :, None]
        return _half_of(blend(e.gather(1, at), e.gather(1, at + 1), x))[0].reshape(-1, 3)
    e = ends.detach().round().clamp(0, 63).long()
    i = (7.0 * idxs.detach().float()).round().clamp(0, 7).long()        # the product in binary32, as the method says
    u = torch.where(e == 0, 0, torch.where(e == 63, 0xFFFF, ((e << 16) + 0x8000) >> 6))
    wt = ((i * 128 + 7) // 14)[:, :, None]
    v = ((64 - wt) * u.gather(1, at) + wt * u.gather(1, at + 1) + 32) >> 6
    value, slope = _half_of(((v * 31) >> 6).double())
    es = ends.double() + (e.double() - ends.double()).detach()
    xs = idxs.double() + (wt[:, :, 0].double() / 64.0 - idxs.double()).detach()
    y = blend(es.gather(1, at), es.gather(1, at + 1), xs[:, :, None])
    return (value + slope * (y - y.detach())).reshape(-1, 3)


def exact(case, seed):
    if case["kind"] == "blocks":
        g = _generator(seed)
        _, halves = _pool(g, case["signed"])
        return halves.to(torch.int16)[_randint(g, 0, POOL, (case["n"],))]
    if case["kind"] == "batch":
        mats, queries, _ = _batch_inputs(case, seed)
        return torch.cat([_exact_decode(m, q) for m, q in zip(mats, queries)])
    if case["kind"] == "decode":
        x = _decode_inputs(case, seed)
        return _exact_decode(x, x["queries"])
    x = _train_inputs(case, seed)
    x["ends"], x["idxs"] = ([t.double().requires_grad_(True) for t in x[k]] for k in ("ends", "idxs"))
    tables = _level_tables(x["sizes"], x["levels"])
    texels = [_train_texels(e, i, p, case["straight"]).index_select(0, t[0])
              for e, i, p, t in zip(x["ends"], x["idxs"], x["parts"], tables)]
    cut = [t.detach().requires_grad_(True) for t in texels]
    weights = x["params"].double().detach().requires_grad_(True)
    total, out = x["target"].numel(), []
    for q, target in zip(x["queries"].double().split(1 << 18), x["target"].double().split(1 << 18)):
        z = [_filter(f, t, l, b, q) for f, t, l, b in zip(cut, tables, x["levels"], x["bias"])]
        y = _mlp(weights, x["dims"], torch.cat(z, 1))
        ((y - target).square().sum() / total).backward()
        out.append(y.detach())
    grads = torch.autograd.grad(texels, x["ends"] + x["idxs"], [c.grad for c in cut])
    return {"out": torch.cat(out), "grads": list(grads) + [weights.grad]}
