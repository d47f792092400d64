"""The calls that a program makes of this decoder, for timing and for comparing outputs.

Each case goes through the package's public entry points on inputs made here
from a seed: synthetic photographs (smooth gradients, plane waves, noise),
forward-transformed and quantised with the example tables of ITU-T T.81
Annex K, and for the bitstream cases Huffman-coded with that annex's tables
into baseline JPEG files.  Everything but the file headers is made on the GPU.

Kinds of case:
  decode      one image of coefficients in device memory -> RGB8
  batch       many images in one planned launch (a plan that a program keeps)
  calls       many small images in one call that plans and launches each time
  variant     the other IDCT methods and samplings, grayscale, scaled output
  corpus      bitstreams already in device memory -> coefficients -> RGB8,
              with both plans kept
  file        one JPEG file in host memory -> RGB8 on the GPU, the whole call
"""
import math
import random
import struct

import numpy as np
import torch

import paper_1311_5304_amd as M

DEV = "cuda:0"
LUMA = {"444": (1, 1), "422": (2, 1), "420": (2, 2), "440": (1, 2), "411": (4, 1)}
_ctx = None


def _context():
    """One context for the process, as a program keeps it."""
    global _ctx
    if _ctx is None:
        _ctx = M.Context(0)
    return _ctx


# ---- the cases --------------------------------------------------------------------------

def listed():
    return [
        # a thumbnail-sized image alone: launch and latency
        {"name": "small_420", "kind": "decode", "width": 256, "height": 256, "sampling": "420", "quality": 75,
         "mode": "simple"},
        # a video-sized frame whose sides are no multiple of the MCU, the rows at odd addresses
        {"name": "hd_422", "kind": "decode", "width": 1921, "height": 1081, "sampling": "422", "quality": 90,
         "mode": "fancy"},
        # a 12 megapixel photograph: the size the benchmark is quoted on
        {"name": "photo_420", "kind": "decode", "width": 4096, "height": 3072, "sampling": "420", "quality": 90,
         "mode": "fancy"},
        # mixed images of a data loader's batch, decoded again and again through a kept plan
        {"name": "batch_mixed", "kind": "batch", "count": 48, "low": 320, "high": 4096, "mode": "fancy"},
        # a page of previews: small images, one call that plans as well
        {"name": "batch_small", "kind": "calls", "count": 32, "low": 64, "high": 640, "mode": "fancy"},
        # the floating-point IDCT on the same photograph
        {"name": "photo_float", "kind": "variant", "width": 4096, "height": 3072, "sampling": "420", "quality": 90,
         "mode": "fancy", "idct": "float", "scale": 1},
        # a scanned page: grayscale, ragged
        {"name": "page_gray", "kind": "variant", "width": 4093, "height": 3070, "sampling": "gray", "quality": 85,
         "mode": "fancy", "idct": "islow", "scale": 1},
        # a screen-sized view of a photograph
        {"name": "half_420", "kind": "variant", "width": 4096, "height": 3072, "sampling": "420", "quality": 90,
         "mode": "fancy", "idct": "islow", "scale": 2},
        # the thumbnail of a 24 megapixel photograph
        {"name": "thumb_422", "kind": "variant", "width": 6000, "height": 4000, "sampling": "422", "quality": 90,
         "mode": "fancy", "idct": "islow", "scale": 8},
        # a corpus of files written for parallel decoding: a marker every 32 MCUs
        {"name": "corpus", "kind": "corpus", "count": 12, "low_mp": 1.0, "high_mp": 12.0, "quality": 85,
         "interval": 32, "mode": "fancy"},
        # one photograph as cameras write it: a marker at the end of each MCU row
        {"name": "file_rows", "kind": "file", "width": 4000, "height": 3000, "sampling": "420", "quality": 85,
         "interval": 250, "mode": "fancy"},
        # a web image: no restart markers at all
        {"name": "file_plain", "kind": "file", "width": 1620, "height": 1080, "sampling": "420", "quality": 85,
         "interval": 0, "mode": "fancy"},
    ]


def _log(rng, low, high):
    return math.exp(rng.uniform(math.log(low), math.log(high)))


def _sides(rng, low_mp, high_mp):
    mp, aspect = _log(rng, low_mp, high_mp) * 1e6, _log(rng, 0.6, 1.7)
    w = max(8, round(math.sqrt(mp * aspect)))
    return w, max(8, round(mp / w))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "batch", "calls", "variant", "variant", "variant", "corpus", "file",
                       "file"])
    quality, mode = rng.randint(50, 95), rng.choice(["fancy", "fancy", "simple"])
    if kind == "decode":
        w, h = _sides(rng, 0.01, 24.0)
        return {"kind": kind, "width": w, "height": h, "sampling": rng.choice(["420", "420", "422", "444"]),
                "quality": quality, "mode": mode}
    if kind == "batch":
        low = rng.randint(64, 1024)
        return {"kind": kind, "count": rng.randint(8, 48), "low": low, "high": rng.randint(low + 64, 4096), "mode": mode}
    if kind == "calls":
        low = rng.randint(32, 256)
        return {"kind": kind, "count": rng.randint(4, 64), "low": low, "high": rng.randint(low + 32, 640), "mode": mode}
    if kind == "variant":
        w, h = _sides(rng, 0.05, 24.0)
        scale = rng.choice([1, 1, 2, 4, 8])
        return {"kind": kind, "width": w, "height": h, "sampling": rng.choice(["420", "422", "444", "440", "411", "gray"]),
                "quality": quality, "mode": mode, "idct": "islow" if scale > 1 else rng.choice(["islow", "ifast", "float"]),
                "scale": scale}
    if kind == "corpus":
        low = _log(rng, 0.3, 4.0)
        return {"kind": kind, "count": rng.randint(4, 12), "low_mp": round(low, 3), "high_mp": round(_log(rng, low, 12.0), 3),
                "quality": min(quality, 85), "interval": rng.choice([8, 16, 32, 64]), "mode": mode}
    if rng.random() < 0.5:  # no markers
        w, h = _sides(rng, 0.05, 1.5)
        return {"kind": kind, "width": w, "height": h, "sampling": rng.choice(["420", "422", "444"]),
                "quality": min(quality, 85), "interval": 0, "mode": mode}
    w, h = _sides(rng, 0.2, 12.0)
    s = rng.choice(["420", "422"])
    return {"kind": kind, "width": w, "height": h, "sampling": s, "quality": quality, "interval": -(-w // 16),
            "mode": mode}


def _images(case):
    """(width, height, sampling, quality) of a case's images; the same for every seed."""
    if "count" not in case:
        return [(case["width"], case["height"], case["sampling"], case["quality"])]
    rng, out = random.Random(repr(sorted((k, v) for k, v in case.items() if k != "name"))), []
    for i in range(case["count"]):
        if case["kind"] == "corpus":
            mp, aspect = rng.uniform(case["low_mp"], case["high_mp"]) * 1e6, rng.choice([4 / 3, 3 / 2, 16 / 9, 3 / 4])
            w = round(math.sqrt(mp * aspect))
            out.append((w, max(8, round(mp / w)), "420", case["quality"]))
        else:
            w, h = rng.randint(case["low"], case["high"]), rng.randint(case["low"], case["high"])
            out.append((w, h, ("444", "422", "420")[i % 3], rng.randint(50, 95)))
    return out


# ---- inputs: pixels -> quantised blocks in MCU order ----------------------------------------

_LUMA_STEPS = np.array([
    16, 11, 10, 16, 24, 40, 51, 61, 12, 12, 14, 19, 26, 58, 60, 55, 14, 13, 16, 24, 40, 57, 69, 56,
    14, 17, 22, 29, 51, 87, 80, 62, 18, 22, 37, 56, 68, 109, 103, 77, 24, 35, 55, 64, 81, 104, 113, 92,
    49, 64, 78, 87, 103, 121, 120, 101, 72, 92, 95, 98, 112, 100, 103, 99])
_CHROMA_STEPS = np.array([
    17, 18, 24, 47, 99, 99, 99, 99, 18, 21, 26, 66, 99, 99, 99, 99, 24, 26, 56, 99, 99, 99, 99, 99,
    47, 66, 99, 99, 99, 99, 99, 99] + [99] * 32)


def _steps(quality):
    """uint16[4][64], natural order: luma, chroma, and two unused tables."""
    s = 5000 // quality if quality < 50 else 200 - 2 * quality
    t = np.ones((4, 64), dtype=np.uint16)
    for i, base in enumerate((_LUMA_STEPS, _CHROMA_STEPS)):
        t[i] = np.clip((base * s + 50) // 100, 1, 255)
    return t


def _frame(width, height, sampling):
    if sampling == "gray":
        return {"width": width, "height": height, "h": (1, 1, 1), "v": (1, 1, 1), "qsel": (0, 0, 0)}
    h, v = LUMA[sampling]
    return {"width": width, "height": height, "h": (h, 1, 1), "v": (v, 1, 1), "qsel": (0, 1, 1)}


def _planes(width, height, seed):
    """Y, Cb and Cr of a synthetic photograph, float32 whole numbers 0..255, [3, H, W]."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    r = random.Random(seed)
    xs = torch.arange(width, device=DEV, dtype=torch.float32)
    ys = torch.arange(height, device=DEV, dtype=torch.float32)
    tex = torch.zeros(height, width, device=DEV)
    for _ in range(6):  # sin(ux + vy + phase) from a row's and a column's vector
        period, amp = math.exp(r.uniform(math.log(4.0), math.log(64.0))), r.uniform(3.0, 16.0)
        theta, phase = r.uniform(0.0, math.pi), r.uniform(0.0, 2 * math.pi)
        u, v = 2 * math.pi * math.cos(theta) / period, 2 * math.pi * math.sin(theta) / period
        row, col = ys[:, None] * v + phase, xs[None, :] * u
        tex += amp * (torch.cos(row) * torch.sin(col) + torch.sin(row) * torch.cos(col))
    rgb = []
    for _ in range(3):
        a, b, c = r.uniform(64, 192), r.uniform(-80, 80), r.uniform(-80, 80)
        p = a + (b / width) * xs[None, :] + (c / height) * ys[:, None] + r.uniform(0.7, 1.3) * tex
        p = p + 5.0 * torch.randn(height, width, generator=g, device=DEV)
        rgb.append(p.round_().clamp_(0, 255))
    r_, g_, b_ = rgb
    ycc = torch.stack([0.299 * r_ + 0.587 * g_ + 0.114 * b_, -0.168736 * r_ - 0.331264 * g_ + 0.5 * b_ + 128.0,
                       0.5 * r_ - 0.418688 * g_ - 0.081312 * b_ + 128.0])
    return ycc.round_().clamp_(0, 255)


def _dct():
    m = np.array([[0.5 * (math.sqrt(0.5) if k == 0 else 1.0) * math.cos((2 * n + 1) * k * math.pi / 16)
                   for n in range(8)] for k in range(8)], dtype=np.float32)
    return torch.from_numpy(m).to(DEV)


def _blocks(width, height, sampling, quality, seed):
    """int16 [n_blocks, 64] on the GPU, MCU order, natural order inside a block."""
    h, v = LUMA.get(sampling, (1, 1))
    mx, my = -(-width // (8 * h)), -(-height // (8 * v))
    steps, d = _steps(quality), _dct()
    planes, grids = _planes(width, height, seed), []
    for c in range(1 if sampling == "gray" else 3):
        p = torch.nn.functional.pad(planes[c][None, None], (0, mx * 8 * h - width, 0, my * 8 * v - height),
                                    mode="replicate")[0, 0]
        hc, vc = (h, v) if c == 0 else (1, 1)
        if c and h * v > 1:
            p = p.reshape(my * 8, v, mx * 8, h).mean(dim=(1, 3)).round_()
        x = (p - 128.0).reshape(my * vc, 8, mx * hc, 8).permute(0, 2, 1, 3).reshape(-1, 8)
        x = (x @ d.t()).reshape(-1, 8, 8).transpose(1, 2).reshape(-1, 8)
        x = (x @ d.t()).reshape(-1, 8, 8).transpose(1, 2).reshape(-1, 64)
        q = torch.from_numpy(steps[0 if c == 0 else 1].astype(np.float32)).to(DEV)
        x = (x / q).round_().to(torch.int16)
        x = x.reshape(my, vc, mx, hc, 64).permute(0, 2, 1, 3, 4).reshape(my, mx, vc * hc, 64)
        grids.append(x)
    return torch.cat(grids, dim=2).reshape(-1, 64).contiguous(), steps


def _image(spec, seed):
    w, h, sampling, quality = spec
    coef, steps = _blocks(w, h, sampling, quality, seed)
    return _frame(w, h, sampling), coef, torch.from_numpy(steps.view(np.int16)).to(DEV)


# ---- inputs: quantised blocks -> baseline JPEG files -----------------------------------------

# T.81 Annex K.3: code counts by length, and symbols
_DC_VALS = list(range(12))
_HUFF = [
    ([0, 1, 5, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0, 0, 0, 0], _DC_VALS),
    ([0, 3, 1, 1, 1, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0, 0], _DC_VALS),
    ([0, 2, 1, 3, 3, 2, 4, 3, 5, 5, 4, 4, 0, 0, 1, 125], list(bytes.fromhex(
        "0102030004110512213141061351610722711432" "8191a1082342b1c11552d1f02433627282090a16" "1718191a25262728292a3435363738393a434445"
        "464748494a535455565758595a63646566676869" "6a737475767778797a838485868788898a929394" "95969798999aa2a3a4a5a6a7a8a9aab2b3b4b5b6"
        "b7b8b9bac2c3c4c5c6c7c8c9cad2d3d4d5d6d7d8" "d9dae1e2e3e4e5e6e7e8e9eaf1f2f3f4f5f6f7f8" "f9fa"))),
    ([0, 2, 1, 2, 4, 4, 3, 4, 7, 5, 4, 4, 0, 1, 2, 119], list(bytes.fromhex(
        "0001020311040521310612415107617113223281" "08144291a1b1c109233352f0156272d10a162434" "e125f11718191a262728292a35363738393a4344"
        "45464748494a535455565758595a636465666768" "696a737475767778797a82838485868788898a92" "939495969798999aa2a3a4a5a6a7a8a9aab2b3b4"
        "b5b6b7b8b9bac2c3c4c5c6c7c8c9cad2d3d4d5d6" "d7d8d9dae2e3e4e5e6e7e8e9eaf2f3f4f5f6f7f8" "f9fa"))),
]


def _zigzag():
    cells = sorted(((r, c) for r in range(8) for c in range(8)),
                   key=lambda p: (p[0] + p[1], p[0] if (p[0] + p[1]) % 2 else p[1]))
    return np.array([8 * r + c for r, c in cells])


def _codes(bits, vals):
    """code and length of each symbol, two int64 tensors of 256."""
    code, k, out = 0, 0, np.zeros((2, 256), dtype=np.int64)
    for length, n in enumerate(bits, 1):
        for _ in range(n):
            out[:, vals[k]] = code, length
            code, k = code + 1, k + 1
        code <<= 1
    return torch.from_numpy(out).to(DEV)


def _segment(marker, payload):
    return struct.pack(">HH", 0xFF00 | marker, len(payload) + 2) + payload


def _headers(frame, steps, interval):
    zz, out = _zigzag(), b"\xff\xd8"
    for i in range(2):
        out += _segment(0xDB, bytes([i]) + bytes(int(x) for x in steps[i][zz]))
    sof = struct.pack(">BHHB", 8, frame["height"], frame["width"], 3)
    for c in range(3):
        sof += bytes([c + 1, frame["h"][c] << 4 | frame["v"][c], min(c, 1)])
    out += _segment(0xC0, sof)
    for i, (bits, vals) in enumerate(_HUFF):
        out += _segment(0xC4, bytes([(i >> 1) << 4 | (i & 1)]) + bytes(bits) + bytes(vals))
    if interval:
        out += _segment(0xDD, struct.pack(">H", interval))
    return out + _segment(0xDA, bytes([3, 1, 0x00, 2, 0x11, 3, 0x11, 0, 63, 0]))


def _size(v):
    """Bits of |v|, T.81's magnitude category."""
    a = v.abs().to(torch.float32)
    return torch.where(a > 0, torch.floor(torch.log2(a.clamp(min=1))).to(torch.int64) + 1, torch.zeros_like(v))


def _jpeg(frame, coef, steps, interval):
    """The file's bytes, uint8 on the host."""
    bpm = frame["h"][0] * frame["v"][0] + 2
    n_mcu = coef.shape[0] // bpm
    ri = interval or n_mcu
    dev = coef.device
    zz = coef.to(torch.int64)[:, torch.from_numpy(_zigzag()).to(dev)]
    block = torch.arange(coef.shape[0], device=dev)
    mcu, inner = block // bpm, block % bpm
    comp = (inner - (bpm - 3)).clamp(min=0)  # 0 for every luma block
    chroma = (comp > 0).to(torch.int64)
    # DC: the difference from the component's last block, from 0 after a marker
    last = torch.where(inner == 0, block - bpm + (bpm - 3), torch.where(comp > 0, block - bpm, block - 1))
    fresh = (mcu % ri == 0) & ((inner == 0) | (comp > 0))
    diff = zz[:, 0] - torch.where(fresh, torch.zeros_like(block), zz[last.clamp(min=0), 0])
    tables = torch.stack([_codes(b, v) for b, v in _HUFF])  # [table, code/length, symbol]
    dc, ac = tables[:2], tables[2:]
    size = _size(diff)
    value = torch.zeros(coef.shape[0], 65, dtype=torch.int64, device=dev)
    length = torch.zeros_like(value)
    low = lambda v, s: torch.where(v < 0, v + (1 << s) - 1, v)  # noqa: E731
    value[:, 0] = dc[chroma, 0, size] << size | low(diff, size)
    length[:, 0] = dc[chroma, 1, size] + size
    # AC: (zero run, size) codes, with a code of its own for every 16 zeros
    v = zz[:, 1:]
    pos = torch.arange(1, 64, device=dev).expand_as(v)
    seen = torch.cummax(torch.where(v != 0, pos, torch.zeros_like(pos)), dim=1).values
    before = torch.cat([torch.zeros_like(seen[:, :1]), seen[:, :-1]], dim=1)
    run, size = pos - before - 1, _size(v)
    t = chroma[:, None].expand_as(v)
    sym = (run & 15) << 4 | size
    val = ac[t, 0, sym] << size | low(v, size)
    n = ac[t, 1, sym] + size
    for i in range(3):
        more = run >> 4 > i
        val = torch.where(more, ac[t, 0, 0xF0] << n | val, val)
        n = torch.where(more, n + ac[t, 1, 0xF0], n)
    value[:, 1:64], length[:, 1:64] = val, torch.where(v != 0, n, torch.zeros_like(n))
    eob = seen[:, -1] < 63
    value[:, 64], length[:, 64] = ac[chroma, 0, 0], torch.where(eob, ac[chroma, 1, 0], torch.zeros_like(chroma))
    del v, pos, seen, before, run, size, t, sym, val, n, zz
    # bit positions: each interval starts on a byte, its last byte filled with ones
    part = mcu // ri
    bits = torch.zeros(int(part[-1]) + 1, dtype=torch.int64, device=dev).index_add_(0, part, length.sum(1))
    start = torch.cumsum((bits + 7) // 8 * 8, 0)
    total = int(start[-1])
    start = start - (bits + 7) // 8 * 8
    flat = length.reshape(-1)
    at = torch.cumsum(flat, 0) - flat
    at = at.reshape(length.shape) + (start - (torch.cumsum(bits, 0) - bits))[part][:, None]
    keep = flat > 0
    flat, at, value = flat[keep], at.reshape(-1)[keep], value.reshape(-1)[keep]
    stream = torch.ones(total, dtype=torch.uint8, device=dev)
    which = torch.repeat_interleave(torch.arange(flat.numel(), device=dev), flat)
    nth = torch.arange(which.numel(), device=dev) - (torch.cumsum(flat, 0) - flat)[which]
    stream[at[which] + nth] = (value[which] >> (flat[which] - 1 - nth) & 1).to(torch.uint8)
    weights = torch.tensor([128, 64, 32, 16, 8, 4, 2, 1], dtype=torch.uint8, device=dev)
    data = (stream.reshape(-1, 8) * weights).sum(1, dtype=torch.int64)
    del which, nth, stream, at, value, flat
    # a zero after each 0xFF, a marker between intervals
    ff = (data == 255).to(torch.int64)
    owner = torch.repeat_interleave(torch.arange(bits.numel(), device=dev), (bits + 7) // 8)
    to = torch.arange(data.numel(), device=dev) + torch.cumsum(ff, 0) - ff + 2 * owner
    size = int(to[-1] + ff[-1]) + 1
    scan = torch.zeros(size, dtype=torch.uint8, device=dev)
    scan[to] = data.to(torch.uint8)
    ends = torch.cumsum((bits + 7) // 8, 0)[:-1]
    if ends.numel():
        mark = to[ends] - 2
        scan[mark] = 0xFF
        scan[mark + 1] = (0xD0 + torch.arange(mark.numel(), device=dev) % 8).to(torch.uint8)
    head = np.frombuffer(_headers(frame, steps, interval), dtype=np.uint8)
    return np.concatenate([head, scan.cpu().numpy(), np.array([0xFF, 0xD9], dtype=np.uint8)])


def _file(spec, interval, seed):
    w, h, sampling, quality = spec
    coef, steps = _blocks(w, h, sampling, quality, seed)
    return _jpeg(_frame(w, h, sampling), coef, steps, interval)


# ---- what a program has in hand -------------------------------------------------------------

def _rgb(frame):
    return torch.empty((frame["height"], frame["width"], 3), dtype=torch.uint8, device=DEV)


def _on_device(data):
    """The file in device memory, readable up to a multiple of 16 bytes."""
    d = torch.empty((data.size + 15) // 16 * 16, dtype=torch.uint8, device=DEV)
    d[:data.size].copy_(torch.from_numpy(data))
    return d


def prepare(case, seed):
    ctx, kind = _context(), case["kind"]
    specs = _images(case)
    if kind in ("decode", "variant"):
        frame, coef, qt = _image(specs[0], seed)
        s = {"frame": frame, "coef": coef.reshape(-1), "qt": qt}
        if kind == "decode":
            s["out"] = _rgb(frame)
        else:
            w, h = -(-frame["width"] // case["scale"]), -(-frame["height"] // case["scale"])
            s["ncomp"] = 1 if case["sampling"] == "gray" else 3
            s["out"] = torch.empty((h, w, 3) if s["ncomp"] == 3 else (h, w), dtype=torch.uint8, device=DEV)
    elif kind in ("batch", "calls"):
        jobs = []
        for i, spec in enumerate(specs):
            frame, coef, qt = _image(spec, seed * 1000 + i)
            jobs.append((frame, coef, qt, _rgb(frame), 3 * frame["width"]))
        s = {"jobs": jobs}
        if kind == "batch":
            s["plan"] = M.Batch(ctx, jobs, M.UPSAMPLE[case["mode"]])
    elif kind == "corpus":
        parts, jobs = [], []
        for i, spec in enumerate(specs):
            data = _file(spec, case["interval"], seed * 1000 + i)
            scan, qt = M.mjd_parse(data)
            offsets = M.mjd_restart_index(data, scan)
            frame = M.scan_frame(scan)
            coef = torch.empty(M.mjd_geometry_of(frame)["n_blocks"] * 64, dtype=torch.int16, device=DEV)
            parts.append((scan, offsets, _on_device(data), data.size, coef))
            jobs.append((frame, coef, torch.from_numpy(qt.view(np.int16)).to(DEV), _rgb(frame), 3 * frame["width"]))
        s = {"jobs": jobs, "entropy": M.EntropyBatch(ctx, parts), "plan": M.Batch(ctx, jobs, M.UPSAMPLE[case["mode"]])}
    else:
        data = _file(specs[0], case["interval"], seed)
        host = torch.empty(data.size, dtype=torch.uint8, pin_memory=True)
        host.copy_(torch.from_numpy(data))
        s = {"file": host}
    s.update(ctx=ctx, case=case)
    return s


def run(s):
    ctx, case = s["ctx"], s["case"]
    kind = case["kind"]
    if kind == "decode":
        return M.decode(ctx, s["frame"], s["coef"], s["qt"], case["mode"], out=s["out"])
    if kind == "variant":
        return M.decode_variant(ctx, s["frame"], s["coef"], s["qt"], case["idct"], case["mode"], s["ncomp"],
                                out=s["out"], scale=case["scale"])
    if kind == "batch":
        s["plan"].launch(use_graph=True)
        return [j[3] for j in s["jobs"]]
    if kind == "calls":
        M.mjd_decode_batch_noalloc(ctx, s["jobs"], M.UPSAMPLE[case["mode"]])
        return [j[3] for j in s["jobs"]]
    if kind == "corpus":
        s["entropy"].launch()
        s["plan"].launch()
        return {"coef": [j[1] for j in s["jobs"]], "rgb": [j[3] for j in s["jobs"]]}
    host = s["file"]
    n = host.numel()
    data = host.numpy()
    stream = torch.empty((n + 15) // 16 * 16, dtype=torch.uint8, device=DEV)
    stream[:n].copy_(host, non_blocking=True)
    scan, qt = M.mjd_parse(data)
    offsets = M.mjd_restart_index(data, scan)
    frame = M.scan_frame(scan)
    coef = torch.empty(M.mjd_geometry_of(frame)["n_blocks"] * 64, dtype=torch.int16, device=DEV)
    entropy = M.EntropyBatch(ctx, [(scan, offsets, stream, n, coef)])
    entropy.launch()
    rgb = M.decode(ctx, frame, coef, torch.from_numpy(qt.view(np.int16)).to(DEV), case["mode"])
    return {"coef": coef, "rgb": rgb}


def work(case):
    """Coefficients read once and pixels written once; for the bitstream cases
    the file read (about 0.3 bytes a pixel) and the coefficients written
    besides.  Operations: two passes of 8-point sums over every sample."""
    total, samples = 0.0, 0.0
    for w, h, sampling, _ in _images(case):
        hy, vy = LUMA.get(sampling, (1, 1))
        blocks = -(-w // (8 * hy)) * -(-h // (8 * vy)) * (1 if sampling == "gray" else hy * vy + 2)
        scale = case.get("scale", 1)
        pixels = -(-w // scale) * -(-h // scale)
        total += 128.0 * blocks + (1 if sampling == "gray" else 3) * pixels + 128
        if case["kind"] in ("corpus", "file"):
            total += 0.3 * w * h + 128.0 * blocks
        samples += 64.0 * blocks / scale ** 2
    return {"bytes": total, "flops": 32.0 * samples}


def exact(case, seed):
    """Every output is whole numbers with one right value (pixels and
    coefficients of integer, or fixed-order single-precision, arithmetic):
    there is nothing that 64 bits would make more exact."""
    return None
