"""The work whose speed this library is judged by: operators launched through the public binding.

A program that uses the library describes an operator, takes a decision trace for it (from an earlier search), builds
the variant once and launches it again and again on its own device buffers.  A case is one such operator with its sizes,
types and options; `prepare` builds the variant and draws the inputs, `run` is one launch.  The traces follow one rule
per operator family (`_schedule`): the structure that 64- to 96-trial searches at several sizes of the family ended
with, scaled to the sizes of the case.
"""
import torch

from paper_2205_13603_amd import binding as B, devmem

_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int8, "i32": torch.int32}
_BYTES = {"f32": 4, "f16": 2, "bf16": 2, "i8": 1, "i32": 4}


def listed():
    """The listed cases, from the smallest call to the largest."""
    return [
        # one small fp32 product on the vector ALUs: what a call costs when the work is next to nothing
        {"name": "gemm_f32_128", "family": "gemm_f32", "dtype": "f32", "m": 128, "n": 128, "k": 128},
        # few rows against a wide weight matrix (a decoding step): bound by reading the weights once
        {"name": "gemm_f16_48x4096x2048", "family": "gemm_rows", "dtype": "f16", "m": 48, "n": 4096, "k": 2048},
        # the library's flagship: 64 independent fp16 products of 1024 x 1024 x 1024
        {"name": "gemm_f16_1024_x64", "family": "gemm", "dtype": "f16", "m": 1024, "n": 1024, "k": 1024, "instances": 64},
        # one large bf16 product (a training step's matrix)
        {"name": "gemm_bf16_4096", "family": "gemm", "dtype": "bf16", "m": 4096, "n": 4096, "k": 4096, "instances": 1},
        # exact integer product, int8 in and int32 out: bound by writing the results
        {"name": "gemm_i8_512_x512", "family": "gemm_i8", "dtype": "i8", "m": 512, "n": 512, "k": 512, "instances": 512},
        # attention scores Q.K^T of 12 heads at a sequence length that is no power of two
        {"name": "scores_f16_208_x512", "family": "bmm", "dtype": "f16", "trans_b": True, "batch": 12, "m": 208, "n": 208,
         "k": 64, "instances": 512},
        # 3x3 convolution + bias + ReLU in the middle of a residual network
        {"name": "conv_f16_56x56x64_x512", "family": "conv2d", "dtype": "f16", "batch": 1, "size": 56, "cin": 64, "cout": 64,
         "kernel": 3, "stride": 1, "dilation": 1, "instances": 512},
        # the first layer of such a network on a batch of RGB images
        {"name": "first_f16_224x224x3_n128", "family": "first", "dtype": "f16", "batch": 128, "size": 224, "cin": 3,
         "cout": 64, "kernel": 7, "stride": 2},
        # the first layer of a video network: 3-D convolution over frames of RGB pixels
        {"name": "conv3d_f16_16x224x224x3_x8", "family": "conv3d", "dtype": "f16", "depth": 16, "size": 224, "cin": 3,
         "cout": 64, "kernel": 7, "stride": 2, "instances": 8},
        # upsampling layer of a generator: transposed convolution that doubles the image
        {"name": "up_bf16_16x16x256_n64", "family": "conv_transposed", "dtype": "bf16", "batch": 64, "size": 16, "cin": 256,
         "cout": 128, "kernel": 4, "stride": 2},
        # depthwise layer of a mobile network on a batch, odd image size, stride 2
        {"name": "depthwise_f32_57x57x144_n128", "family": "depthwise", "dtype": "f32", "batch": 128, "size": 57, "channels": 144,
         "kernel": 3, "stride": 2},
        # softmax over 1000 classes: rows whose length is no power of two
        {"name": "softmax_f32_65536x1000", "family": "softmax", "dtype": "f32", "rows": 65536, "cols": 1000},
    ]


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    family = rng.choice(["gemm_f32", "gemm_rows", "gemm", "gemm", "gemm_i8", "bmm", "conv2d", "first", "conv3d",
                         "conv_transposed", "depthwise", "softmax"])
    return _DRAW[family](rng)


def _log(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], spread evenly over its logarithm."""
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random() / step) * step))


def _draw_gemm_f32(rng):
    return {"family": "gemm_f32", "dtype": "f32", "m": _log(rng, 32, 256, 2), "n": _log(rng, 32, 256, 16), "k": _log(rng, 32, 256, 32)}


def _draw_gemm_rows(rng):
    return {"family": "gemm_rows", "dtype": rng.choice(["f16", "bf16"]), "m": _log(rng, 16, 128, 16), "n": _log(rng, 1024, 8192, 64),
            "k": _log(rng, 512, 4096, 256)}


def _draw_gemm(rng):
    # sizes of whole workgroup tiles of 128, 192 or 256, from one product to a batch of independent ones
    m, n = (_log(rng, 384, 4608, rng.choice([128, 192, 256])) for _ in range(2))
    m, n = (max(128, x // 128 * 128) if x % 192 and x % 128 else x for x in (m, n))
    k = _log(rng, 256, 4096, 64)
    most = max(1, min(64, int(1.37e11 / (2.0 * m * n * k))))
    return {"family": "gemm", "dtype": rng.choice(["f16", "bf16"]), "m": m, "n": n, "k": k, "instances": _log(rng, 1, most, 1)}


def _draw_gemm_i8(rng):
    m, n = (_log(rng, 256, 1024, 128) for _ in range(2))
    k = _log(rng, 256, 1024, 64)
    most = max(1, int(1.37e11 / (2.0 * m * n * k)))
    return {"family": "gemm_i8", "dtype": "i8", "m": m, "n": n, "k": k, "instances": _log(rng, 8, max(8, min(512, most)), 1)}


def _draw_bmm(rng):
    seq = _log(rng, 64, 512, 16)
    while _wave_split(seq // 16)[0] < 4:
        seq += 16
    dim, nt = rng.choice([32, 64, 128]), rng.random() < 0.6
    batch = rng.choice([8, 12, 16])
    most = max(1, int(4.5e8 / (batch * (2 * seq * dim + seq * seq))))
    return {"family": "bmm", "dtype": rng.choice(["f16", "bf16"]), "trans_b": nt, "batch": batch, "m": seq, "n": seq if nt else dim,
            "k": dim if nt else seq, "instances": _log(rng, 1, min(512, most), 1)}


def _draw_conv2d(rng):
    size = rng.choice([14, 16, 20, 28, 32, 40, 48, 56])
    cin, cout = rng.choice([32, 64, 96, 128, 256]), rng.choice([32, 64, 128, 256])
    kernel, stride, dilation = rng.choice([(1, 1, 1), (3, 1, 1), (3, 1, 1), (3, 2, 1), (3, 1, 2), (5, 1, 1)])
    if rng.random() < 0.4:
        cin = cout = 64
    flop = 2.0 * (size // stride) ** 2 * cin * cout * kernel * kernel
    n = max(8, min(512, int(6e10 * rng.uniform(0.05, 1.0) / flop) // 8 * 8))
    # a batch of images that share the weights, or independent instances
    shared = rng.random() < 0.6 or (size // stride) ** 2 % 16 != 0
    return {"family": "conv2d", "dtype": rng.choice(["f16", "bf16"]), "batch": n if shared else 1, "size": size, "cin": cin, "cout": cout,
            "kernel": kernel, "stride": stride, "dilation": dilation, "instances": 1 if shared else n}


def _draw_first(rng):
    size = _log(rng, 64, 256, 32)
    kernel, stride = rng.choice([(3, 2), (5, 2), (7, 2)])
    most = 128 * 224 * 224 // (size * size)
    return {"family": "first", "dtype": rng.choice(["f16", "bf16"]), "batch": _log(rng, 1, most, 1), "size": size, "cin": rng.choice([3, 3, 4]),
            "cout": rng.choice([32, 64, 96]), "kernel": kernel, "stride": stride}


def _draw_conv3d(rng):
    size, depth = _log(rng, 48, 224, 16), rng.choice([4, 8, 12, 16])
    most = max(1, 8 * 16 * 224 * 224 // (depth * size * size))
    return {"family": "conv3d", "dtype": rng.choice(["f16", "bf16"]), "depth": depth, "size": size, "cin": rng.choice([1, 3, 3, 4]),
            "cout": rng.choice([32, 64]), "kernel": rng.choice([3, 5, 7]), "stride": 2, "instances": _log(rng, 1, min(32, most), 1)}


def _draw_conv_transposed(rng):
    size = rng.choice([4, 8, 12, 16, 24, 32])
    cin, cout = rng.choice([64, 128, 256, 512]), rng.choice([64, 128, 256])
    kernel, stride = rng.choice([(4, 2), (4, 2), (3, 1), (2, 2), (4, 4)])
    flop = 2.0 * size * size * cin * cout * kernel * kernel
    n = max(8, min(256, int(1.7e10 * rng.uniform(0.05, 1.0) / flop) // 8 * 8))
    return {"family": "conv_transposed", "dtype": rng.choice(["f16", "bf16"]), "batch": n, "size": size, "cin": cin, "cout": cout,
            "kernel": kernel, "stride": stride}


def _draw_depthwise(rng):
    size, channels = _log(rng, 14, 112, 1), _log(rng, 24, 384, 8)
    stride, kernel = rng.choice([1, 2]), rng.choice([3, 3, 5])
    most = max(1, int(2.4e8 / (4 * channels * size * size)))
    return {"family": "depthwise", "dtype": "f32", "batch": _log(rng, 1, min(256, most), 1), "size": size, "channels": channels,
            "kernel": kernel, "stride": stride}


def _draw_softmax(rng):
    cols = _log(rng, 128, 4096, 8)
    rows = _log(rng, 256, max(256, 65536 * 1000 // cols // 64 * 64), 64)
    return {"family": "softmax", "dtype": rng.choice(["f32", "f32", "f16", "bf16"]), "rows": rows, "cols": cols}


_DRAW = {"gemm_f32": _draw_gemm_f32, "gemm_rows": _draw_gemm_rows, "gemm": _draw_gemm, "gemm_i8": _draw_gemm_i8, "bmm": _draw_bmm,
         "conv2d": _draw_conv2d, "first": _draw_first, "conv3d": _draw_conv3d, "conv_transposed": _draw_conv_transposed,
         "depthwise": _draw_depthwise, "softmax": _draw_softmax}


# ------------------------------------------------------------------ operators

def _pad(case):
    """Zero padding: centred filters, and the transposed ones that scale the image by their stride."""
    if case["family"] == "conv_transposed":
        return (case["kernel"] - case["stride"]) // 2
    return case.get("dilation", 1) * (case["kernel"] - 1) // 2


def _operator(case):
    f, dt = case["family"], case["dtype"]
    if f in ("gemm_f32", "gemm_rows", "gemm", "gemm_i8"):
        return B.gemm_op(case["m"], case["n"], case["k"], dt)
    if f == "bmm":
        return B.bmm_op(case["batch"], case["m"], case["n"], case["k"], case["trans_b"], dt)
    if f in ("conv2d", "first"):
        return B.conv2d_op(case["batch"], case["size"], case["size"], case["cin"], case["cout"], case["kernel"], case["kernel"],
                           stride=case["stride"], pad=_pad(case), in_dtype=dt, dilation=case.get("dilation", 1))
    if f == "conv3d":
        return B.conv3d_op(1, case["depth"], case["size"], case["size"], case["cin"], case["cout"], case["kernel"],
                           stride=case["stride"], pad=_pad(case), in_dtype=dt)
    if f == "conv_transposed":
        return B.conv2d_transposed_op(case["batch"], case["size"], case["size"], case["cin"], case["cout"], case["kernel"],
                                      case["kernel"], stride=case["stride"], pad=_pad(case), in_dtype=dt)
    if f == "depthwise":
        return B.dwconv2d_op(case["batch"], case["size"], case["size"], case["channels"], case["kernel"], case["kernel"],
                             stride=case["stride"], pad=_pad(case))
    if f == "softmax":
        return B.softmax_op(1, case["rows"], case["cols"], dt)
    raise ValueError(f)


def _out_shape(case):
    """(shape of one instance's output, its type)."""
    f, dt = case["family"], case["dtype"]
    if f in ("gemm_f32", "gemm_rows", "gemm"):
        return (case["m"], case["n"]), dt
    if f == "gemm_i8":
        return (case["m"], case["n"]), "i32"
    if f == "bmm":
        return (case["batch"], case["m"], case["n"]), dt
    if f == "softmax":
        return (1, case["rows"], case["cols"]), dt
    if f == "conv_transposed":
        o = (case["size"] - 1) * case["stride"] - 2 * _pad(case) + case["kernel"]
        return (case["batch"], o, o, case["cout"]), dt
    span = case.get("dilation", 1) * (case["kernel"] - 1) + 1
    o = (case["size"] + 2 * _pad(case) - span) // case["stride"] + 1
    if f == "conv3d":
        return (1, (case["depth"] + 2 * _pad(case) - span) // case["stride"] + 1, o, o, case["cout"]), dt
    return (case["batch"], o, o, case.get("cout", case.get("channels"))), dt


def _in_shapes(case):
    """Shapes of one instance's inputs, the bias excepted."""
    f = case["family"]
    if f in ("gemm_f32", "gemm_rows", "gemm", "gemm_i8"):
        return [(case["m"], case["k"]), (case["k"], case["n"])]
    if f == "bmm":
        b = (case["n"], case["k"]) if case["trans_b"] else (case["k"], case["n"])
        return [(case["batch"], case["m"], case["k"]), (case["batch"],) + b]
    if f == "softmax":
        return [(1, case["rows"], case["cols"])]
    s, k = case["size"], case["kernel"]
    if f == "depthwise":
        return [(case["batch"], s, s, case["channels"]), (k, k, case["channels"])]
    if f == "conv3d":
        return [(1, case["depth"], s, s, case["cin"]), (k, k, k, case["cin"], case["cout"])]
    return [(case["batch"], s, s, case["cin"]), (k, k, case["cin"], case["cout"])]


# ------------------------------------------------------------------ schedules

_SLOTS = {"mfma": B.SLOT_TENSORIZE, "i": B.SLOT_TILE_I, "j": B.SLOT_TILE_J, "c": B.SLOT_TILE_C, "k": B.SLOT_TILE_K,
          "unroll": B.SLOT_UNROLL, "cache_read": B.SLOT_CACHE_READ, "vec": B.SLOT_VECTORIZE, "vec_b": B.SLOT_VECTORIZE_B,
          "align": B.SLOT_STORAGE_ALIGN, "reorder": B.SLOT_REORDER, "cache_write": B.SLOT_CACHE_WRITE,
          "compute_at": B.SLOT_COMPUTE_AT, "rfactor": B.SLOT_RFACTOR}
_PLAIN = {"unroll": 0, "cache_read": 1, "vec": 1, "vec_b": 1, "align": 0, "reorder": 0, "cache_write": 0, "compute_at": 0, "rfactor": 1}


def _trace(space, decisions):
    """The trace that makes these decisions and the plain ones elsewhere."""
    by_slot = {_SLOTS[k]: v for k, v in dict(_PLAIN, **decisions).items()}
    return B.make_trace(space, [by_slot[space.slots[i].slot_id] for i in range(space.n_slots)])


def _tile(extent, *inner):
    """[outer, inner...] if the inner factors divide the extent, else None."""
    p = inner[0] * inner[1] * inner[2]
    return [extent // p, *inner] if extent % p == 0 else None


def _largest(extent, candidates):
    return next((c for c in candidates if extent % c == 0), 1)


def _wave_split(units):
    """(wavefronts, tiles per wavefront) that cover as much of `units` tiles as one workgroup takes."""
    best = (1, 1)
    for w in range(1, 14):
        for t in (1, 2, 3, 4):
            if units % (w * t) == 0 and w * t <= 16 and (w * t, w) > (best[0] * best[1], best[0]):
                best = (w, t)
    return best


def _gemm_tiles(m, n, products):
    """Workgroup tile: as square and large as the sizes allow while the tiles still fill the 256 compute units evenly."""
    best = None
    for bm in (256, 192, 128):
        for bn in (256, 192, 128):
            if m % bm or n % bn:
                continue
            tiles = (m // bm) * (n // bn) * products
            score = bm * bn / (bm + bn) * tiles / (256.0 * -(-tiles // 256))
            if best is None or score > best[0]:
                best = (score, bm, bn)
    return best[1:]


def _schedules(case):
    """(module mask, candidate decisions in order of preference); the first that validates is the case's trace."""
    f = case["family"]
    if f == "gemm_f32":
        yield 0xFF, {"i": _tile(case["m"], 1, 2, 1), "j": _tile(case["n"], 1, 16, 1), "k": _tile(case["k"], 1, 4, 8), "unroll": 64,
                     "cache_read": 0, "vec": 4, "vec_b": 2, "reorder": 1}
    elif f == "gemm_rows":
        groups = case["m"] // 16 * (case["n"] // 64)
        k0 = case["k"] // 256
        # too few workgroups for the chip: the reduction is split across several
        split = max((s for s in (1, 2, 4, 8) if k0 % s == 0 and (s == 1 or groups * s <= 256)), default=1)
        yield 0x4FF, {"mfma": 161616, "i": _tile(case["m"] // 16, 1, 1, 1), "j": _tile(case["n"] // 16, 1, 4, 1),
                      "k": _tile(case["k"] // 16, 2, 8, 1), "unroll": 16, "cache_read": 3, "vec": 8, "vec_b": 8, "align": 2,
                      "cache_write": 1 if split == 1 else 0, "rfactor": split}
    elif f == "gemm":
        bm, bn = _gemm_tiles(case["m"], case["n"], case["instances"])
        wi, wj = (2, 4) if bn != 192 else (4, 2)
        for wi, wj in ((wi, wj), (2, 2)):
            yield 0xFF, {"mfma": 323216, "i": _tile(case["m"] // 32, 1, wi, max(1, bm // 32 // wi)),
                         "j": _tile(case["n"] // 32, 1, wj, max(1, bn // 32 // wj)), "k": _tile(case["k"] // 16, 1, 1, 2),
                         "cache_read": 10, "vec": 8, "vec_b": 8, "reorder": 3, "cache_write": 1}
    elif f == "gemm_i8":
        # wavefronts of (2 or 1) x (4 or 2) strided 32 x 32 tiles where a side is a multiple of 256, small tiles elsewhere
        bm, bn = (256 if case[x] % 256 == 0 else 128 for x in ("m", "n"))
        if bm + bn > 256:
            yield 0xFF, {"mfma": 323232, "i": _tile(case["m"] // 32, bm // 128, 4, 1), "j": _tile(case["n"] // 32, bn // 64, 2, 1),
                         "k": _tile(case["k"] // 32, 1, 1, 2), "unroll": 16, "cache_read": 10, "vec": 16, "vec_b": 16, "reorder": 3,
                         "cache_write": 1}
        yield 0xFF, {"mfma": 161632, "i": _tile(case["m"] // 16, 2, 2, 2), "j": _tile(case["n"] // 16, 2, 4, 1),
                     "k": _tile(case["k"] // 32, 1, 2, 1), "unroll": 64, "cache_read": 1, "vec": 16, "vec_b": 4, "align": 1, "reorder": 2}
    elif f == "bmm":
        w, t = _wave_split(case["m"] // 16)
        steps = case["k"] // 32
        if case["trans_b"]:
            cols = max(d for d in range(1, 14) if (case["n"] // 16) % d == 0)
            yield 0xFF, {"mfma": 161632, "i": _tile(case["m"] // 16, 1, w, t), "j": _tile(case["n"] // 16, cols, 1, 1),
                         "k": _tile(steps, 1, _largest(steps, (4, 2, 1)), 1), "unroll": 16, "vec": 8, "vec_b": 8, "cache_write": 1}
        steps = case["k"] // 16
        inner = _largest(steps, (13, 12, 11, 10, 9, 8, 7, 6, 5, 4, 3, 2))
        yield 0xFF, {"mfma": 161616, "i": _tile(case["m"] // 16, 1, w, t), "j": _tile(case["n"] // 16, 1, 1, min(4, case["n"] // 16)),
                     "k": _tile(steps, 1, inner, 1), "unroll": 16, "vec": 8, "vec_b": 8, "align": 2, "cache_write": 1}
    elif f == "conv2d":
        shape, _ = _out_shape(case)
        pixels, steps = shape[1] * shape[2], case["kernel"] ** 2 * case["cin"] // 16
        if case["cout"] <= 64 and case["cin"] <= 64 and case["kernel"] > 1:
            # weights and input rows resident in LDS under persistent workgroups
            for mi, mfma, inner in ((32, 323216, 2), (16, 161632, 1)):
                for w in (7, 8, 6, 5, 4):
                    yield 0xFF, {"mfma": mfma, "i": _tile(case["batch"] * pixels // mi, 1, w, 1) if pixels % (mi * w) == 0 else None,
                                 "j": [1, 1, 1, case["cout"] // mi], "k": [case["kernel"], 1, steps // case["kernel"] // 2, inner],
                                 "unroll": 64, "cache_read": 2, "vec": 8, "align": 1, "cache_write": 1, "compute_at": 3}
        rows = case["batch"] * pixels
        for tm, tn in ((4, 2), (2, 2), (7, 2), (4, 1), (2, 1), (1, 1)):
            yield 0xFF, {"mfma": 161632, "i": _tile(rows // 16, 1, 2, tm) if rows % 16 == 0 else None, "j": _tile(case["cout"] // 16, 1, 2, tn),
                         "k": [steps // 2, 1, 1, 1], "unroll": 64, "cache_read": 3, "vec": 8, "align": 1, "reorder": 2, "cache_write": 1}
        yield 0xFF, {"mfma": 161632, "i": _tile(rows // 16, 1, 1, 1), "j": _tile(case["cout"] // 16, 1, 2, 1),
                     "k": [steps // 2, 1, 1, 1], "unroll": 64, "cache_read": 3, "vec": 8, "align": 1, "reorder": 2, "cache_write": 1}
    elif f == "first":
        shape, _ = _out_shape(case)
        run = -(-case["kernel"] * case["cin"] // 32)  # matrix-core k steps per filter row
        for rows in (16, 14, 8, 7, 4, 2, 1):
            units = rows * shape[2] // 16
            if shape[1] % rows or rows * shape[2] % 16:
                continue
            w = _largest(units, (8, 7, 6, 5, 4, 3, 2))
            yield 0x2FF, {"mfma": 161632, "i": _tile(case["batch"] * shape[1] * shape[2] // 16, _largest(units // w, (2,)), w,
                                                     units // w // _largest(units // w, (2,))),
                          "j": [1, case["cout"] // 16, 1, 1] if case["cout"] % 32 else [2, case["cout"] // 32, 1, 1],
                          "k": [1, 1, case["kernel"] * run, 1], "unroll": 64, "reorder": 2, "cache_write": 1, "compute_at": 1}
    elif f == "conv3d":
        shape, _ = _out_shape(case)
        rows, steps = shape[1] * shape[2] * shape[3] // 32, -(-case["kernel"] ** 3 * case["cin"] // 16)
        for w in (4, 2, 1):
            yield 0xFF, {"mfma": 323216, "i": _tile(rows, 1, w, 1), "j": [1, 1, case["cout"] // 32, 1], "k": [steps, 1, 1, 1],
                         "vec": 1, "reorder": 2, "cache_write": 1}
    elif f == "conv_transposed":
        shape, _ = _out_shape(case)
        rows, steps = shape[0] * shape[1] * shape[2] // 32, case["kernel"] ** 2 * case["cin"] // 16
        wj = case["cout"] // 32
        for tm, wi, tn in ((2, 4, 1), (2, 4, 2), (1, 4, 1), (1, 4, 2), (1, 2, 2), (1, 1, 2)):
            yield 0xFF, {"mfma": 323216, "i": _tile(rows, tm, wi, 1), "j": _tile(wj, 1, max(1, min(4, wj) // tn), tn),
                         "k": _tile(steps, 2, 1, 2), "unroll": 64, "cache_read": 2, "vec": 8, "align": 1, "reorder": 2, "cache_write": 1}
    elif f == "depthwise":
        shape, _ = _out_shape(case)
        o, ch = shape[1], case["channels"]
        lanes = max(d for d in range(1, 257) if ch % d == 0)
        row, col = _largest(o, (2, 3)), max(d for d in range(1, 8) if o % d == 0)
        if row > 1 and col > 1:
            # 2 or 3 rows of up to 7 outputs per thread, channels across the lanes
            across = max(d for d in range(1, 33) if o // col % d == 0 and d * lanes <= 512)
            yield 0xFF, {"i": _tile(o, 1, 1, row), "j": _tile(o, 1, across, col), "c": _tile(ch, 1, lanes, 1), "unroll": 64,
                         "cache_read": 0, "reorder": 2}
        lanes = _largest(ch, (16, 8))
        if o <= 32:
            yield 0xFF, {"i": _tile(o, 1, o, 1), "j": _tile(o, 1, 1, o), "c": _tile(ch, 1, lanes, 1), "unroll": 64, "cache_read": 0,
                         "reorder": 2}
        yield 0xFF, {"i": _tile(o, 1, 1, 1), "j": _tile(o, 1, max(d for d in range(1, 65) if o % d == 0), 1), "c": _tile(ch, 1, lanes // 4, 4),
                     "unroll": 64, "cache_read": 0, "reorder": 2}
    elif f == "softmax":
        cols = case["cols"]
        lanes = next(l for l in (64, 32, 16, 8) if cols % l == 0)
        vec = next(v for v in (2, 1) if cols % (lanes * v) == 0)
        rest = cols // lanes // vec
        group = 512 // lanes
        per = next(p for p in (4, 2, 1) if case["rows"] % (group * p) == 0) if lanes < 64 else 1
        group = group if case["rows"] % (group * per) == 0 else 64 // min(lanes, 64)
        if lanes == 64:
            group = 2
        yield 0xFF, {"i": _tile(case["rows"], per, group, 1), "k": [rest, 1, lanes, vec] if lanes == 64 else None, "cache_read": 1}
        for serial in range(1, rest + 1):
            if rest % serial == 0 and rest // serial <= 32:
                yield 0xFF, {"i": _tile(case["rows"], per, group, 1), "k": [serial, rest // serial, lanes, vec], "cache_read": 0}


def _schedule(op, case):
    spaces = {}
    for flags, decisions in _schedules(case):
        if any(v is None for v in decisions.values()):
            continue
        if flags not in spaces:
            spaces[flags] = op.space(flags)
        try:
            trace = _trace(spaces[flags], decisions)
            B.trace_validate(op, spaces[flags], trace)
        except (B.MsError, ValueError):
            continue
        return spaces[flags], trace
    raise ValueError("no schedule for %r" % (case,))


# ------------------------------------------------------------------ what is timed

def _inputs(case, g):
    """Seeded inputs with the distributions of paper_2205_13603_amd/inputs.py, drawn on the GPU."""
    f, dt, r = case["family"], case["dtype"], case.get("instances", 1)
    shapes = [((r,) if r > 1 else ()) + s for s in _in_shapes(case)]

    def normal(shape, sigma):
        return (torch.randn(shape, generator=g, device="cuda") * sigma).to(_TORCH[dt])

    def uniform(shape, lo, hi):
        return (torch.rand(shape, generator=g, device="cuda") * (hi - lo) + lo).to(_TORCH[dt])

    if f == "gemm_i8":
        return [torch.randint(-128, 128, s, generator=g, device="cuda", dtype=torch.int8) for s in shapes]
    if f in ("gemm_f32", "depthwise"):
        return [uniform(s, -1.0, 1.0) for s in shapes]
    if f in ("gemm", "gemm_rows"):
        return [normal(s, 0.1) for s in shapes]
    if f == "bmm":
        return [normal(s, 1.0) for s in shapes]
    if f == "softmax":
        return [normal(s, 2.0) for s in shapes]
    bias = torch.randn(((r,) if r > 1 else ()) + (case["cout"],), generator=g, device="cuda") * 0.05
    return [uniform(shapes[0], 0.0, 1.0) if f != "conv_transposed" else normal(shapes[0], 1.0), normal(shapes[1], 0.05), bias]


class _State:
    """What a program holds: the built variant, its inputs, an output buffer and the workspace if the variant needs one."""

    def __init__(self, case, seed):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        self.instances = case.get("instances", 1)
        op = _operator(case)
        space, trace = _schedule(op, case)
        self.variant = B.Variant(op, space, trace)
        self.variant.prepare()
        self.inputs = _inputs(case, g)
        shape, dt = _out_shape(case)
        self.output = torch.empty(((self.instances,) if self.instances > 1 else ()) + shape, dtype=_TORCH[dt], device="cuda")
        need = self.variant.workspace_bytes() * self.instances
        self.workspace = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    """One launch on the current stream; the output is the state's own buffer."""
    state.variant.launch([t.data_ptr() for t in state.inputs], state.output.data_ptr(), instances=state.instances,
                         stream=devmem.current_stream(), workspace=state.workspace.data_ptr() if state.workspace is not None else None)
    return state.output


def work(case):
    """Operations of the operator's definition and every input and output moved once."""
    f, r = case["family"], case.get("instances", 1)
    shape, odt = _out_shape(case)
    out, ins = 1, 0
    for x in shape:
        out *= x
    for s in _in_shapes(case):
        p = 1
        for x in s:
            p *= x
        ins += p
    size = ins * _BYTES[case["dtype"]] + out * _BYTES[odt] + (4 * case["cout"] if "cout" in case else 0)
    if f in ("gemm_f32", "gemm_rows", "gemm", "gemm_i8", "bmm"):
        flop = 2.0 * out * case["k"]
    elif f == "softmax":
        flop = 5.0 * out  # maximum, difference, exponential, sum, scaling
    elif f == "depthwise":
        flop = 2.0 * out * case["kernel"] ** 2
    elif f == "conv_transposed":
        flop = 2.0 * case["batch"] * case["size"] ** 2 * case["cin"] * case["cout"] * case["kernel"] ** 2
    else:
        flop = 2.0 * out * case["cin"] * case["kernel"] ** (3 if f == "conv3d" else 2)
    return {"bytes": float(size) * r, "flops": flop * r}


def tolerance(case):
    """int32 results are exact; floats differ by the order of the fp32 sums and the one rounding to the output type.
    Against float64 references the kernels show rel 0.9e-7 .. 2.9e-7 (max 1.6e-6) with fp32, 2.1e-4 (max 4.9e-4) with fp16
    and 1.7e-3 (max 3.9e-3) with bf16 results; the bounds are four times that."""
    return {"i8": "exact", "f32": {"rel": 1.2e-6, "max": 6.5e-6}, "f16": {"rel": 8.5e-4, "max": 2e-3},
            "bf16": {"rel": 7e-3, "max": 1.6e-2}}[case["dtype"]]


def exact(case, seed):
    """What `run` returns for these inputs, from the operator's definition in float64."""
    f, r = case["family"], case.get("instances", 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x, *rest = [t.double().reshape((r, t.numel() // r)) for t in _inputs(case, g)]
    shapes = _in_shapes(case)
    shape, _ = _out_shape(case)
    x = x.reshape((r,) + shapes[0])
    if f == "softmax":
        y = torch.softmax(x, -1)
    else:
        w = rest[0].reshape((r,) + shapes[1])
        if f in ("gemm_f32", "gemm_rows", "gemm", "gemm_i8"):
            y = torch.stack([p @ q for p, q in zip(x, w)])
        elif f == "bmm":
            w = w.transpose(-1, -2).contiguous() if case["trans_b"] else w
            y = torch.stack([a @ b for p, q in zip(x, w) for a, b in zip(p, q)]).reshape((r,) + shape)
        else:
            bias = rest[1] if len(rest) > 1 else None
            y = torch.stack([_exact_conv(case, x[i], w[i], shape) for i in range(r)])
            if bias is not None:
                y = torch.relu(y + bias.reshape((r,) + (1,) * (len(shape) - 1) + (shape[-1],)))
    y = y.to(torch.int32) if f == "gemm_i8" else y
    return y if r > 1 else y[0]


def _exact_conv(case, x, w, shape):
    """Sum over the filter's taps; x [N, (D,) H, W, C], w [(KD,) KH, KW, C(, Cout)], result of `shape`."""
    f, s, p = case["family"], case["stride"], _pad(case)
    if f == "conv_transposed":
        # every tap writes a grid of pixels `stride` apart into an image that has the padding still around it
        k, n = case["kernel"], case["size"]
        y = torch.zeros((shape[0], shape[1] + 2 * p, shape[2] + 2 * p, shape[3]), dtype=torch.float64, device=x.device)
        for kh in range(k):
            for kw in range(k):
                y[:, kh:kh + (n - 1) * s + 1:s, kw:kw + (n - 1) * s + 1:s] += x @ w[kh, kw]
        return y[:, p:p + shape[1], p:p + shape[2]]
    dims = len(shape) - 2
    x = torch.nn.functional.pad(x, (0, 0) + (p, p) * dims)
    y = torch.zeros(shape, dtype=torch.float64, device=x.device)
    for tap in torch.cartesian_prod(*[torch.arange(case["kernel"])] * dims).tolist():
        at = [t * case.get("dilation", 1) for t in tap]
        part = x[(slice(None),) + tuple(slice(a, a + (o - 1) * s + 1, s) for a, o in zip(at, shape[1:-1]))]
        y += part * w[tuple(tap)] if f == "depthwise" else part @ w[tuple(tap)]
    return y
