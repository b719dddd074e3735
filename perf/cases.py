"""Performance cases of the detection library: what its users have it do, from one image to whole batches.

Five kinds of work, each through the public entry points of paper_2509_02447_amd (include/qrm.h):

  detect   a batch of planar images resident in device memory -> logits, bits, messages, code words (qrm_detect)
  request  a few raw camera / web images -> pre-processing -> tile selection -> detection -> verdict against a key
  forward  the extractor alone on ready-made tiles of any height and width, with every option of its last layer
  decode   Reed-Solomon decoding alone of received words
  ingest   the front end alone: pre-processing of raw images, tile selection, tile crops
  stream   chunks of images in pinned host memory through the pipelined entry point (qrm_detect_host)

Images are smooth ones (a level, a ramp) under noise of several strengths, the way natural images range from flat
to busy; weights are random He-normal ones (there are no trained ones here), code words are real code words with
0 .. t+1 symbol errors.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2509_02447_amd as qrm

KEY_FPR = 1e-6
PRIM_POLY = {2: 0x7, 3: 0xB, 4: 0x13, 5: 0x25, 6: 0x43, 7: 0x89, 8: 0x11D}


# ---------------------------------------------------------------------------------------------- the cases
# (channels, blocks, bits, m, n, k): the three networks and codes of the benchmark configurations
_NET_SMALL = dict(channels=32, blocks=4, bits=60, m=4, n=15, k=11)
_NET_48 = dict(channels=64, blocks=8, bits=48, m=4, n=12, k=8)
_NET_96 = dict(channels=64, blocks=8, bits=96, m=8, n=12, k=8)


def listed():
    return [
        # one uploaded photograph, checked while somebody waits for the answer: launches and latency are all of it
        dict(name="request_1", kind="request", images=1, raw_h=480, raw_w=640, size=256, tile=64, stride=32, **_NET_48),
        # the smallest configuration: a handful of images, small tiles, the small network (60 bits, RS(15,11))
        dict(name="detect_16_tile32", kind="detect", images=16, side=256, tile=32, **_NET_SMALL),
        # one page of a gallery, large tiles
        dict(name="detect_7_tile128", kind="detect", images=7, side=512, tile=128, **_NET_96),
        # an ordinary service batch whose size no compute-unit count divides
        dict(name="detect_333_tile64", kind="detect", images=333, side=256, tile=64, **_NET_48),
        # the paper's own shape in bulk: 256 x 256 images, 64 x 64 tiles, 48 bits
        dict(name="detect_4096_tile64", kind="detect", images=4096, side=256, tile=64, **_NET_48),
        # large images, large tiles, 96 bits, RS over GF(256), in bulk
        dict(name="detect_2048_tile128", kind="detect", images=2048, side=512, tile=128, **_NET_96),
        # no tiling: the whole image goes through the extractor
        dict(name="detect_256_tile256", kind="detect", images=256, side=256, tile=256, **_NET_48),
        # an extractor whose last convolution has its own affine and ReLU, on ragged tiles, an odd number of blocks
        dict(name="forward_100_75x100_relu", kind="forward", images=100, tile_h=75, tile_w=100, channels=64, blocks=7,
             bits=30, final_relu=True),
        # a million received words of the 96-bit code
        dict(name="decode_1m_12_8", kind="decode", words=1 << 20, m=8, n=12, k=8),
        # a long code: one word per image payload, t = 8
        dict(name="decode_20k_255_239", kind="decode", words=20000, m=8, n=255, k=239),
        # the front end of a crawler: decode buffers of one camera format -> 256 x 256 planes, tiles picked by variance
        dict(name="ingest_600_480x640", kind="ingest", images=600, raw_h=480, raw_w=640, size=256, tile=64, stride=32),
        # a collection that lives in host memory, streamed through the card
        dict(name="stream_6x1024", kind="stream", chunks=6, chunk_images=1024, side=256, tile=64, depth=3, **_NET_48),
    ]


# no drawn case does more than the largest listed one of its kind
_MAX_FLOPS = 17.0e12          # extractor work of detect_2048_tile128
_MAX_IMAGE_BYTES = 1.7e9      # its images


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _fit(case, key, flops_cap=_MAX_FLOPS):
    """Lowers the count `key` until the case stays under the caps."""
    one = dict(case)
    one[key] = 1
    n = min(case[key], int(flops_cap / max(1.0, work(one)["flops"])))
    if "side" in case:
        n = min(n, int(_MAX_IMAGE_BYTES / (3 * case["side"] ** 2)))
    case[key] = max(1, n)
    return case


def draw(rng):
    kind = rng.choice(["detect"] * 5 + ["forward"] * 3 + ["decode"] * 2 + ["request", "ingest", "stream"])
    net = dict(rng.choice([_NET_SMALL, _NET_48, _NET_48, _NET_96]))
    if kind == "detect":
        tile = _log_int(rng, 24, 256)
        side = max(tile, rng.choice([256, 256, 320, 512]))
        return _fit(dict(kind="detect", images=_log_int(rng, 1, 4096), side=side, tile=tile, **net), "images")
    if kind == "forward":
        case = dict(kind="forward", images=_log_int(rng, 1, 2048), tile_h=_log_int(rng, 16, 256),
                    tile_w=_log_int(rng, 16, 256), channels=rng.choice([32, 64, 64]), blocks=rng.randint(2, 9),
                    bits=rng.randint(16, 128), final_relu=rng.random() < 0.4)
        return _fit(case, "images")
    if kind == "decode":
        m = rng.choice([4, 4, 5, 6, 8, 8])
        n = rng.randint(8, (1 << m) - 1)
        t = rng.randint(1, min(8, (n - 1) // 2))
        words = min(_log_int(rng, 64, 1 << 20), (16 << 20) // n, (1 << 22) // (t * n) * 4)
        return dict(kind="decode", words=max(64, words), m=m, n=n, k=n - 2 * t)
    stride = rng.choice([16, 32])
    tile = stride * rng.randint(1, 4)
    size = rng.choice([224, 256, 384])
    raw_h, raw_w = _log_int(rng, 300, 1100), _log_int(rng, 300, 1100)
    if kind == "request":
        return _fit(dict(kind="request", images=_log_int(rng, 1, 64), raw_h=raw_h, raw_w=raw_w, size=size, tile=max(32, tile),
                         stride=stride, **net), "images")
    if kind == "ingest":
        images = max(1, min(_log_int(rng, 1, 2000), int(6e8 / (3 * raw_h * raw_w))))
        return dict(kind="ingest", images=images, raw_h=raw_h, raw_w=raw_w, size=size, tile=tile, stride=stride)
    chunk = _log_int(rng, 32, 1024)
    chunks = rng.randint(1, 8)
    return _fit(dict(kind="stream", chunks=chunks, chunk_images=chunk, side=256, tile=rng.choice([32, 48, 64, 96, 128]),
                     depth=rng.randint(1, 3), **net), "chunk_images", 8e12 / chunks)


# ---------------------------------------------------------------------------------------------- inputs
def _images(shape, gen, interleaved=False):
    """u8 images [N,3,H,W] (or [N,H,W,3]): per image and colour a level and a ramp, per image noise of one of four
    strengths, clipped."""
    n, h, w = shape
    out = torch.empty((n, h, w, 3) if interleaved else (n, 3, h, w), dtype=torch.uint8, device="cuda")
    yy = torch.linspace(-0.5, 0.5, h, device="cuda").view(1, 1, h, 1)
    xx = torch.linspace(-0.5, 0.5, w, device="cuda").view(1, 1, 1, w)
    strengths = torch.tensor([2.0, 12.0, 48.0, 120.0], device="cuda")
    step = max(1, (96 << 20) // (3 * h * w))
    for lo in range(0, n, step):
        c = min(step, n - lo)
        level = torch.rand((c, 3, 1, 1), generator=gen, device="cuda") * 255.0
        ramp = torch.rand((c, 3, 2, 1, 1), generator=gen, device="cuda") * 320.0 - 160.0
        amp = strengths[torch.randint(0, 4, (c, 1, 1, 1), generator=gen, device="cuda")]
        v = torch.rand((c, 3, h, w), generator=gen, device="cuda").mul_(2.0).sub_(1.0).mul_(amp)
        v.add_(level).add_(ramp[:, :, 0] * yy).add_(ramp[:, :, 1] * xx).round_().clamp_(0.0, 255.0)
        out[lo:lo + c] = (v.permute(0, 2, 3, 1) if interleaved else v).to(torch.uint8)
    return out


def _origins(count, limit, gen):
    """Uniformly random tile origins i32 [count,2] in 0..limit."""
    return torch.randint(0, limit + 1, (count, 2), generator=gen, device="cuda", dtype=torch.int32)


def _weights(case, seed):
    """Random weights: He-normal convolutions, folded batch norm near one."""
    g = np.random.default_rng([seed, 17])
    c, nb, bits = case["channels"], case["blocks"], case["bits"]
    affine = bool(case.get("final_relu"))
    conv = [g.normal(0.0, math.sqrt(2.0 / 27), (c, 3, 3, 3))]
    conv += [g.normal(0.0, math.sqrt(2.0 / (9 * c)), (c, c, 3, 3)) for _ in range(nb - 1)]
    conv.append(g.normal(0.0, math.sqrt(2.0 / (9 * c)), (bits, c, 3, 3)))
    rows = nb * c + (bits if affine else 0)
    return dict(in_ch=3, n_blocks=nb, channels=c, n_bits=bits,
                conv_w=np.concatenate([p.reshape(-1) for p in conv]).astype(np.float32),
                scale=g.normal(1.0, 0.1, rows).astype(np.float32), bias=g.normal(0.0, 0.1, rows).astype(np.float32),
                lin_w=g.normal(0.0, math.sqrt(2.0 / bits), (bits, bits)).astype(np.float32),
                lin_b=g.normal(0.0, 0.1, bits).astype(np.float32),
                mean=np.array([0.485, 0.456, 0.406], np.float32), std=np.array([0.229, 0.224, 0.225], np.float32))


def _code(case):
    return dict(m=case["m"], prim_poly=PRIM_POLY[case["m"]], n=case["n"], k=case["k"], fcr=1)


def _received_words(case, gen):
    """u8 [words,n]: systematic code words (roots alpha^1 .. alpha^2t) with 0 .. t+1 random symbol errors each."""
    m, n, k, count = case["m"], case["n"], case["k"], case["words"]
    q, two_t = 1 << m, n - k
    exp, log = [0] * (2 * q), [0] * q
    x = 1
    for i in range(q - 1):
        exp[i] = exp[i + q - 1] = x
        log[x] = i
        x <<= 1
        if x & q:
            x ^= PRIM_POLY[m]
    mul = lambda a, b: exp[log[a] + log[b]] if a and b else 0
    gpoly = [1]                                           # highest power first
    for r in range(1, two_t + 1):
        gpoly = [(gpoly[i] if i < len(gpoly) else 0) ^ (mul(gpoly[i - 1], exp[r]) if i else 0) for i in range(len(gpoly) + 1)]
    products = torch.tensor([[mul(a, gc) for gc in gpoly[1:]] for a in range(q)], dtype=torch.uint8, device="cuda")
    word = torch.zeros((count, n), dtype=torch.uint8, device="cuda")
    word[:, :k] = torch.randint(0, q, (count, k), generator=gen, device="cuda", dtype=torch.uint8)
    parity = torch.zeros((count, two_t), dtype=torch.uint8, device="cuda")
    for i in range(k):
        lead = (word[:, i] ^ parity[:, 0]).long()
        parity = torch.cat([parity[:, 1:], torch.zeros_like(parity[:, :1])], dim=1) ^ products[lead]
    word[:, k:] = parity
    errors = torch.randint(0, two_t // 2 + 2, (count, 1), generator=gen, device="cuda")
    place = torch.rand((count, n), generator=gen, device="cuda").argsort(dim=1)
    value = torch.randint(1, q, (count, n), generator=gen, device="cuda", dtype=torch.uint8)
    return torch.where(place < errors, word ^ value, word)


def _detect_outputs(case, n, bits=True):
    out = dict(msg=torch.empty((n, case["k"]), dtype=torch.uint8, device="cuda"),
               codeword=torch.empty((n, case["n"]), dtype=torch.uint8, device="cuda"),
               nerr=torch.empty((n,), dtype=torch.int8, device="cuda"))
    if bits:
        out["logits"] = torch.empty((n, case["bits"]), dtype=torch.float32, device="cuda")
        out["bits"] = torch.empty((n, case["bits"]), dtype=torch.uint8, device="cuda")
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    st = dict(case=case, kind=kind)
    if kind == "detect":
        n = case["images"]
        st["ctx"] = qrm.Context(weights=_weights(case, seed), rs=_code(case))
        st["img"] = _images((n, case["side"], case["side"]), gen)
        st["off"] = _origins(n, case["side"] - case["tile"], gen)
        st["out"] = _detect_outputs(case, n)
    elif kind == "request":
        n, size, tile = case["images"], case["size"], case["tile"]
        ctx = st["ctx"] = qrm.Context(weights=_weights(case, seed), rs=_code(case))
        key = torch.randint(0, 1 << case["m"], (case["k"],), generator=gen, device="cuda").cpu().numpy()
        ctx.qrm_set_key(key, qrm.binding.qrm_key_threshold(case["k"] * case["m"], KEY_FPR))
        st["raw"] = _images((n, case["raw_h"], case["raw_w"]), gen, interleaved=True)
        st["img"] = torch.empty((n, 3, size, size), dtype=torch.uint8, device="cuda")
        st["off"] = torch.empty((n, 2), dtype=torch.int32, device="cuda")
        st["out"] = _detect_outputs(case, n)
        st["out"]["matches"] = torch.empty((n,), dtype=torch.int32, device="cuda")
        st["out"]["detected"] = torch.empty((n,), dtype=torch.uint8, device="cuda")
    elif kind == "forward":
        n = case["images"]
        st["ctx"] = qrm.Context(weights=_weights(case, seed), final_relu=int(case["final_relu"]))
        st["tiles"] = _images((n, case["tile_h"], case["tile_w"]), gen)
        st["logits"] = torch.empty((n, case["bits"]), dtype=torch.float32, device="cuda")
        st["bits"] = torch.empty((n, case["bits"]), dtype=torch.uint8, device="cuda")
    elif kind == "decode":
        st["ctx"] = qrm.Context(rs=_code(case))
        st["words"] = _received_words(case, gen)
        st["out"] = _detect_outputs(case, case["words"], bits=False)
    elif kind == "ingest":
        n, size, tile = case["images"], case["size"], case["tile"]
        st["ctx"] = qrm.Context(rs=_code(dict(m=4, n=12, k=8)))
        st["raw"] = _images((n, case["raw_h"], case["raw_w"]), gen, interleaved=True)
        st["img"] = torch.empty((n, 3, size, size), dtype=torch.uint8, device="cuda")
        st["off"] = torch.empty((n, 2), dtype=torch.int32, device="cuda")
        st["tiles"] = torch.empty((n, 3, tile, tile), dtype=torch.uint8, device="cuda")
    else:
        c, chunks, side = case["chunk_images"], case["chunks"], case["side"]
        st["ctx"] = qrm.Context(weights=_weights(case, seed), rs=_code(case))
        bufs = min(3, chunks)                             # a caller refills a few pinned buffers round-robin
        img = [_images((c, side, side), gen).cpu().pin_memory() for _ in range(bufs)]
        off = [_origins(c, side - case["tile"], gen).cpu().pin_memory() for _ in range(bufs)]
        st["img"], st["off"] = [img[i % bufs] for i in range(chunks)], [off[i % bufs] for i in range(chunks)]
        n = c * chunks
        st["out"] = dict(msg=torch.empty((n, case["k"]), dtype=torch.uint8).pin_memory(),
                         codeword=torch.empty((n, case["n"]), dtype=torch.uint8).pin_memory(),
                         nerr=torch.empty((n,), dtype=torch.int8).pin_memory())
    torch.cuda.synchronize()
    return st


# ---------------------------------------------------------------------------------------------- one pass
def run(st):
    case, ctx, kind = st["case"], st["ctx"], st["kind"]
    if kind == "detect":
        o = st["out"]
        ctx.qrm_detect(st["img"], case["images"], case["side"], case["side"], st["off"], case["tile"], o["logits"],
                       o["bits"], o["msg"], o["codeword"], o["nerr"])
        return o
    if kind == "request":
        n, size, tile, o = case["images"], case["size"], case["tile"], st["out"]
        ctx.qrm_preprocess(st["raw"], n, case["raw_h"], case["raw_w"], size, None, 0, st["img"])
        ctx.qrm_select_tiles_variance(st["img"], n, size, size, tile, case["stride"], st["off"])
        ctx.qrm_detect_verify(st["img"], n, size, size, st["off"], tile, o["logits"], o["bits"], o["msg"], o["codeword"],
                              o["nerr"], o["matches"], o["detected"])
        return dict(o, images=st["img"], origins=st["off"])
    if kind == "forward":
        ctx.qrm_extractor_forward(st["tiles"], case["images"], case["tile_h"], case["tile_w"], st["logits"], st["bits"])
        return dict(logits=st["logits"], bits=st["bits"])
    if kind == "decode":
        o = st["out"]
        ctx.qrm_rs_decode(st["words"], case["words"], o["msg"], o["codeword"], o["nerr"])
        return o
    if kind == "ingest":
        n, size, tile = case["images"], case["size"], case["tile"]
        ctx.qrm_preprocess(st["raw"], n, case["raw_h"], case["raw_w"], size, None, 0, st["img"])
        ctx.qrm_select_tiles_variance(st["img"], n, size, size, tile, case["stride"], st["off"])
        ctx.qrm_extract_tiles(st["img"], n, size, size, st["off"], tile, st["tiles"])
        return dict(images=st["img"], origins=st["off"], tiles=st["tiles"])
    o = st["out"]
    ctx.qrm_detect_host(st["img"], case["chunk_images"], case["side"], case["side"], st["off"], case["tile"], case["depth"],
                        o["msg"], o["codeword"], o["nerr"])
    return o


# ---------------------------------------------------------------------------------------------- what a pass needs
def _extractor_work(case, n, h, w):
    """(bytes, flops) of the extractor on n tiles: tiles and weights read once, logits and bits written once.  Without
    a final ReLU the last convolution and the average pool are linear and need channel sums only."""
    c, nb, bits = case["channels"], case["blocks"], case["bits"]
    last = 2 * 9 * c * bits * (h * w if case.get("final_relu") else 1)
    flops = n * (2 * 9 * 3 * c * h * w + (nb - 1) * 2 * 9 * c * c * h * w + last + 2 * bits * bits)
    nbytes = n * (3 * h * w + 5 * bits) + 2 * (27 * c + (nb - 1) * 9 * c * c + 9 * c * bits) + 4 * bits * bits
    return nbytes, flops


def work(case):
    kind = case["kind"]
    if kind == "decode":
        return dict(bytes=case["words"] * (2 * case["n"] + case["k"] + 1), flops=0)
    if kind == "forward":
        b, f = _extractor_work(case, case["images"], case["tile_h"], case["tile_w"])
        return dict(bytes=b, flops=f)
    if kind == "ingest" or kind == "request":
        n, short = case["images"], min(case["raw_h"], case["raw_w"])
        front = n * (3 * short * short + 3 * case["size"] ** 2 + 8)
        if kind == "ingest":
            return dict(bytes=front + n * 3 * case["tile"] ** 2, flops=0)
        b, f = _extractor_work(case, n, case["tile"], case["tile"])
        return dict(bytes=front + b + n * (case["k"] + case["n"] + 6), flops=f)
    n = case["images"] if kind == "detect" else case["chunks"] * case["chunk_images"]
    b, f = _extractor_work(case, n, case["tile"], case["tile"])
    return dict(bytes=b + n * (8 + case["k"] + case["n"] + 1), flops=f)


def tolerance(case):
    """Against the same extractor in 64 bits (unrounded weights), over these ranges: relative error of the logits up to
    5.0e-4 and largest difference 2.6e-3 without a final ReLU, 1.8e-3 and 8.3e-3 with one; bits differing in 0.03 % of
    the places and decoded symbols in 0.2 %, all of them next to a logit of zero.  Four times that is allowed."""
    if case["kind"] in ("decode", "ingest"):
        return "exact"
    if case.get("final_relu"):
        return dict(rel=7e-3, max=3.3e-2, differ=0.01)
    return dict(rel=2e-3, max=1e-2, differ=0.01)
