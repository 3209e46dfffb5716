"""The work whose speed is followed: calls of the library's public entry points.

A case is a dict of plain values.  Its "kind" names the entry point:
  call     one drelu / relu call on a share pair (k_in > 0: trunc_drelu /
           trunc_relu, a layer's product truncated on the way in)
  step     the key-bit step: trunc_det of a product, then the DReLU
  stream   one trunc_det or mul_trunc call
  batch    one ragged batch (every activation of a network pass) in one launch
  records  precomputed randomness: the offline expansion and the online ReLU
  rss      one DReLU / ReLU call on replicated (2-of-3) shares
  apart    the DReLU with the parties apart: both sends, P2's reply, both finishes
"setting" is one of SETTINGS, "n" the number of elements.
"""

import torch

from paper_2309_04909_amd import batch as BT
from paper_2309_04909_amd import bicop as B

# name: (l, l_x, k_lo, standard deviation of the values in units of 2^-f, f, bound of |x|)
SETTINGS = {
    "key18": (64, 18, 13, 8.0, 13, 1 << 30),      # |x| < 2^30: 17 integer bits and the guard bit
    "key7": (64, 7, 11, 1.0, 13, 1 << 17),        # the paper's 5 + 2 key bits
    "chain11": (51, 11, 13, 64.0, 13, 1 << 23),   # a matrix product's outputs after truncation by 13
    "ring24": (24, 7, 10, 64.0, 8, 1 << 16),      # the same in the 32-bit ring, after truncation by 8
    "ring32": (32, 8, 8, 8.0, 8, 1 << 15),        # a serving job in the 32-bit ring
    "full31": (64, 31, 0, 37.0, 13, 1 << 30),     # no key bits: every bit of the window
    "full32": (64, 32, 0, 37.0, 13, 1 << 31),
}

# The ReLU activations of a ResNet-18-shaped pass on 224 x 224 inputs.
RESNET18 = [64 * 112 * 112] + [64 * 56 * 56] * 4 + [128 * 28 * 28] * 4 + [256 * 14 * 14] * 4 + [512 * 7 * 7] * 4


def sizes_text(sizes):
    return ",".join(str(s) for s in sizes)


def listed():
    return [
        # A layer of a small network, or the tail of a batch: latency and the host's share of a call.
        {"name": "drelu_1000", "kind": "call", "op": "drelu", "setting": "key7", "n": 1000, "k_in": 0},
        # The plain DReLU without key bits on 65,536 values, the widest window there is.
        {"name": "plain_drelu_65536", "kind": "call", "op": "drelu", "setting": "full32", "n": 65536, "k_in": 0},
        # A mid-sized serving job in the 32-bit ring, a ragged size.
        {"name": "serving_relu_50021", "kind": "call", "op": "relu", "setting": "ring32", "n": 50021, "k_in": 0},
        # The key-bit step on 2^24 elements: 13-bit truncation of the products and the DReLU of the values.
        {"name": "keybit_step_2p24", "kind": "step", "op": "drelu", "setting": "key18", "n": 1 << 24, "k_in": 13},
        # The secure product of two tensors with truncation of the factors first.
        {"name": "mul_trunc_2p24", "kind": "stream", "op": "mul", "setting": "key18", "n": 1 << 24, "k_in": 26},
        # ReLU after a [4096 x 4096] . [4096 x 1024] fixed-point product, in both rings.
        {"name": "matmul_relu_l64", "kind": "call", "op": "relu", "setting": "chain11", "n": 4096 * 1024, "k_in": 13},
        {"name": "matmul_relu_l32", "kind": "call", "op": "relu", "setting": "ring24", "n": 4096 * 1024, "k_in": 8},
        # Every ReLU of a network pass in one launch: a single image and a batch of 32.
        {"name": "resnet_relu_batch1", "kind": "batch", "op": "relu", "setting": "key7", "sizes": sizes_text(RESNET18),
         "k_in": 0},
        {"name": "resnet_relu_batch32", "kind": "batch", "op": "relu", "setting": "key7",
         "sizes": sizes_text(32 * s for s in RESNET18), "k_in": 0},
        # One layer's ReLU from randomness expanded beforehand, offline and online part.
        {"name": "records_relu_3m", "kind": "records", "op": "relu", "setting": "key7", "n": 32 * 128 * 28 * 28, "k_in": 0},
        # The ReLU on replicated shares, a ragged size.
        {"name": "rss_relu_4m", "kind": "rss", "op": "relu", "setting": "key18", "n": 4000003, "k_in": 0},
        # The DReLU as three machines would run it, each party's own call.
        {"name": "parties_apart_1m", "kind": "apart", "op": "drelu", "setting": "key18", "n": 1000003, "k_in": 0},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(2.0 ** rng.uniform(lo, hi))) + rng.randrange(3)

    kind = rng.choice(["call", "call", "call", "step", "stream", "batch", "records", "rss", "apart"])
    if kind == "call":
        setting = rng.choice(sorted(SETTINGS))
        wide = setting.startswith("full")
        case = {"kind": kind, "op": rng.choice(["drelu", "relu"]), "setting": setting, "n": size(0, 20 if wide else 23.5),
                "k_in": {"chain11": 13, "ring24": 8}.get(setting, 0)}
    elif kind == "step":
        case = {"kind": kind, "op": "drelu", "setting": "key18", "n": size(10, 23.5), "k_in": 13}
    elif kind == "stream":
        case = {"kind": kind, "op": rng.choice(["trunc", "mul"]), "setting": "key18", "n": size(10, 24),
                "k_in": rng.choice([13, 26])}
    elif kind == "batch":
        case = {"kind": kind, "op": "mixed", "setting": rng.choice(["key7", "key18", "chain11", "ring32"]),
                "sizes": sizes_text(size(10, 20) for _ in range(rng.randrange(2, 33))), "k_in": 0}
        if case["setting"] == "chain11":
            case["k_in"] = 13
    elif kind == "records":
        case = {"kind": kind, "op": rng.choice(["drelu", "relu"]), "setting": rng.choice(["key7", "key18", "ring32"]),
                "n": size(8, 22), "k_in": 0}
    elif kind == "rss":
        case = {"kind": kind, "op": rng.choice(["drelu", "relu"]), "setting": rng.choice(["key7", "key18", "ring32"]),
                "n": size(4, 23), "k_in": 0}
    else:
        case = {"kind": kind, "op": "drelu", "setting": rng.choice(["key7", "key18"]), "n": size(4, 21), "k_in": 0}
    return case


# ------------------------------------------------------------------- inputs


def values(gen, n, setting, k_in, bound=None):
    """n fixed-point values of the setting (a layer's product before its truncation when k_in > 0), int64."""
    _, _, _, std, f, lim = SETTINGS[setting]
    if setting.startswith("full"):
        v = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * 128.0 - 64.0
    else:
        v = torch.randn(n, generator=gen, device="cuda", dtype=torch.float64) * std
    x = torch.round(v * float(1 << (f + k_in)))
    top = (bound if bound is not None else lim << k_in) - 1
    return x.clamp_(-top, top).to(torch.int64)


def uniform64(gen, n):
    return torch.randint(-(1 << 63), (1 << 63) - 1, (n,), generator=gen, device="cuda", dtype=torch.int64)


def stored(x, ell):
    """int64 ring elements (wrapping) as shares of Z_2^ell in their storage width."""
    if ell < 64:
        x = x & ((1 << ell) - 1)
    if ell <= 32:
        x = torch.where(x >= 1 << 31, x - (1 << 32), x).to(torch.int32)
    return x.contiguous()


def shares(gen, x, ell, parties=2):
    parts = [uniform64(gen, x.numel()) for _ in range(parties - 1)]
    first = x
    for r in parts:
        first = first - r
    return [stored(s, ell) for s in [first] + parts]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ell, lx, k_lo = SETTINGS[case["setting"]][:3]
    kind, k_in = case["kind"], case["k_in"]
    prm = B.Params(ell, lx, k_lo)
    sd = B.Seeds(seed * 3 + 101, seed * 5 + 202, seed * 7 + 303, seed + 404)
    state = {"case": case, "prm": prm, "sd": sd}
    if kind == "batch":
        segs = []
        for i, n in enumerate(int(s) for s in case["sizes"].split(",")):
            x0, x1 = shares(gen, values(gen, n, case["setting"], k_in), ell + k_in)
            op = B.BC_OP_DRELU if case["op"] == "mixed" and i % 2 else B.BC_OP_RELU
            segs.append(BT.Segment(x0, x1, torch.empty_like(x0), torch.empty_like(x1), op=op, nonce=seed + i, k_in=k_in))
        state["batch"] = BT.RaggedBatch(prm, B.Seeds(sd.seed01, sd.seed02, sd.seed12), segs)
        state["out"] = [t for s in segs for t in (s.y0, s.y1)]
        return state
    n = case["n"]
    if kind == "rss":
        state["x"] = tuple(shares(gen, values(gen, n, case["setting"], 0), ell, 3))
        state["sd"] = B.RssSeeds(sd.seed01, sd.seed02, sd.seed12, seed + 505, seed + 606, sd.nonce)
    elif kind == "step":
        state["x"] = shares(gen, values(gen, n, case["setting"], 0), ell)
        z = values(gen, n, case["setting"], 0) * values(gen, n, case["setting"], 0)     # wraps in Z_2^64
        state["z"] = shares(gen, z, 64)
    elif kind == "stream":
        # factors of 5 integer and 26 fractional bits; a product of two values for the truncation
        state["x"] = shares(gen, torch.randint(-(1 << 31) + 1, 1 << 31, (n,), generator=gen, device="cuda"), 64)
        state["y"] = shares(gen, torch.randint(-(1 << 31) + 1, 1 << 31, (n,), generator=gen, device="cuda"), 64)
    else:
        state["x"] = shares(gen, values(gen, n, case["setting"], k_in), ell + k_in)
    if kind == "records":
        state["op"] = B.BC_OP_RELU if case["op"] == "relu" else B.BC_OP_DRELU
        state["record"] = torch.zeros(B.rand_bytes(state["op"], prm, n), dtype=torch.uint8, device="cuda")
    # output and message buffers that a serving loop keeps from call to call
    state["out"] = tuple(torch.empty_like(t) for t in state["x"])
    if kind == "step":
        state["zout"] = tuple(torch.empty_like(t) for t in state["z"])
    if kind == "apart":
        words = B.msg_words(prm.npos)
        state["msg"] = tuple(torch.empty((words, n), dtype=torch.int32, device="cuda") for _ in range(2))
        state["reply"] = tuple(torch.empty_like(t) for t in state["x"])
    return state


def run(state):
    case, prm, sd, out = state["case"], state["prm"], state["sd"], state["out"]
    kind, relu = case["kind"], case["op"] == "relu"
    if kind == "call":
        x0, x1 = state["x"]
        if case["k_in"]:
            fn = B.trunc_relu if relu else B.trunc_drelu
            return fn(x0, x1, prm.ell + case["k_in"], case["k_in"], prm, sd, out=out)
        return (B.relu if relu else B.drelu)(x0, x1, prm, sd, out=out)
    if kind == "step":
        return B.trunc_det(*state["z"], 64, case["k_in"], out=state["zout"]) + B.drelu(*state["x"], prm, sd, out=out)
    if kind == "stream":
        if case["op"] == "mul":
            return B.mul_trunc(*state["x"], *state["y"], 64, case["k_in"], B.BC_TRUNC_BEFORE, sd, out=out)
        return B.trunc_det(*state["x"], 64, case["k_in"], out=out)
    if kind == "batch":
        state["batch"].run()
        return out
    if kind == "records":
        rec = B.rand_expand(state["op"], prm, sd, case["n"], out=state["record"])
        return (B.relu_pre if relu else B.drelu_pre)(*state["x"], prm, rec, out=out) + (rec,)
    if kind == "rss":
        return (B.rss_relu if relu else B.rss_drelu)(state["x"], prm, sd, out=out)
    m0 = B.drelu_send(0, state["x"][0], prm, sd, out=state["msg"][0])
    m1 = B.drelu_send(1, state["x"][1], prm, sd, out=state["msg"][1])
    d0, d1 = B.drelu_reply(m0, m1, prm, sd, out=state["reply"])
    return m0, m1, B.drelu_finish(0, d0, prm, sd, out=out[0]), B.drelu_finish(1, d1, prm, sd, out=out[1])


# --------------------------------------------------------------------- work


def draw_blocks(lx):
    """128-bit generator blocks of the shuffle and of the masks of one element."""
    n = lx + 1
    shuffle = 1 if n <= 19 else 2 if n <= 32 else 3
    return shuffle, (2 * n * n + 127) // 128 if n >= 17 else (n + 1) // 2


def work(case):
    """Bytes: shares, messages and records read and written once.  Operations: 32-bit integer operations of the
    method (60 a generator block, 46 a window slot, 64 + 6 where the field is wider than 32 bits, and the end)."""
    ell, lx, _ = SETTINGS[case["setting"]][:3]
    kind, relu, np = case["kind"], case["op"] != "drelu", lx + 1
    w = 4 if ell <= 32 else 8
    n = sum(int(s) for s in case["sizes"].split(",")) if kind == "batch" else case["n"]
    shuffle, masks = draw_blocks(lx)
    slots = np * ((70 if lx == 32 else 46))
    if kind == "stream":
        return {"bytes": n * (48 if case["op"] == "mul" else 32), "flops": n * (220 if case["op"] == "mul" else 10)}
    if kind == "rss":
        blocks = shuffle + masks + (7 if relu else 6)
        return {"bytes": n * 6 * w, "flops": n * (60 * blocks + slots + (160 if relu else 100))}
    if kind == "apart":
        words = (np * np + 31) // 32
        return {"bytes": n * (2 * (w + 4 * words) + 8 * words + 2 * w + 4 * w),
                "flops": n * (60 * (2 * (shuffle + masks) + 3) + 2 * slots)}
    ops = 60 * (shuffle + masks + (3 if relu else 1)) + slots + (40 if relu else 12)
    if kind == "records":
        k = 64 // np
        record = 4 * ((np + 3) // 4) + 8 * ((2 * np + k - 1) // k) + (w if relu else 0)
        return {"bytes": n * (4 * w + 2 * record), "flops": n * (ops + 60 * (3 if relu else 1))}
    if kind == "step":
        return {"bytes": n * 64, "flops": n * (ops + 10)}
    return {"bytes": n * 4 * w, "flops": n * ops}


def exact(case, seed):
    """Every output is a whole number (shares, messages, records) that depends on the library's own generator layout:
    there is no value in 64 bits for it to be near to, except where no draw enters."""
    if case["kind"] == "stream" and case["op"] == "trunc":
        x0, x1 = prepare(case, seed)["x"]
        k, keep = case["k_in"], (1 << (64 - case["k_in"])) - 1
        return [(x0 >> k) & keep, -((-x1 >> k) & keep) & keep]
    return None
