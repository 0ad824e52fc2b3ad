"""What the library is timed on: its public entry points over the sizes a served Qwen3-shaped model uses.

A case names a kind of call and its sizes.  prepare() holds what a serving program has in hand (packed
codes, row scales, activations, outputs, the prompt product's workspace), run() makes the calls, exact()
gives the same outputs in float64 from the method's definition, without the library.

Words are uniformly random (every 48-bit value is a legal code word, and the kernels' work does not depend
on them); row scales, tails, activations and 4-bit tables follow the distributions of the test workloads.
The encoder gets Gaussian blocks, as rotated weights are.
"""

import functools
import itertools
import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2609_35465_amd as tt

# hidden, q, kv and inner widths of the dense Qwen3 layers
WIDTHS = {"4B": (2560, 4096, 1024, 9728), "8B": (4096, 4096, 1024, 12288), "14B": (5120, 5120, 1024, 17408)}


def listed():
    def layer(model):
        return dict(zip(("hidden", "q", "kv", "inter"), WIDTHS[model]))

    return [
        # one small projection of one token: the smallest call, launch latency and little else
        {"name": "gemv-1536-b1", "kind": "gemv", "M": 1536, "K": 1536, "batch": 1},
        # q, k and v of a 4B layer for two sequences, one launch; K has a ragged tail of 16
        {"name": "qkv-4b-b2", "kind": "qkv", **layer("4B"), "batch": 2},
        # the headline: all projections of four 14B layers for one token, one launch
        {"name": "decode-14b-b1", "kind": "decode", **layer("14B"), "layers": 4, "batch": 1},
        # the same for four sequences served together
        {"name": "decode-14b-b4", "kind": "decode", **layer("14B"), "layers": 4, "batch": 4},
        # the projections of a 14B layer for a 203-token prompt, one product each
        {"name": "prompt-14b-203", "kind": "prompt", **layer("14B"), "N": 203},
        # the gate projection of an 8B layer for a long prompt
        {"name": "gemm-8b-4096", "kind": "gemm", "M": 12288, "K": 4096, "N": 4096},
        # a short chunk of a prompt through a small shard: rows, columns and tokens off every tile
        {"name": "gemm-ragged-33", "kind": "gemm", "M": 1000, "K": 2576, "N": 33},
        # an int4 projection (the 14B gate) of a served file, one token
        {"name": "int4-14b-b1", "kind": "int4", "M": 17408, "K": 5120, "batch": 1},
        # the 4-bit output head, one token
        {"name": "head-14b-b1", "kind": "head", "M": 151936, "K": 5120, "batch": 1},
        # the rotation before the 14B down projection of a 203-token prompt
        {"name": "rotate-14b-203", "kind": "rotate", "K": 17408, "block": 1024, "rows": 203},
        # the embedding rows of a 203-token prompt
        {"name": "embed-14b-203", "kind": "embed", "vocab": 151936, "K": 5120, "N": 203},
        # the offline encoder on the paper's 20,000 Gaussian blocks
        {"name": "encode-20000", "kind": "encode", "N": 20000},
    ]


def _log(rng, lo, hi, step=1):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step
    return max(-(-lo // step) * step, min(hi // step * step, v))


def draw(rng):
    kind = rng.choice(["gemv", "qkv", "decode", "prompt", "gemm", "gemm", "int4", "head", "rotate", "embed", "encode"])
    if kind == "gemv":
        return {"kind": kind, "M": _log(rng, 64, 17408), "K": _log(rng, 256, 17408, 2), "batch": rng.randint(1, 8)}
    if kind in ("qkv", "decode", "prompt"):
        hidden = _log(rng, 1024, 5120, 8)
        c = {"kind": kind, "hidden": hidden, "q": _log(rng, 1024, 5120, 8), "kv": _log(rng, 128, 1024, 8),
             "inter": int(hidden * rng.uniform(2.0, 3.4)) // 8 * 8}
        if kind == "prompt":
            return {**c, "N": _log(rng, 16, 512)}
        if kind == "decode":
            c["layers"] = rng.randint(1, 4)
        return {**c, "batch": rng.randint(1, 8)}
    if kind == "gemm":
        c = {"kind": kind, "M": _log(rng, 256, 17408), "K": _log(rng, 1024, 17408, 8)}
        most = 12288 * 4096 * 4096 // (c["M"] * c["K"])
        return {**c, "N": _log(rng, 9, min(4096, most))}
    if kind == "int4":
        return {"kind": kind, "M": _log(rng, 1024, 17408), "K": _log(rng, 1024, 17408, 128), "batch": rng.randint(1, 8)}
    if kind == "head":
        return {"kind": kind, "M": _log(rng, 30000, 151936), "K": _log(rng, 1024, 5120, 64), "batch": rng.randint(1, 8)}
    if kind == "rotate":
        n = 2 ** rng.randint(6, 12)
        return {"kind": kind, "K": n * rng.randint(1, 17408 // n), "block": n, "rows": _log(rng, 1, 512)}
    if kind == "embed":
        return {"kind": kind, "vocab": _log(rng, 30000, 151936), "K": _log(rng, 1024, 5120, 64), "N": _log(rng, 1, 2048)}
    return {"kind": kind, "N": _log(rng, 100, 20000)}


# ------------------------------------------------------------------ inputs

def _matrices(case):
    """[(M, K)] of the code matrices of one call, in the order of its outputs."""
    if case["kind"] in ("gemv", "gemm"):
        return [(case["M"], case["K"])]
    h, q, kv = case["hidden"], case["q"], case["kv"]
    group = [(q, h), (kv, h), (kv, h)]
    if case["kind"] == "qkv":
        return group
    f = case["inter"]
    return (group + [(h, q), (f, h), (f, h), (h, f)]) * case.get("layers", 1)


PHASES = (3, 1, 2, 1)          # q k v | o | gate up | down: matrices that may run side by side


def _groups(mats):
    """The dependency group of each matrix, over all layers."""
    return [g for g, n in enumerate(PHASES * (len(mats) // 7 + 1)) for _ in range(n)][:len(mats)]


def _rng(seed, index):
    return np.random.Generator(np.random.PCG64([int(seed), int(index)]))


def _code_matrix(seed, index, M, K):
    rng = _rng(seed, index)
    words = rng.integers(0, 1 << 48, size=(M, K // 24), dtype=np.uint64)
    sigma = (rng.uniform(0.5, 2.0, M) * 1e-2).astype(np.float16)
    tail = (rng.standard_normal((M, K % 24)) * sigma.astype(np.float64)[:, None]).astype(np.float16)
    return words, sigma, tail


def _activations(seed, index, rows, K):
    return _rng(seed, 1000 + index).standard_normal((rows, K), dtype=np.float32).astype(np.float16)


def _four_bit(seed, M, K, group):
    """(q uint8 [M, K/2], scale and offset fp16 [M, K/group, 2]) on the device."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    q = torch.randint(0, 256, (M, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    scale = (torch.rand((M, K // group), device="cuda", generator=gen) * 1.5 + 0.5) * (1e-2 / 8)
    return q, torch.stack([scale, -7.5 * scale], dim=-1).half()


def _inputs(case, seed):
    """Host matrices and activations of a call on code words: [(words, sigma, tail)], [x]; matrices of one
    dependency group and one width share an x, as the projections of a layer do."""
    mats = _matrices(case)
    rows = case.get("batch", case.get("N"))
    with ThreadPoolExecutor(8) as pool:
        host = list(pool.map(lambda a: _code_matrix(seed, a[0], *a[1]), enumerate(mats)))
    group = _groups(mats)
    xs = {g: _activations(seed, g, rows, K) for g, (_, K) in zip(group, mats)}
    return mats, host, [xs[g] for g in group], group


def _blocks(case, seed):
    rng = _rng(seed, 0)
    n = case["N"]
    return rng.standard_normal((n, 24), dtype=np.float32), np.ones(n, np.float32)


def _rotate_inputs(case, seed):
    rng = _rng(seed, 0)
    x = rng.standard_normal((case["rows"], case["K"]), dtype=np.float32).astype(np.float16)
    return x, rng.integers(0, 256, -(-case["K"] // 8), dtype=np.uint8)


def _tokens(case, seed):
    return _rng(seed, 0).integers(0, case["vocab"], case["N"]).astype(np.int32)


# ------------------------------------------------------------------ the calls

def prepare(case, seed):
    kind = case["kind"]

    def dev(a):
        return torch.from_numpy(a).cuda()

    def new(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device="cuda")

    if kind in ("int4", "head"):
        M, K, b = case["M"], case["K"], case["batch"]
        q, so = _four_bit(seed, M, K, 128 if kind == "int4" else 64)
        return {"kind": kind, "args": (q, so, dev(_activations(seed, 0, b, K)), new(b, M), M, K, b)}
    if kind == "rotate":
        x, bits = _rotate_inputs(case, seed)
        return {"kind": kind, "args": (dev(x), dev(bits), new(case["rows"], case["K"], dtype=torch.float16),
                                       case["K"], case["block"], case["rows"])}
    if kind == "embed":
        q, so = _four_bit(seed, case["vocab"], case["K"], 64)
        return {"kind": kind, "args": (q, so, case["vocab"], case["K"], dev(_tokens(case, seed)), new(case["N"], case["K"]))}
    if kind == "encode":
        w, sigma = _blocks(case, seed)
        return {"kind": kind, "args": (dev(w), dev(sigma), case["N"], new(case["N"], 6, dtype=torch.uint8))}

    mats, host, xs, group = _inputs(case, seed)
    with ThreadPoolExecutor(8) as pool:
        packed = list(pool.map(lambda a: tt.pack_rows(a[0][0], a[0][2], *a[1]), zip(host, mats)))
    on_dev = {g: dev(x) for g, x in zip(group, xs)}
    rows = case.get("batch", case.get("N"))
    items = [(dev(p), dev(h[1]), on_dev[g], new(rows, M), M, K)
             for p, h, g, (M, K) in zip(packed, host, group, mats)]
    state = {"kind": kind, "items": items, "rows": rows, "out": [i[3] for i in items]}
    if kind in ("qkv", "decode"):
        state["problems"] = tt.make_problems(items)
        state["phases"] = PHASES * case.get("layers", 1)
    if kind in ("gemm", "prompt"):
        state["workspace"] = tt.gemm_workspace()
    return state


def run(state):
    kind = state["kind"]
    if kind == "gemv":
        tt.gemv(*state["items"][0], state["rows"])
    elif kind == "qkv":
        tt.gemv_grouped(state["problems"], state["rows"])
    elif kind == "decode":
        tt.gemv_chain(state["problems"], state["phases"], state["rows"])
    elif kind in ("gemm", "prompt"):
        for item in state["items"]:
            tt.gemm(*item, state["rows"], state["workspace"])
    else:
        a = state["args"]
        if kind == "int4":
            tt.int4_gemv(*a)
        elif kind == "head":
            tt.head4_gemv(*a)
        elif kind == "rotate":
            tt.rotate(*a)
            return a[2]
        elif kind == "embed":
            tt.emb4_gather(*a)
            return a[5]
        else:
            tt.encode(*a)
        return a[3]
    return state["out"]


def work(case):
    kind = case["kind"]
    if kind in ("int4", "head"):
        M, K, b, g = case["M"], case["K"], case["batch"], 128 if kind == "int4" else 64
        return {"bytes": M * K // 2 + 4 * M * (K // g) + 2 * b * K + 4 * b * M, "flops": 2 * b * M * K}
    if kind == "rotate":
        n = case["rows"] * case["K"]
        return {"bytes": 4 * n + case["K"] // 8, "flops": n * int(math.log2(case["block"]))}
    if kind == "embed":
        N, K = case["N"], case["K"]
        return {"bytes": N * (K // 2 + 4 * (K // 64) + 4 + 4 * K), "flops": 2 * N * K}
    if kind == "encode":
        # the search's operations have no definite least count (it is a nearest-point search): the join of the
        # three sections over the 4096 paths and the free parities alone, at two radii
        return {"bytes": 106 * case["N"], "flops": case["N"] * 2 * 32768 * 2}
    rows = case.get("batch", case.get("N"))
    nbytes = flops = 0
    mats = _matrices(case)
    for M, K in mats:
        nbytes += M * (6 * (K // 24) + 2 * (K % 24) + 2) + 4 * rows * M
        flops += 2 * rows * M * K
    nbytes += sum(2 * rows * K for K in {g: K for g, (_, K) in zip(_groups(mats), mats)}.values())
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind in ("encode", "embed"):
        return "exact"                         # words; one rounded multiply and add per value
    if kind == "rotate":
        return {"rel": 8e-4}                   # results rounded to fp16 (measured: 2.1e-4 from float64)
    if kind in ("gemm", "prompt"):
        return {"rel": 8e-4}                   # each weight rounded once to fp16, then f32 sums (2.0e-4)
    if kind in ("int4", "head"):
        return {"rel": 4.5e-5}                 # f32 sums of 1024 + q, whose 1024 cancels (1.1e-5)
    return {"rel": 6e-7}                       # f32 sums of exact products (1.3e-7)


# ------------------------------------------------------------------ float64

@functools.lru_cache(maxsize=None)
def _tables():
    """The decoder's tables from the method's definition: pattern bytes of a path [4096, 3], ranks of the
    two class halves [4096, 8] and of the middle list [2048, 8], and the middle list's class-0 length."""
    gen = sum(1 << e for e in (0, 2, 4, 5, 6, 10, 11))      # of the cyclic [23, 12] Golay code
    code = set()
    for m in range(4096):
        c = 0
        for i in range(12):
            if m >> i & 1:
                c ^= gen << i
        code.add(c | (bin(c).count("1") & 1) << 23)
    octads = sorted(tuple(i for i in range(24) if c >> i & 1) for c in code if bin(c).count("1") == 8)
    first = octads[0]
    second = next(o for o in octads if not set(o) & set(first))
    order = [*first, *second, *(i for i in range(24) if i not in first and i not in second)]
    sections = [[sum((c >> order[8 * s + t] & 1) << t for t in range(8)) for s in range(3)] for c in code]
    low1 = sorted({min(s[0], s[0] ^ 255) for s in sections})
    low3 = sorted({min(s[2], s[2] ^ 255) for s in sections})
    edges = {p: sorted({(s[1], low3.index(min(s[2], s[2] ^ 255))) for s in sections if min(s[0], s[0] ^ 255) == p})
             for p in low1}
    paths = np.zeros((4096, 3), np.int64)      # index s8 | b1 << 6 | b2 << 7 | b3 << 11
    for s8, b1, b2, b3 in itertools.product(range(64), range(2), range(16), range(2)):
        p2, s16 = edges[low1[s8]][b2]
        paths[s8 | b1 << 6 | b2 << 7 | b3 << 11] = low1[s8] ^ 255 * b1, p2, low3[s16] ^ 255 * b3
    # rank vectors by (cost, packed value); the 2,048 cheapest of either class cost at most 96, so ranks stay below 5
    ranks = np.stack(np.meshgrid(*[np.arange(5)] * 8, indexing="ij"), -1).reshape(-1, 8)
    key = ((2 * ranks + 1) ** 2).sum(1) << 32 | (ranks << 4 * np.arange(8)).sum(1)
    ranks = ranks[np.argsort(key)]
    cls = np.isin(ranks, (1, 2, 5, 6)).sum(1) & 1
    rows = np.concatenate([ranks[cls == 0][:2048], ranks[cls == 1][:2048]])
    n0 = int((cls[:2048] == 0).sum())
    middle = np.concatenate([ranks[:2048][cls[:2048] == 0], ranks[:2048][cls[:2048] == 1]])
    return paths, rows, middle, n0


def _weights(words, sigma, tail):
    """float64 [rows, K] of code words int64 [rows, nblk] on the device (Eq. 2)."""
    paths, rows, middle, n0 = (torch.as_tensor(t, device=words.device) for t in _tables())

    def field(lsb, width):
        return words >> lsb & ((1 << width) - 1)

    p, r, i2 = field(6, 1), field(7, 1), field(26, 11)
    path = paths[field(0, 6) | field(8, 1) << 6 | field(9, 4) << 7 | field(13, 1) << 11]
    r3 = p ^ r ^ (i2 >= n0).long()
    rho = torch.cat([rows[2048 * r + field(15, 11)], middle[i2], rows[2048 * r3 + field(37, 11)]], -1)
    bits = (path[..., None] >> torch.arange(8, device=words.device) & 1).flatten(-2)
    # rank k of p + 2c + 4Z outward from zero, positive first at equal size
    u = 2 * rho + 1
    p = p[..., None]
    y = torch.where((rho ^ bits ^ p ^ 1) & 1 == 1, -u, u) + 1 - p
    norm = (y * y).sum(-1, keepdim=True).double().sqrt()
    gain = torch.tensor([4.3, 5.4], dtype=torch.float32, device=words.device).double()[field(14, 1)][..., None]
    w = torch.where(norm > 0, y * gain / norm.clamp(min=1.0), torch.zeros_like(norm)).flatten(1)
    return torch.cat([w * sigma[:, None].double(), tail.double()], 1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "encode":
        return None                            # whole numbers, compared exactly
    if kind == "rotate":
        x, bits = _rotate_inputs(case, seed)
        x = torch.from_numpy(x).cuda().double()
        sign = 1.0 - 2.0 * torch.from_numpy(np.unpackbits(bits, bitorder="little")[:case["K"]]).cuda().double()
        n = case["block"]
        h = torch.ones((1, 1), dtype=torch.float64, device="cuda")
        while h.shape[0] < n:
            h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
        return ((x * sign).reshape(-1, n) @ h / math.sqrt(n)).reshape(x.shape)
    if kind in ("int4", "head", "embed"):
        group = 128 if kind == "int4" else 64
        M, K = case.get("M", case.get("vocab")), case["K"]
        q, so = _four_bit(seed, M, K, group)
        if kind == "embed":
            at = torch.from_numpy(_tokens(case, seed)).cuda().long()
            q, so = q[at], so[at]
        x = None if kind == "embed" else torch.from_numpy(_activations(seed, 0, case["batch"], K)).cuda().double()
        out = []
        for i in range(0, q.shape[0], 16384):
            part, s = q[i:i + 16384].long(), so[i:i + 16384].double().repeat_interleave(group, 1)
            w = torch.stack([part & 15, part >> 4], -1).flatten(1) * s[..., 0] + s[..., 1]
            out.append(w if x is None else x @ w.T)
        return torch.cat(out, 0 if x is None else 1)
    out = []
    mats, host, xs, _ = _inputs(case, seed)
    for (M, K), (words, sigma, tail), x in zip(mats, host, xs):
        x = torch.from_numpy(x).cuda().double()
        step = max(1, (1 << 21) // (K // 24))
        out.append(torch.cat([x @ _weights(*(torch.from_numpy(a[i:i + step]).cuda() for a in
                                             (words.view(np.int64), sigma, tail))).T
                              for i in range(0, M, step)], 1))
    return out
