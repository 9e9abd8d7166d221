"""The performance cases of the framework: what its users have it do, from one minibatch of a
small table to whole launch-sets, and the one-off work that builds a packed table.

A case is a dict of plain values; `kind` says which calls it makes:

  step     one training iteration's loads: the input nodes' rows decoded (`gather_dequant`) and
           the fused neighbourhood mean of every hop's block (`gather_mean`)
  mean     the fused mean of the outermost block alone (a model's first layer)
  two_hop  two rounds of the mean in one call (linear propagation)
  rounds   rounds of averaging of 32-bit rows over a whole graph (`aggregate_rows`): what the
           layers after the first and the aggregation scale profile do
  build    fit a scalar quantizer to a table streamed in chunks, then encode and pack it
  train    codebook training on a row sample
  encode   nearest-entry search and packing of a chunk with given codebooks

Tables, graphs and features are synthetic: codes of normally distributed features, node degrees
with a power-law tail (exponent 2.1, capped at 10 000) and neighbours drawn in proportion to
degree, so blocks have the short and repeated lists that neighbourhood sampling gives.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2207_14696_amd as bf

KINDS = {"uniform": bf.UNIFORM, "log": bf.LOG, "vq": bf.VQ}
CAP = 10_000        # largest degree
TAIL = 1.1          # Pareto exponent of the degrees minus one
E_MIN, E_MAX = -6.0, 1.75   # log2 of the magnitudes the logarithmic codes span
FANOUTS = [(10,), (25, 10), (25, 15), (15, 10, 5), (10, 25), (5, 10, 15)]


def _load(name, kind, scheme, N, D, batch, fanouts, minibatches, **kw):
    case = {"name": name, "kind": kind, "scheme": scheme, "bits": 8, "width": 0, "length": 0, "cosine": False,
            "N": N, "D": D, "graph": "powerlaw", "degree": 15, "batch": batch, "minibatches": minibatches,
            "fanouts": ",".join(map(str, fanouts)), "promise": True, "idx32": False, "row_align": 16}
    case.update(kw)
    return case


def _table(name, kind, scheme, rows, D, **kw):
    case = {"name": name, "kind": kind, "scheme": scheme, "bits": 8, "width": 0, "length": 0, "cosine": False,
            "rows": rows, "D": D, "half": False, "clip": 0.0, "chunks": 1}
    case.update(kw)
    return case


def listed():
    return [
        # one minibatch of a small graph: launches and latency are what count
        _load("step_8bit_d128_small", "step", "uniform", 10_000, 128, 1024, (10,), 1, graph="uniform"),
        # one minibatch of a products-sized graph, two hops, as a plain training loop calls it
        _load("step_4bit_d100_one_batch", "step", "uniform", 2_400_000, 100, 1024, (25, 10), 1, bits=4),
        # eight prefetched minibatches of three hops on narrow rows (a citation graph at 2 bits)
        _load("step_2bit_d128_three_hops", "step", "uniform", 16_000_000, 128, 1024, (15, 10, 5), 8, bits=2),
        # first layer of a wide table (768 columns at 4 bits), 32 prefetched minibatches
        _load("mean_4bit_d768", "mean", "uniform", 4_000_000, 768, 1024, (25, 15), 32, bits=4, degree=12),
        # first layer from the paper's own logarithmic codes, 32-bit list entries
        _load("mean_log4_d128", "mean", "log", 16_000_000, 128, 1024, (15, 10, 5), 8, bits=4, idx32=True),
        # a training iteration from vector codes: 96 parts, 256 entries of 8 columns
        _load("step_vq_96x256x8", "step", "vq", 8_000_000, 768, 4096, (25, 10), 4, width=8, length=256),
        # the paper's large-graph vector setting: 16 columns a part, 2048 entries, two-byte indices
        _load("step_vq_8x2048x16", "step", "vq", 16_000_000, 128, 1024, (15, 10, 5), 4, width=16, length=2048,
              cosine=True),
        # two rounds of propagation with nothing in between, on the wide table
        _load("two_hop_4bit_d768", "two_hop", "uniform", 4_000_000, 768, 1024, (25, 15), 32, bits=4, degree=12),
        # the profiling run that chooses a compression ratio: rounds of averaging over a whole graph
        {"name": "rounds_d100_1m", "kind": "rounds", "N": 1 << 20, "D": 100, "degree": 15, "layers": 2},
        # one-off preprocessing: a half-precision table fitted and packed to 4 bits, two chunks
        _table("build_4bit_d768_half", "build", "uniform", 1 << 20, 768, bits=4, half=True, chunks=2),
        # codebooks of the 96-part setting trained on the usual 65 536-row sample
        _table("train_vq_96x256x8", "train", "vq", 65_536, 768, width=8, length=256),
        # a chunk of the table encoded with those codebooks
        _table("encode_vq_96x256x8", "encode", "vq", 262_144, 768, width=8, length=256),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "mean", "mean", "two_hop", "rounds", "build", "train", "encode"])
    vq = kind in ("train", "encode") or (kind != "build" and rng.random() < 0.3)
    scheme = "vq" if vq else rng.choice(["uniform", "uniform", "log"])
    width = rng.choice([4, 8, 8, 16, 16, 12, 32]) if vq else 0
    parts = _log_uniform(rng, 6, 96)
    D = max(width, min(768, parts * width)) if vq else rng.choice([100, 128, 256, 602, 768, _log_uniform(rng, 40, 768)])
    if vq:
        D = D // width * width - (rng.randrange(width) if rng.random() < 0.2 and D >= 2 * width else 0)
    common = {"bits": rng.choice([1, 2, 4, 8]), "width": width,
              "length": rng.choice([64, 256, 256, 1000, 2048]) if vq else 0,
              "cosine": bool(vq and rng.random() < 0.3)}
    if kind == "rounds":
        case = {"kind": kind, "N": _log_uniform(rng, 20_000, 1 << 20), "D": rng.choice([100, 64, 37, 128, 101]),
                "degree": rng.choice([8, 12, 15]), "layers": rng.choice([1, 2])}
    elif kind in ("build", "train", "encode"):
        rows = {"build": _log_uniform(rng, 20_000, 1 << 20), "train": _log_uniform(rng, 4096, 65_536),
                "encode": _log_uniform(rng, 1000, 262_144)}[kind]
        case = _table("", kind, scheme, rows, D, half=rng.random() < 0.5,
                      clip=0.01 if scheme == "log" and rng.random() < 0.5 else 0.0,
                      chunks=rng.choice([1, 2, 3]) if kind == "build" else 1, **common)
    else:
        fan = rng.choice(FANOUTS[1:] if kind == "two_hop" else FANOUTS)
        case = _load("", kind, scheme, _log_uniform(rng, 10_000, 16_000_000), D, rng.choice([256, 1000, 1024, 4096]), fan,
                     _log_uniform(rng, 1, 32), degree=rng.choice([8, 12, 15]), promise=rng.random() < 0.7,
                     idx32=kind != "two_hop" and rng.random() < 0.3, row_align=rng.choice([16, 16, 16, 128]), **common)
        case["N"] = min(case["N"], (2 << 30) // D)
    case.pop("name", None)
    # no dearer than the listed ones of the same kind
    same = [work(c) for c in listed() if c["kind"] == kind]
    most_bytes = max(w["bytes"] for w in same)
    most_flops = max(w["flops"] for w in same) * (0.15 if kind in ("train", "encode") else 1.0)
    while True:
        w = work(case)
        if w["bytes"] <= most_bytes and w["flops"] <= most_flops:
            return case
        key = "rows" if "rows" in case else "N" if kind == "rounds" else "minibatches"
        if case[key] > 1:
            case[key] = case[key] // 2
        else:
            case["batch"] //= 2
        if kind == "train":
            case["length"] = min(case["length"], case["rows"] // 4)


# ------------------------------------------------------------------ inputs

def _gen(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    return g


class _Graph:
    """Degrees floor(d_min * x^(-1/TAIL)) capped at CAP over node ranks x in (0, 1)."""

    def __init__(self, N, degree, uniform, gen, device):
        self.N, self.degree, self.uniform, self.gen, self.device = N, degree, uniform, gen, device
        lo, hi = 0.01, float(degree)
        for _ in range(60):
            self.d_min = 0.5 * (lo + hi)
            if self._mean() < degree:
                lo = self.d_min
            else:
                hi = self.d_min

    def _mean(self):
        self.top = (self.d_min / CAP) ** TAIL    # share of nodes at the cap
        return CAP * self.top + self.d_min * 11.0 * (1.0 - self.top ** (1 / 11.0))

    def nodes(self, n):
        return torch.randint(0, self.N, (n,), generator=self.gen, device=self.device)

    def degrees(self, rank):
        if self.uniform:
            return torch.full_like(rank, int(self.degree))
        x = (rank.double() + 0.5) / self.N
        return (self.d_min * x.pow(-1 / TAIL)).floor().clamp(1, CAP).long()

    def neighbours(self, n):
        if self.uniform:
            return self.nodes(n)
        m = self._mean()
        u = torch.rand(n, generator=self.gen, device=self.device, dtype=torch.float64) * m
        head = u / CAP
        tail = (self.top ** (1 / 11.0) + (u - CAP * self.top).clamp(min=0) / (11.0 * self.d_min)).pow(11.0)
        x = torch.where(head < self.top, head, tail)
        return (x * self.N).long().clamp(0, self.N - 1)

    def ids(self, rank):    # ranks scattered over the table's rows
        return (rank * 1_000_003 + 12_345) % self.N


def _blocks(case, gen, device, counts=None):
    """Sampled blocks of all minibatches concatenated: per hop (indptr, table rows, positions of
    the entries in the next hop's destinations), and the rows of the input nodes.
    counts: destinations of every hop after the first and input nodes; blocks are cut or filled
    up to them, as a loader does whose buffers have one size."""
    g = _Graph(case["N"], case["degree"], case["graph"] == "uniform", gen, device)
    n = case["batch"] * case["minibatches"]
    dst = g.nodes(n)                                       # ranks of the seeds
    batch = torch.arange(n, device=device) // case["batch"]
    hops = []
    for hop, fan in enumerate(map(int, case["fanouts"].split(","))):
        cnt = torch.minimum(g.degrees(dst), torch.tensor(fan, device=device))
        indptr = torch.zeros(dst.numel() + 1, dtype=torch.int64, device=device)
        torch.cumsum(cnt, 0, out=indptr[1:])
        src = g.neighbours(int(indptr[-1]))
        key, local = torch.unique(torch.repeat_interleave(batch, cnt) * case["N"] + src, return_inverse=True)
        hops.append((indptr, g.ids(src), local))
        if counts is not None:
            key = torch.cat([key, key[:max(0, counts[hop] - key.numel())]])[:counts[hop]]
        dst, batch = key % case["N"], key // case["N"]
    return hops, g.ids(dst)


def _row_bytes(case):
    if case["scheme"] == "vq":
        n = -(-case["D"] // case["width"]) * (1 if case["length"] <= 256 else 2)
    else:
        n = -(-case["D"] * case["bits"] // 8)
    return -(-n // 16) * 16


def _scalar_codes(case, rows, gen, device):
    """Codes of normally distributed values, one per column."""
    z = torch.randn(rows, case["D"], generator=gen, device=device)
    if case["scheme"] == "uniform":
        top = (1 << case["bits"]) - 1
        return ((z + 3.5) * (top / 7.0)).round_().clamp_(0, top).to(torch.uint8)
    half = 1 << (case["bits"] - 1)
    level = ((z.abs().log2() - E_MIN) * (half / (E_MAX - E_MIN))).floor_().clamp_(0, half - 1)
    return torch.where(z > 0, half + level, half - 1 - level).to(torch.uint8)


def _pack(codes, bits, width):
    """Column j's code at bit (j*bits) % 8 of byte j*bits // 8, rows padded with zeros to width."""
    per = 8 // bits
    rows, D = codes.shape
    full = torch.zeros(rows, -(-D // per) * per, dtype=torch.uint8, device=codes.device)
    full[:, :D] = codes
    out = torch.zeros(rows, width, dtype=torch.uint8, device=codes.device)
    cells = full.view(rows, -1, per)
    for k in range(per):
        out[:, :cells.shape[1]] |= cells[:, :, k] << (bits * k)
    return out


def _stride(case):
    n = _row_bytes(case)
    if case["row_align"] == 16:
        return n
    return 1 << max(4, (n - 1).bit_length()) if n <= 128 else -(-n // 128) * 128


def _packed_table(case, gen, device):
    N, stride = case["N"], _stride(case)
    table = torch.zeros(N, stride, dtype=torch.uint8, device=device)
    step = max(1, (1 << 27) // case["D"])
    for r0 in range(0, N, step):
        rows = min(step, N - r0)
        if case["scheme"] == "vq":
            P = -(-case["D"] // case["width"])
            c = torch.randint(0, case["length"], (rows, P), generator=gen, device=device, dtype=torch.int32)
            if case["length"] <= 256:
                table[r0:r0 + rows, :P] = c.to(torch.uint8)
            else:
                table[r0:r0 + rows, 0:2 * P:2] = (c & 255).to(torch.uint8)
                table[r0:r0 + rows, 1:2 * P:2] = (c >> 8).to(torch.uint8)
        else:
            table[r0:r0 + rows] = _pack(_scalar_codes(case, rows, gen, device), case["bits"], stride)
    return table


def _columns(D, gen, device):
    """Location and scale of every column."""
    mu = torch.rand(D, generator=gen, device=device) * 2 - 1
    return mu, torch.rand(D, generator=gen, device=device) * 1.5 + 0.5


def _features(case, gen, device):
    mu, sigma = _columns(case["D"], gen, device)
    x = torch.randn(case["rows"], case["D"], generator=gen, device=device) * sigma + mu
    return x.half() if case["half"] else x


def _codebooks(case, gen, device):
    """[P, length, width]: points of the columns' own distribution (a short last part is padded with 0)."""
    P, w, D = -(-case["D"] // case["width"]), case["width"], case["D"]
    mu, sigma = _columns(D, gen, device)
    cb = torch.zeros(case["length"], P * w, device=device)
    cb[:, :D] = torch.randn(case["length"], D, generator=gen, device=device) * (0.9 * sigma) + mu
    return cb.view(case["length"], P, w).permute(1, 0, 2).contiguous()


def _ranges(case, gen, device):
    mu, sigma = _columns(case["D"], gen, device)
    return mu - 3.5 * sigma, mu + 3.5 * sigma


def _scheme(case):
    return bf.Scheme(KINDS[case["scheme"]], case["bits"], case["width"], case["length"],
                     bf.VQ_COSINE if case["cosine"] else bf.VQ_L2)


def _inputs(case, seed, device):
    """Everything that is made from the seed, apart from the framework's own objects."""
    gen = _gen(seed, device)
    if case["kind"] == "rounds":
        g = _Graph(case["N"], case["degree"], False, gen, device)
        rank = torch.arange(case["N"], device=device)
        deg = torch.empty_like(rank)
        deg[g.ids(rank)] = g.degrees(rank) + 1              # every node lists itself first
        indptr = torch.zeros(case["N"] + 1, dtype=torch.int64, device=device)
        torch.cumsum(deg, 0, out=indptr[1:])
        indices = g.ids(g.neighbours(int(indptr[-1])))
        indices[indptr[:-1]] = rank
        return {"x": torch.randn(case["N"], case["D"], generator=gen, device=device), "indptr": indptr,
                "indices": indices}
    if case["kind"] in ("build", "train", "encode"):
        # the codebooks and the rows have the same columns: both start from the same generator
        s = {"x": _features(case, gen, device)}
        if case["kind"] == "encode":
            s["cb"] = _codebooks(case, _gen(seed, device), device)
        return s
    s = {"codes": _packed_table(case, gen, device)}
    # two_hop gives a row per seed; the positions of its entries need the blocks as they are
    counts = None if case["kind"] == "two_hop" else _counts(case)
    s["hops"], s["nodes"] = _blocks(case, gen, device, counts)
    if case["scheme"] == "vq":
        s["cb"] = _codebooks(case, gen, device)
    elif case["scheme"] == "uniform":
        s["mn"], s["mx"] = _ranges(case, gen, device)
    return s


def prepare(case, seed):
    s = _inputs(case, seed, "cuda")
    if case["kind"] == "rounds":
        return {"case": case, **s}
    q = bf.Quantizer(_scheme(case), case["D"], case.get("row_align", 16))
    state = {"case": case, "q": q}
    if case["kind"] in ("build", "train", "encode"):
        state["chunks"] = list(s["x"].chunk(case["chunks"]))
        if case["kind"] == "encode":
            q.params_set_codebooks(s["cb"].cpu().numpy())
        if case["clip"] > 0:
            q.fit_set_log_clip(case["clip"])
        if case["kind"] != "train":
            state["codes"] = torch.empty(case["rows"], q.row_bytes, dtype=torch.uint8, device="cuda")
        return state
    if case["scheme"] == "vq":
        q.params_set_codebooks(s["cb"].cpu().numpy())
    elif case["scheme"] == "uniform":
        q.params_set_uniform(s["mn"].cpu().numpy(), s["mx"].cpu().numpy())
    else:
        q.params_set_log(E_MIN, E_MAX)
    if case["promise"]:
        q.set_option("mean_max_degree", max(map(int, case["fanouts"].split(","))))
    state["codes"], state["nodes"] = s["codes"], s["nodes"]
    hops = s["hops"] if case["kind"] != "mean" else s["hops"][-1:]
    state["hops"] = [(p, i.int() if case["idx32"] else i, l if case["kind"] == "two_hop" else None)
                     for p, i, l in hops]
    return state


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "rounds":
        h = [state["x"]]
        for _ in range(case["layers"]):
            h.append(bf.aggregate_rows(h[-1], state["indptr"], state["indices"]))
        return h[1:]
    q = state["q"]
    if kind == "train":
        q.fit_reset()
        q.fit_update(state["chunks"][0])
        q.fit_finalize()
        return q.params_get_codebooks(), q.vq_distortion(10)
    if kind == "encode":
        q.quantize(state["chunks"][0], state["codes"], 0)
        return state["codes"]
    if kind == "build":
        q.fit_reset()
        again = True
        while again:
            for chunk in state["chunks"]:
                q.fit_update(chunk)
            again = q.fit_finalize()
        row0 = 0
        for chunk in state["chunks"]:
            q.quantize(chunk, state["codes"], row0)
            row0 += chunk.shape[0]
        # what is saved beside the packed table
        params = q.params_get_uniform() if case["scheme"] == "uniform" else q.params_get_log()[2:]
        return (state["codes"],) + tuple(params)
    codes, hops = state["codes"], state["hops"]
    if kind == "mean":
        return q.gather_mean(codes, hops[0][0], hops[0][1])
    if kind == "two_hop":
        (p2, _, local), (p1, i1, _) = hops[-2], hops[-1]
        return q.gather_mean_2hop(codes, p1, i1, p2, local)
    return [q.gather_dequant(codes, state["nodes"])] + [q.gather_mean(codes, p, i) for p, i, _ in hops]


# ------------------------------------------------------------------ what a pass cannot do without

@functools.lru_cache(maxsize=None)
def _sizes(items):
    """Sizes of one draw of the blocks (they hardly change from seed to seed)."""
    case = dict(items)
    device = "cuda" if torch.cuda.is_available() else "cpu"
    hops, nodes = _blocks(case, _gen(0, device), device)
    out = []
    for p, rows, local in hops:
        out.append((p.numel() - 1, rows.numel(), int(torch.unique(rows).numel())))
    inner = 0
    if len(hops) > 1:   # packed rows that the last two hops' lists need in all, one list per entry
        p1 = hops[-1][0]
        inner = int((p1[1:] - p1[:-1])[hops[-2][2]].sum())
    return out, int(nodes.numel()), inner


def _block_sizes(case):
    return _sizes(tuple(sorted((k, v) for k, v in case.items() if k in (
        "N", "degree", "graph", "batch", "minibatches", "fanouts"))))


def _counts(case):
    hops, nodes, _ = _block_sizes(case)
    return [V for V, _, _ in hops[1:]] + [nodes]


def work(case):
    D = case["D"]
    if case["kind"] == "rounds":
        N, layers = case["N"], case["layers"]
        entries = N * (case["degree"] + 1)
        return {"bytes": layers * (8 * N + 8 * entries + 8 * D * N), "flops": layers * D * entries}
    if case["kind"] in ("build", "train", "encode"):
        rows, size = case["rows"], 2 if case["half"] else 4
        if case["kind"] == "build":
            passes = 4 if case["clip"] > 0 else 2
            return {"bytes": rows * (passes * size * D + _row_bytes(case)), "flops": rows * D * (passes + 2)}
        P = -(-D // case["width"])
        rounds = 10 if case["kind"] == "train" else 1
        books = 4 * P * case["length"] * case["width"]
        out = books if case["kind"] == "train" else rows * _row_bytes(case)
        # a distance is a dot product: one multiply and one add per column
        return {"bytes": size * rows * D + out + (books if case["kind"] == "encode" else 0),
                "flops": 2 * rounds * rows * P * case["width"] * case["length"]}
    hops, nodes, inner = _block_sizes(case)
    rb, ib = _row_bytes(case), 4 if case["idx32"] else 8
    bytes_ = flops = 0
    if case["kind"] == "two_hop":
        (V2, E2, _), (V1, E1, U1) = hops[-2], hops[-1]
        return {"bytes": 8 * (V1 + V2 + E2 + E1) + rb * U1 + 4 * D * V2, "flops": D * (inner + E2)}
    for V, E, U in hops if case["kind"] == "step" else hops[-1:]:
        bytes_ += 8 * V + ib * E + rb * U + 4 * D * V
        flops += D * E
    if case["kind"] == "step":
        bytes_ += nodes * (8 + rb + 4 * D)
        flops += 2 * D * nodes
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["kind"] in ("build", "encode"):
        return "exact"          # codes and the parameters beside them are defined bit by bit
    if case["kind"] == "train":
        # k-means is iterated: a part at nearly the same distance from two entries goes to the
        # other one when the sums before it were added in another order
        # (twice the same inputs: 6e-4; against 64 bits: 1.2e-3)
        return {"rel": 5e-3}
    # sums in 32 bits, at most 4.6e-7 from the 64-bit result (two rounds)
    return {"rel": 2e-6}


# ------------------------------------------------------------------ 64-bit results in plain torch

def _decoder(case, s):
    """rows -> [n, D] doubles."""
    D, bits = case["D"], case["bits"]
    if case["scheme"] == "vq":
        P, w = -(-D // case["width"]), case["width"]
        books, part = s["cb"].double(), torch.arange(P, device=s["cb"].device)

        def decode(rows):
            raw = s["codes"][rows].long()
            c = raw[:, :P] if case["length"] <= 256 else raw[:, 0:2 * P:2] + 256 * raw[:, 1:2 * P:2]
            return books[part, c].reshape(rows.numel(), P * w)[:, :D]
        return decode
    per = 8 // bits
    shift = torch.arange(per, device=s["codes"].device) * bits

    def codes_of(rows):
        raw = s["codes"][rows][:, :-(-D // per)].long()
        return ((raw[:, :, None] >> shift) & ((1 << bits) - 1)).reshape(rows.numel(), -1)[:, :D]
    if case["scheme"] == "uniform":
        mn, mx = s["mn"].double(), s["mx"].double()
        scale = ((mx - mn) / ((1 << bits) - 1)).float().double()    # stored in 32 bits
        return lambda rows: mn + codes_of(rows) * scale
    table = torch.from_numpy(_log_tables(bits, E_MIN, E_MAX)[1]).to(s["codes"].device).double()
    return lambda rows: table[codes_of(rows)]


def _log_tables(bits, e_min, e_max):
    half = 1 << (bits - 1)
    step = (e_max - e_min) / half
    edges = np.array([2.0 ** (e_min + i * step) for i in range(1, half)], np.float64).astype(np.float32)
    mid = np.array([2.0 ** (e_min + (i + 0.5) * step) for i in range(half)], np.float64).astype(np.float32)
    return edges, np.concatenate([-mid[::-1], mid])


def _list_means(fetch, indptr, indices, D):
    """Mean over every list of fetch(indices), an empty list giving zeros."""
    V, n = indptr.numel() - 1, indptr[1:] - indptr[:-1]
    out = torch.zeros(V, D, dtype=torch.float64, device=indptr.device)
    dst = torch.repeat_interleave(torch.arange(V, device=indptr.device), n)
    step = max(1, (1 << 27) // D)
    for e0 in range(0, indices.numel(), step):
        out.index_add_(0, dst[e0:e0 + step], fetch(indices[e0:e0 + step]))
    return out / n.clamp(min=1)[:, None]


def _decode_all(decode, rows, D):
    out = torch.empty(rows.numel(), D, dtype=torch.float64, device=rows.device)
    step = max(1, (1 << 27) // D)
    for r0 in range(0, rows.numel(), step):
        out[r0:r0 + step] = decode(rows[r0:r0 + step])
    return out


def _nearest(case, x, cb):
    """The encoder's rule: 32-bit scores, columns in order, multiply and add rounded apart, the
    lowest index of equal ones."""
    P, w = cb.shape[:2][0], case["width"]
    norm = cb.double().pow(2).sum(2)
    rnorm = torch.where(norm > 0, 1 / norm.sqrt(), torch.zeros_like(norm)).float()
    out = torch.empty(x.shape[0], P, dtype=torch.int64, device=x.device)
    pad = torch.zeros(x.shape[0], P * w, dtype=torch.float32, device=x.device)
    pad[:, :x.shape[1]] = x.float()
    step = max(1, (1 << 27) // case["length"])
    for p in range(P):
        for r0 in range(0, x.shape[0], step):
            rows = pad[r0:r0 + step, p * w:(p + 1) * w]
            acc = torch.zeros(rows.shape[0], case["length"], device=x.device)
            for d in range(w):
                if case["cosine"]:
                    acc += rows[:, d:d + 1] * cb[p, :, d]
                else:
                    t = rows[:, d:d + 1] - cb[p, :, d]
                    acc += t.mul_(t)
            if case["cosine"]:
                acc = -(acc * rnorm[p])
            best = acc.min(1, keepdim=True).values
            out[r0:r0 + step, p] = (acc == best).int().argmax(1)
    return out


def _exact_train(case, x):
    """Ten Lloyd rounds in 64 bits from the sample's first rows."""
    P, w, D, length = -(-case["D"] // case["width"]), case["width"], case["D"], case["length"]
    pad = torch.zeros(x.shape[0], P * w, dtype=torch.float64, device=x.device)
    pad[:, :D] = x.double()
    books, dist = torch.empty(P, length, w, dtype=torch.float64, device=x.device), np.zeros(10)
    for p in range(P):
        rows = pad[:, p * w:(p + 1) * w]
        cb = rows[:length].clone()
        for k in range(10):
            sq = cb.pow(2).sum(1)
            if case["cosine"]:
                score = -(rows @ cb.T) * torch.where(sq > 0, 1 / sq.sqrt(), torch.zeros_like(sq))
            else:
                score = sq - 2 * (rows @ cb.T)
            best = score.argmin(1)
            dist[k] += float((rows - cb[best]).pow(2).sum())
            sums = torch.zeros_like(cb).index_add_(0, best, rows)
            count = torch.bincount(best, minlength=length)[:, None]
            cb = torch.where(count > 0, sums / count.clamp(min=1), cb)
        books[p] = cb
    return books.cpu().numpy(), dist / x.shape[0]


def _exact_build(case, x):
    # codes compare 32-bit values by rule; the parameters are 64-bit results rounded once
    if case["scheme"] == "uniform":
        mn, mx = x.amin(0).float() + 0.0, x.amax(0).float() + 0.0
        span, top = mx.double() - mn.double(), float((1 << case["bits"]) - 1)
        scale = span / top
        inv = torch.where(span > 0, top / span, torch.zeros_like(span))
        codes = ((x.float() - mn) * inv.float()).round_().clamp_(0, top).to(torch.uint8)
        return (_pack(codes, case["bits"], _row_bytes(case)), mn.double().cpu().numpy(), mx.double().cpu().numpy(),
                scale.cpu().numpy(), inv.cpu().numpy())
    mag = x.float().abs().flatten()
    mag = mag[mag > 0]
    n, f = mag.numel(), case["clip"]
    if f > 0:
        mag = mag.sort().values
        lo, hi = float(mag[math.floor(f * (n - 1))]), float(mag[math.ceil((1 - f) * (n - 1))])
    else:
        lo, hi = float(mag.min()), float(mag.max())
    edges, values = _log_tables(case["bits"], math.log2(lo), math.log2(hi))
    del mag
    half = 1 << (case["bits"] - 1)
    level = torch.zeros(x.shape, dtype=torch.uint8, device=x.device)
    for t in edges:
        level += x.float().abs() >= float(t)
    codes = torch.where(x > 0, half + level, half - 1 - level)
    return (_pack(codes, case["bits"], _row_bytes(case)), edges.astype(np.float64), values.astype(np.float64))


def exact(case, seed):
    s = _inputs(case, seed, "cuda")
    D = case["D"]
    if case["kind"] == "rounds":
        h = [s["x"].double()]
        for _ in range(case["layers"]):
            h.append(_list_means(lambda i: h[-1][i], s["indptr"], s["indices"], D))
        return h[1:]
    if case["kind"] == "train":
        return _exact_train(case, s["x"])
    if case["kind"] == "encode":
        c = _nearest(case, s["x"], s["cb"])
        if case["length"] > 256:
            c = torch.stack([c & 255, c >> 8], 2).flatten(1)
        return _pack(c.to(torch.uint8), 8, _row_bytes(case))
    if case["kind"] == "build":
        return _exact_build(case, s["x"])
    decode = _decoder(case, s)
    hops = s["hops"]
    if case["kind"] == "mean":
        return _list_means(decode, hops[-1][0], hops[-1][1], D)
    if case["kind"] == "two_hop":
        first = _list_means(decode, hops[-1][0], hops[-1][1], D)
        return _list_means(lambda i: first[i], hops[-2][0], hops[-2][2], D)
    return [_decode_all(decode, s["nodes"], D)] + [_list_means(decode, p, i, D) for p, i, _ in hops]
