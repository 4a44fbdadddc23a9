"""The work whose speed is measured: what programs built on this library have it do, through its public entry points.

An index is trained or given centroids, filled with `encode_add`, and searched; some programs keep several indexes,
rank by inner product or distance of raw vectors, re-rank on raw rows, encode without storing, or read an index back
as vectors.  The listed cases are points of those uses at the sizes of `workloads/synth.py`, `bench.py` and the tests
(tiny 20,000 x 64; 1M x 128; 10M x 96; 10M x 200); `draw` spreads over the ranges between and around them.

Data are mixtures as in `workloads/synth.py`, drawn on the GPU from the seed: "iso" = components of different isotropic
width, "aniso" = anisotropic components scaled to unit length, "shifted" = the same without scaling and with queries
from shifted, wider components, "flat" = no clusters at all.  Centroids come from a few Lloyd iterations written here
(sums in integers, so that they depend on the seed alone), as a program would load them from an earlier training.
"""
from __future__ import annotations

import math

import torch

import paper_2605_17415_amd as pkg

DEV = "cuda:0"


def listed():
    return [
        # one user's query against a 1M index, as an interactive service sends it: latency
        {"name": "search_single", "kind": "search", "data": "iso", "n": 1_000_000, "d": 128, "nlist": 1024, "bits": 4, "sign": False,
         "metric": "cosine", "nq": 1, "nprobe": 32, "k": 10},
        # the handful of queries a server has gathered within a millisecond, against 10M vectors
        {"name": "search_16", "kind": "search", "data": "aniso", "n": 10_000_000, "d": 96, "nlist": 4096, "bits": 4, "sign": False,
         "metric": "cosine", "nq": 16, "nprobe": 32, "k": 10},
        # a medium batch with long results (candidates for a later stage), queries unlike the database
        {"name": "search_256_k100", "kind": "search", "data": "shifted", "n": 10_000_000, "d": 200, "nlist": 4096, "bits": 4, "sign": False,
         "metric": "cosine", "nq": 256, "nprobe": 64, "k": 100},
        # offline search of a whole query set: the two 10M configurations of the benchmark
        {"name": "search_10k_d96", "kind": "search", "data": "aniso", "n": 10_000_000, "d": 96, "nlist": 4096, "bits": 4, "sign": False,
         "metric": "cosine", "nq": 10_000, "nprobe": 32, "k": 10},
        {"name": "search_10k_d200", "kind": "search", "data": "shifted", "n": 10_000_000, "d": 200, "nlist": 4096, "bits": 4, "sign": False,
         "metric": "cosine", "nq": 10_000, "nprobe": 64, "k": 100},
        # nearest by distance of raw vectors, dimension and counts that are no multiples of anything
        {"name": "search_l2", "kind": "search", "data": "iso", "n": 1_000_003, "d": 100, "nlist": 1000, "bits": 4, "sign": False,
         "metric": "l2", "nq": 1000, "nprobe": 16, "k": 20},
        # finer codes (sign bit), data without clusters, the 50 best re-scored on the raw rows
        {"name": "rerank_flat", "kind": "rerank", "data": "flat", "n": 1_000_000, "d": 128, "nlist": 1024, "bits": 4, "sign": True,
         "metric": "cosine", "nq": 4096, "nprobe": 32, "k": 10, "keep": 50},
        # rows encoded for someone else to store (another shard, a file)
        {"name": "encode_rows", "kind": "encode", "data": "shifted", "n": 262_147, "d": 200, "nlist": 4096, "bits": 4, "sign": False},
        # a small collection built and searched from nothing: the tiny configuration whole
        {"name": "build_tiny", "kind": "build", "data": "iso", "n": 20_000, "d": 64, "nlist": 64, "bits": 4, "sign": False,
         "metric": "cosine", "nq": 200, "nprobe": 8, "k": 10},
        # a large one: the benchmark's step
        {"name": "build_10m", "kind": "build", "data": "aniso", "n": 10_000_000, "d": 96, "nlist": 4096, "bits": 4, "sign": False,
         "metric": "cosine", "nq": 10_000, "nprobe": 32, "k": 10},
        # an index read back as vectors (what the adaptive refresh of the partition starts with, and export)
        {"name": "reconstruct_1m", "kind": "reconstruct", "data": "codes", "n": 1_000_000, "d": 128, "nlist": 1024, "bits": 4, "sign": False},
        # the coarse partition trained on the benchmark's sample
        {"name": "train_500k", "kind": "train", "data": "aniso", "n": 500_000, "d": 96, "nlist": 4096, "bits": 4, "sign": False, "iters": 10},
    ]


#: Most that a drawn case may cost: floating operations of `work` and bytes of packed codes that its queries look at.
MOST_FLOPS = 8.2e12
MOST_SCANNED = 1.6e11


def draw(rng):
    while True:
        case = _draw(rng)
        w = work(case)
        scanned = case.get("nq", 0) * case.get("nprobe", 0) * (case["n"] / case["nlist"]) * _vector_bytes(case)
        # codes too wide for the matrix-core scan are read once per query: their share of the range is smaller
        if w["flops"] <= MOST_FLOPS and scanned <= (MOST_SCANNED if _stored(case) <= 5 else MOST_SCANNED / 32):
            return case


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choice(["search"] * 6 + ["rerank", "encode", "build", "build", "reconstruct", "train"])
    d = rng.choice([64, 96, 100, 128, 200, _log(rng, 32, 256), _log(rng, 32, 256)])
    bits, sign = rng.choice([(2, False), (3, False), (4, False), (4, False), (4, False), (4, True), (8, False)])
    most = {"search": 10_000_000, "build": 10_000_000, "rerank": 2_000_000, "encode": 1_000_000, "reconstruct": 2_000_000, "train": 500_000}[kind]
    n = min(_log(rng, {"encode": 500, "train": 20_000}.get(kind, 20_000), most), 2_000_000_000 // d)
    nlist = max(16, min(4096, int(rng.uniform(0.5, 1.6) * math.sqrt(max(n, 250_000 if kind == "encode" else 0)))))
    case = {"kind": kind, "data": rng.choice(["iso", "aniso", "shifted", "flat"]), "n": n, "d": d, "nlist": nlist, "bits": bits, "sign": sign}
    if kind in ("search", "rerank", "build"):
        case["metric"] = rng.choice(["cosine"] * 6 + ["ip", "l2"]) if kind == "search" else "cosine"
        case["nq"] = _log(rng, 1, 10_000)
        case["nprobe"] = min(_log(rng, 4, 128), max(4, nlist // 4))
        case["k"] = _log(rng, 1, 100)
        if kind == "rerank":
            case["k"] = min(case["k"], 20)
            case["keep"] = min(200, case["k"] * rng.choice([2, 5, 10]))
    if kind == "reconstruct":
        case["data"] = "codes"
    if kind == "train":
        case["iters"] = rng.choice([2, 5, 10])
    return case


# ---- inputs ------------------------------------------------------------------------------------------------------


def _mixture(case, g):
    """(means, widths) of the components, as many as the index has cells"""
    c, d = case["nlist"], case["d"]
    means = torch.randn((c, d), generator=g, device=DEV)
    if case["data"] == "iso":
        return means, (0.2 + 0.4 * torch.rand((c, 1), generator=g, device=DEV)).expand(c, d).contiguous()
    return means, 0.5 * torch.pow(10.0, 0.5 * (torch.rand((c, d), generator=g, device=DEV) - 0.5))


def _rows(case, n, mix, g, queries=False):
    out = torch.empty((n, case["d"]), device=DEV)
    if case["data"] == "flat":
        return out.normal_(generator=g)
    means, width = mix
    if queries and case["data"] == "shifted":       # every component moved by half its width, twice the variance
        step = torch.nn.functional.normalize(torch.randn(means.shape, generator=g, device=DEV), dim=1)
        means, width = means + 0.5 * width.mean(1, keepdim=True) * step, width * math.sqrt(2.0)
    for lo in range(0, n, 1 << 20):
        part = out[lo:lo + (1 << 20)]
        which = torch.randint(0, len(means), (len(part),), generator=g, device=DEV)
        part.normal_(generator=g).mul_(width[which]).add_(means[which])
        if case["data"] == "aniso":
            part.div_(part.norm(dim=1, keepdim=True))
    return out


def _centroids(rows, nlist, iters=3):
    """Lloyd iterations on the sphere from the first rows; integer sums, so the result does not depend on the order of additions"""
    x = torch.nn.functional.normalize(rows[:max(24 * nlist, 2000)], dim=1)
    fixed = (x * 2.0 ** 30).to(torch.int64)
    c = x[torch.arange(nlist, device=DEV) % len(x)].clone()
    for _ in range(iters):
        cell = torch.cat([(part @ c.T).argmax(1) for part in x.split(16384)])
        total = torch.zeros((nlist, x.shape[1]), dtype=torch.int64, device=DEV).index_add_(0, cell, fixed)
        mean = total.to(torch.float64)
        norm = mean.norm(dim=1, keepdim=True)
        c = torch.where(norm > 0, (mean / norm.clamp(min=1.0)).to(torch.float32), c)
    return c.cpu().numpy()


def _index(case):
    ix = pkg.Index(case["d"], case["bits"], case["nlist"], rotation_seed=7, sign_bit=case["sign"])
    if case.get("metric") in ("ip", "l2"):
        ix.set_metric(pkg.binding.METRIC_IP if case["metric"] == "ip" else pkg.binding.METRIC_L2)
    return ix


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    state = {"case": case, "index": _index(case)}
    ix, n, d, nlist = state["index"], case["n"], case["d"], case["nlist"]
    if case["kind"] == "reconstruct":
        # an index filled with codes that were made elsewhere: cells of different sizes, codes as the quantiser's input
        # is distributed (each coordinate about normal with variance 1/d)
        _, tau = ix.get_codebook()
        cell = (nlist * torch.rand(n, generator=g, device=DEV).pow(1.3)).to(torch.int32).clamp_(max=nlist - 1)
        codes = torch.empty((n, d), dtype=torch.uint8, device=DEV)
        for lo in range(0, n, 1 << 20):
            part = torch.randn((min(n - lo, 1 << 20), d), generator=g, device=DEV) / math.sqrt(d)
            codes[lo:lo + len(part)] = torch.bucketize(part, torch.from_numpy(tau).to(DEV), right=True).to(torch.uint8)
        gamma = (0.3 + 0.5 * torch.rand(n, generator=g, device=DEV)).to(torch.float16)
        ix.set_coarse(torch.nn.functional.normalize(torch.randn((nlist, d), generator=g, device=DEV), dim=1).cpu().numpy())
        ix.add_encoded(cell, codes, gamma)
        return state
    mix = None if case["data"] == "flat" else _mixture(case, g)
    if case["kind"] == "encode":         # centroids from data of the same source, not from the rows to be encoded
        ix.set_coarse(_centroids(_rows(case, max(24 * nlist, 2000), mix, g), nlist))
        state["x"] = _rows(case, n, mix, g)
        return state
    x = _rows(case, n, mix, g)
    if case["kind"] == "train":
        state["x"] = x
        state["init"] = torch.randperm(n, generator=g, device=DEV)[:nlist].cpu().numpy()
        return state
    ix.set_coarse(_centroids(x, nlist))
    state["q"] = _rows(case, case["nq"], mix, g, queries=True)
    if case["kind"] != "build":
        ix.encode_add(x)
    if case["kind"] != "search":
        state["x"] = x
    torch.cuda.synchronize()             # the rows of a search case are given back here
    return state


def run(state):
    case, ix = state["case"], state["index"]
    if case["kind"] == "search":
        return ix.search(state["q"], case["nprobe"], case["k"])
    if case["kind"] == "rerank":
        _, near = ix.search(state["q"], case["nprobe"], case["keep"])
        return pkg.ivftq_rerank(state["q"], state["x"], near, case["k"])
    if case["kind"] == "build":
        ix.reset()
        ix.encode_add(state["x"])
        return ix.search(state["q"], case["nprobe"], case["k"])
    if case["kind"] == "encode":
        return ix.encode_only(state["x"])
    if case["kind"] == "reconstruct":
        return ix.reconstruct()
    inertia = ix.train_coarse(state["x"], case["iters"], init_rows=state["init"])
    return ix.get_coarse(), inertia


# ---- what a pass cannot do without, and how far two correct passes can be apart ------------------------------------


def _stored(case):
    return case["bits"] + (1 if case["sign"] else 0)


def _vector_bytes(case):
    """packed code and float16 norm of one stored vector; the raw metrics read its length too"""
    return (_stored(case) * case["d"] + 7) // 8 + 2 + (4 if case.get("metric") in ("ip", "l2") else 0)


def work(case):
    n, d, nlist = case["n"], case["d"], case["nlist"]
    b = f = 0.0
    if case["kind"] in ("search", "rerank", "build"):
        nq, nprobe, k = case["nq"], case["nprobe"], case["k"]
        seen = n * (1.0 - (1.0 - nprobe / nlist) ** nq)                  # stored vectors that some query looks at
        b += 4.0 * nq * d + 4.0 * nlist * d + 4.0 * d * d + seen * _vector_bytes(case) + 12.0 * nq * k
        f += 2.0 * nq * nlist * d + 2.0 * nq * d * d + 2.0 * nq * nprobe * (n / nlist) * d
    if case["kind"] == "rerank":
        b += 4.0 * min(n, case["nq"] * case["keep"]) * d
        f += 4.0 * case["nq"] * case["keep"] * d
    if case["kind"] == "build":
        b += 4.0 * n * d + n * (_vector_bytes(case) + 8.0)
        f += 2.0 * n * nlist * d + 2.0 * n * d * d
    if case["kind"] == "encode":
        b += 4.0 * n * d + 4.0 * nlist * d + 4.0 * d * d + n * (d + 4.0 + 2.0)
        f += 2.0 * n * nlist * d + 2.0 * n * d * d
    if case["kind"] == "reconstruct":
        b += n * (_vector_bytes(case) + 8.0) + n * (4.0 * d + 8.0)
        f += 2.0 * n * d * d
    if case["kind"] == "train":
        b += 4.0 * n * d + 4.0 * nlist * d
        f += case["iters"] * 2.0 * n * nlist * d
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["kind"] == "encode":
        # whole values: cells and codes within float32 rounding of a decision; norms are float16
        return {"rel": 1e-3, "max": 2e-3, "differ": 1e-4}
    if case["kind"] == "reconstruct":
        return {"rel": 1e-5, "max": 1e-4}                                 # float32 sums of d products
    if case["kind"] == "train":
        # float32 sums; a row whose two nearest means tie to rounding may go to either, which moves a mean of about
        # a hundred rows by a hundredth of its spread (and a few of its neighbours' means in later iterations)
        return {"rel": 1e-3, "max": 0.3}
    # estimates in float32; a stored code within rounding of a decision may be one bin off in a few vectors of a
    # million, and results closer than rounding may change places
    return {"rel": 1e-4, "max": 1e-2, "differ": 3e-3}
