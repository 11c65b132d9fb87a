"""The calls that the speed of this library is judged by: graph builds and searches, through the public entry points.

Graph construction (rnnd_build) is what the library is for, and searching the finished graph (rnnd_search) is what
its users do with it.  Both are called here as a program calls them: X (and the queries) in device memory, outputs
allocated by the binding.  The listed cases cover the smallest calls (launches and latency), ordinary ones and the
largest; uint8, float32 and 16-bit storage; row lengths that fit the matrix tiles and row lengths that do not.

Data: synthetic, from the seed, with the value ranges and rough statistics of the workloads this repository
measures itself on (workloads.py holds the same recipes in numpy; here they are drawn on the device).
"""
import math

import torch

import paper_2310_20419_amd as rn

CHUNK = 65536      # rows drawn at a time
DTYPES = {"u8": torch.uint8, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"u8": 1, "f32": 4, "f16": 2, "bf16": 2}


def _build(name, dtype, data, N, d, S, R, T1, T2, M=0):
    return {"name": name, "op": "build", "dtype": dtype, "data": data, "N": N, "d": d, "S": S, "R": R, "M": M or R,
            "T1": T1, "T2": T2}


def _search(name, dtype, data, N, d, nq, L, K, k):
    return {"name": name, "op": "search", "dtype": dtype, "data": data, "N": N, "d": d, "nq": nq, "L": L, "K": K, "k": k}


def listed():
    return [
        # the smallest build of this repository's configurations: a few thousand short rows, few rounds
        _build("build_u8_5k_32", "u8", "gauss", 5_000, 32, 10, 32, 2, 4),
        # a mid-sized index over local image descriptors (128 bytes per row), the paper's parameters
        _build("build_u8_100k_128", "u8", "heavy", 100_000, 128, 20, 96, 4, 15),
        # the headline workload: one million local descriptors
        _build("build_u8_1m_128", "u8", "heavy", 1_000_000, 128, 20, 96, 4, 15),
        # small grey-scale images (28 x 28 bytes): long byte rows, a length no matrix tile divides
        _build("build_u8_60k_784", "u8", "heavy", 60_000, 784, 20, 96, 4, 15),
        # a small index over unit-length float features, as one rebuilds often
        _build("build_f32_20k_96", "f32", "unit", 20_000, 96, 20, 96, 4, 15),
        # one million short float descriptors
        _build("build_f32_1m_96", "f32", "unit", 1_000_000, 96, 20, 96, 4, 15),
        # word-vector-like float rows: 100 coordinates, not a multiple of 16
        _build("build_f32_200k_100", "f32", "unit", 200_000, 100, 20, 96, 4, 15),
        # the largest build: one million long float rows (global image descriptors)
        _build("build_f32_1m_960", "f32", "beta", 1_000_000, 960, 20, 96, 4, 15),
        # text-embedding-like rows stored in 16 bits
        _build("build_bf16_300k_768", "bf16", "unit", 300_000, 768, 20, 96, 4, 15),
        # offline batch search on the headline index
        _search("search_u8_1m_10k", "u8", "heavy", 1_000_000, 128, 10_000, 64, 32, 10),
        # one interactive query: latency only
        _search("search_f32_100k_1", "f32", "unit", 100_000, 96, 1, 64, 32, 10),
        # a batch of long float queries with a wide candidate list (high recall)
        _search("search_f32_300k_960", "f32", "beta", 300_000, 960, 1_000, 100, 48, 10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more build or search: sizes over the ranges of the listed ones, odd row lengths and counts among them."""
    dtype = rng.choice(["u8", "u8", "u8", "f32", "f32", "f32", "f16", "bf16"])
    N = _log_int(rng, 2_000, 1_000_000)
    d = _log_int(rng, 16, 960)
    # most rows have a length that somebody chose: a multiple of 4, 16 or 32; the rest any
    step = rng.choice([1, 4, 4, 16, 32, 32])
    d = max(16, d // step * step)
    if dtype == "u8":
        data = "gauss" if d < 48 else "heavy"
    else:
        data = "beta" if d % 32 == 0 and rng.random() < 0.4 else "unit"
    if rng.random() < 0.7:
        S = rng.choice([10, 16, 20, 20, 24])
        R = rng.choice([32, 48, 64, 96, 96, 128])
        T1, T2 = rng.choice([(2, 4), (2, 8), (3, 10), (4, 15), (4, 15)])
        M = 128 if rng.random() < 0.15 else R      # rows wider than the degree cap
        while N * (d + 64) * S * T1 > 2.4e9:       # far below the largest listed build
            N = N * 2 // 3
        c = _build("", dtype, data, N, d, S, R, T1, T2, M)
    else:
        while N * (d + 64) > 1.2e8:                # the index behind the search is built in prepare()
            N = N * 2 // 3
        L = _log_int(rng, 16, 128)
        c = _search("", dtype, data, N, d, _log_int(rng, 1, 10_000), L, rng.choice([8, 16, 32, 32, 48, 96]),
                    min(L, rng.choice([1, 10, 10, 100])))
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _gamma_half(n, d, g):
    """Gamma(1/2, scale 30): half a squared standard normal, scaled."""
    return torch.randn(n, d, device="cuda", generator=g).square_().mul_(15.0)


def _beta25(n, d, g):
    """Beta(2, 5): the second smallest of six uniform numbers."""
    a = torch.rand(n, d, device="cuda", generator=g)
    b = torch.rand(n, d, device="cuda", generator=g)
    lo, second = torch.minimum(a, b), torch.maximum(a, b)
    for _ in range(4):
        x = torch.rand(n, d, device="cuda", generator=g)
        second = torch.minimum(second, torch.maximum(lo, x))
        lo = torch.minimum(lo, x)
    return second


class _Source:
    """Rows of one mixture: the centres come from the seed, so database and queries share them."""

    def __init__(self, data, d, dtype, seed):
        self.data, self.d, self.dtype, self.g = data, d, DTYPES[dtype], _gen(seed)
        if data == "gauss":        # 16 Gaussian clusters, sigma 20, rounded to bytes
            self.c = torch.rand(16, d, device="cuda", generator=self.g) * 192.0 + 32.0
        elif data == "heavy":      # 256 clusters of sparse heavy-tailed byte features, about 40 % zeros
            on = (torch.rand(256, d, device="cuda", generator=self.g) < 0.5).float()
            self.c = (_gamma_half(256, d, self.g) + 12.0) * on
        elif data == "unit":       # 1,024 Gaussian clusters, sigma 0.5, rows scaled to unit length
            self.c = torch.randn(1024, d, device="cuda", generator=self.g)
        else:                      # 512 centres, features correlated in groups of 32, values in [0, 1]
            self.c = _beta25(512, d, self.g)

    def _chunk(self, n):
        g, d = self.g, self.d
        c = self.c[torch.randint(0, self.c.shape[0], (n,), device="cuda", generator=g)]
        if self.data == "gauss":
            return (c + 20.0 * torch.randn(n, d, device="cuda", generator=g)).round_().clamp_(0, 255)
        if self.data == "heavy":
            return (c + _gamma_half(n, d, g) - 15.0).round_().clamp_(0, 255)
        if self.data == "unit":
            x = c + 0.5 * torch.randn(n, d, device="cuda", generator=g)
            return x / x.norm(dim=1, keepdim=True)
        f = _beta25(n, (d + 31) // 32, g).repeat_interleave(32, dim=1)[:, :d]
        return 0.5 * c + 0.25 * f + 0.25 * _beta25(n, d, g)

    def rows(self, n):
        out = torch.empty(n, self.d, dtype=self.dtype, device="cuda")
        for lo in range(0, n, CHUNK):
            hi = min(n, lo + CHUNK)
            out[lo:hi] = self._chunk(hi - lo).to(self.dtype)
        return out


def prepare(case, seed):
    src = _Source(case["data"], case["d"], case["dtype"], seed)
    X = src.rows(case["N"])
    if case["op"] == "build":
        return {"case": case, "X": X, "seed": seed % 1000 + 1}
    Q = src.rows(case["nq"])
    # the finished index that a search runs on
    S = min(20, case["N"] - 1)
    graph, degree = rn.rnnd_build(X, S, 96, 4, 15, seed % 1000 + 1)
    return {"case": case, "X": X, "Q": Q, "graph": graph, "degree": degree, "seed": seed % 1000 + 7}


def run(state):
    c, X = state["case"], state["X"]
    if c["op"] == "build":
        if c["M"] > c["R"]:
            graph, degree, _, _ = rn.rnnd_build_wide(X, c["S"], c["R"], c["M"], c["T1"], c["T2"], state["seed"],
                                                     want_keys=False)
        else:
            graph, degree = rn.rnnd_build(X, c["S"], c["R"], c["T1"], c["T2"], state["seed"])
        return {"graph": graph, "degree": degree}
    ids, dist, evals = rn.rnnd_search(X, state["graph"], state["degree"], state["Q"], c["L"], c["K"], c["k"],
                                      state["seed"], want_dist=True)
    return {"ids": ids, "dist": dist if c["dtype"] == "u8" else dist.view(torch.float32), "evals": evals}


def work(case):
    """Inputs read once, outputs written once, and the distance evaluations of the method: RandomGraph makes S per
    vertex, the refinement rounds between 0.65 and 1.6 times S^2 T1 per vertex on these data (counted by
    rnnd_stats), a search about 20 per place of its candidate list; three operations per coordinate."""
    N, d, size = case["N"], case["d"], SIZE[case["dtype"]]
    if case["op"] == "build":
        evals = N * (case["S"] + case["S"] ** 2 * case["T1"])
        return {"bytes": N * d * size + N * case["M"] * 4 + N * 4, "flops": 3.0 * d * evals}
    evals = case["nq"] * min(N, 21 * case["L"])
    rows = min(N, evals)
    return {"bytes": rows * (d * size + 4) + case["nq"] * (d * size + case["k"] * 8), "flops": 3.0 * d * evals}


def tolerance(case):
    """uint8 rows: distances are whole numbers and the graph is a function of them, so nothing may differ.

    Float rows: a stored distance is a sum in double rounded once to float, and every decision is taken on such
    floats.  Two orders of summation give another float where the doubles straddle a rounding boundary, about
    once in 10^8 distances, and the graph changes only where that reverses a comparison; the builds of this
    library and of the index-order CPU oracle, which add in different orders, agree in every entry at 300,000 x 96
    and at 100,000 x 960.  Where one comparison does go the other way, the lists near that vertex differ: a few
    hundred of 10^7 to 10^8 entries."""
    if case["dtype"] == "u8":
        return "exact"
    return {"rel": 2.4e-7, "max": 2.4e-7, "differ": 1e-5}


def exact(case, seed):
    """Graphs and neighbour ids are whole numbers, and the distances of a search belong to ids that follow from the
    whole build: there is no 64-bit value to state without running the method, which plain torch cannot do in 20 s."""
    return None
