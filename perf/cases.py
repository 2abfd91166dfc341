"""The work that a user of this framework has it do, as cases that can be timed.

Every case goes through the public classes of ``paper_2307_05740_amd.binding``: ``ArrowSpMM`` (the
product ``Y = A X``, the chained product ``A^l X``, the sampled product ``S = A .* (U V^T)``) and
``Csf3Mttkrp`` (the order-3 product of a sparse tensor with two factor matrices).  A handle with its
image, workspace and entry map is made once per operand and kept, as a program that multiplies by
the same operand again and again does; the dense inputs and outputs are the caller's tensors.

The operands are those of the named workloads (``synth.make_config``, ``synth.make_tensor_config``)
and of the tests, over their range of sizes: R-MAT and Chung-Lu graphs, the five-point grid,
operands with dense diagonal blocks, uniform and skewed order-3 tensors.  They are generated on the
GPU and handed over as host arrays, which is what the framework takes.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2307_05740_amd import binding

DEV = "cuda:0"


# ------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------
def _graph(op, kind, n, deg, k, b, l=1, directed=False, values="uniform"):
    """`deg` samples per vertex (each gives two entries of an undirected graph)."""
    return {"op": op, "kind": kind, "n": n, "deg": deg, "k": k, "b": b, "l": l, "directed": directed, "values": values}


def _tensor(kind, i, j, k, samples, R):
    return {"op": "mttkrp", "kind": kind, "I": i, "J": j, "K": k, "samples": samples, "R": R}


def listed():
    c = []

    def add(name, case):
        c.append(dict(case, name=name))

    # a product on a small graph, as in a serving loop or an iterative solver: a few microseconds
    # of work, where launches and the call itself count
    add("spmm rmat 4k k16", _graph("spmm", "rmat", 4096, 16, 16, 512))
    # a stencil operator on a 1024 x 1024 grid times a block of 32 vectors (block Krylov, multigrid):
    # three or four neighbours per row, all streaming
    add("spmm grid 1024 k32", _graph("spmm", "grid", 1024 * 1024, 0, 32, 65536))
    # one propagation step of features over a social-network-like graph: the headline workload
    add("spmm rmat 8m k128", _graph("spmm", "rmat", 1 << 23, 16, 128, 262144))
    # the same on a directed graph whose vertex count and feature width are no powers of two
    add("spmm directed 300k k50", _graph("spmm", "rmat", 300007, 24, 50, 20000, directed=True))
    # communities: dense diagonal blocks and a few hubs, wide features
    add("spmm blocks 256k k128", _graph("spmm", "blocks", 262144, 48, 128, 512))
    # three steps of a random walk over a mid-size graph (row-stochastic values)
    add("A^3 rmat 1m k64", _graph("iter", "rmat", 1 << 20, 8, 64, 65536, l=3, values="rows"))
    # five steps over a hub-heavy power-law graph with few columns
    add("A^5 chunglu 2m k32", _graph("iter", "chunglu", 1 << 21, 10, 32, 65536, l=5, values="rows"))
    # edge scores of a graph (attention, matrix completion): the gradient-side counterpart of the product
    add("sddmm rmat 1m k128", _graph("sddmm", "rmat", 1 << 20, 16, 128, 65536))
    # the same for a small graph with few features
    add("sddmm rmat 30k k24", _graph("sddmm", "rmat", 30011, 12, 24, 2048))
    # one mode of an alternating-least-squares sweep: uniform tensor of the paper's density
    add("mttkrp uniform 4096 R64", _tensor("uniform", 4096, 4096, 4096, 68719477, 64))
    # real multi-way data: hub slices, fibres of one entry, most slices nearly empty
    add("mttkrp skewed 512k R32", _tensor("skewed", 1 << 19, 1 << 16, 1 << 16, 16 << 20, 32))
    # a small tensor with an odd rank
    add("mttkrp uniform 250 R25", _tensor("uniform", 250, 231, 307, 17730, 25))
    return c


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def columns():     # usual feature widths, or any number of columns
        return rng.choice((8, 16, 32, 64, 96, 128, 256)) if rng.random() < 0.5 else logint(5, 200)

    op = rng.choice(("spmm", "spmm", "spmm", "iter", "sddmm", "mttkrp"))
    k = columns()
    if op == "mttkrp":
        if rng.random() < 0.5:
            dims = [logint(128, 4096) for _ in range(3)]
            return _tensor("uniform", *dims, max(1000, round(1e-3 * dims[0] * dims[1] * dims[2])), min(k, 128))
        i = logint(2000, 1 << 19)
        return _tensor("skewed", i, i // rng.randint(5, 12), i // rng.randint(5, 12), 32 * i, min(k, 128))
    kind = rng.choice(("rmat", "rmat", "rmat", "chunglu", "grid", "blocks"))
    l = rng.randint(2, 5) if op == "iter" else 1
    deg = {"rmat": rng.randint(6, 16), "chunglu": rng.randint(6, 12), "grid": 0, "blocks": rng.randint(24, 64)}[kind]
    # no more entries, elements of X or multiplications than the largest listed case has
    per_row = {"grid": 5, "blocks": deg}.get(kind, 2 * deg)
    top = min(1 << 23, (1 << 28) // per_row, (1 << 30) // k, (1 << 35) // (per_row * k * l), (1 << 22) if kind != "rmat" else 1 << 23)
    n = logint(2000, top)
    if kind == "grid":
        n = math.isqrt(n) ** 2
    if kind == "blocks":
        return _graph(op, kind, n, deg, k, min(512, n // 2), l, values="rows" if l > 1 else "uniform")
    return _graph(op, kind, n, deg, k, max(256, n // rng.choice((8, 16, 32))), l,
                  directed=kind == "rmat" and rng.random() < 0.25, values="rows" if l > 1 else "uniform")


# ------------------------------------------------------------------------------------------------
# operands
# ------------------------------------------------------------------------------------------------
def _rmat_ends(n, m, g):
    """m edges by the recursive quadrant walk (0.57, 0.19, 0.19, 0.05); vertex ids of the next power
    of two are scaled down to n."""
    scale = max(1, (n - 1).bit_length())
    u = torch.zeros(m, dtype=torch.int64, device=DEV)
    v = torch.zeros(m, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        r = torch.rand(m, device=DEV, generator=g)
        u.mul_(2).add_(r >= 0.76)
        v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    if n != 1 << scale:
        u, v = u * n >> scale, v * n >> scale
    return u, v


def _chunglu_weights(n, deg):
    """Expected degrees of mean 2 deg falling as id^(-1/1.1) (exponent 2.1), clipped at min(1e6, n / 4)."""
    w = torch.arange(1, n + 1, dtype=torch.float64, device=DEV).pow_(-1.0 / 1.1)
    w *= 2.0 * deg * n / w.sum()
    w.clamp_(max=min(1e6, n / 4))
    return w


def _chunglu_ends(n, m, deg, g):
    cum = _chunglu_weights(n, deg).cumsum(0)
    t = torch.rand(2 * m, dtype=torch.float64, device=DEV, generator=g) * cum[-1]
    return torch.searchsorted(cum, t).clamp_(max=n - 1).split(m)


def _grid_ends(n):
    side = math.isqrt(n)
    i = torch.arange(n, device=DEV)
    x, y = i % side, i // side
    src, dst = [i], [i]
    for ok, step in ((x > 0, -1), (x < side - 1, 1), (y > 0, -side), (y < side - 1, side)):
        src.append(i[ok])
        dst.append(i[ok] + step)
    return torch.cat(src), torch.cat(dst)


def _blocks_ends(n, deg, b, g):
    """`deg` columns per row inside the row's block of b, and two among 64 hubs."""
    i = torch.arange(n, device=DEV).repeat_interleave(deg + 2)
    r = torch.rand(i.numel(), device=DEV, generator=g).view(n, deg + 2)
    lo = (torch.arange(n, device=DEV) // b * b)[:, None]
    inside = lo + (r[:, :deg] * torch.clamp(n - lo, max=b)).long()
    return i, torch.cat([inside.clamp_(max=n - 1), (r[:, deg:] * 64).long()], 1).view(-1)


def _distinct(key):
    key = torch.sort(key)[0]
    return key[torch.cat([torch.ones(1, dtype=torch.bool, device=DEV), key[1:] != key[:-1]])]


def _csr(case, seed):
    n, kind = case["n"], case["kind"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    if kind == "grid":
        u, v = _grid_ends(n)
    elif kind == "blocks":
        u, v = _blocks_ends(n, case["deg"], case["b"], g)
    else:
        m = n * case["deg"]
        u, v = _rmat_ends(n, m, g) if kind == "rmat" else _chunglu_ends(n, m, case["deg"], g)
    both = kind in ("rmat", "chunglu") and not case["directed"]
    key = _distinct(torch.minimum(u, v) * n + torch.maximum(u, v) if both else u * n + v)
    del u, v
    if case["op"] == "sddmm" and kind != "grid":
        # the result has one element per stored entry: the same number of them whatever the seed
        if both:
            key = key[key // n != key % n]
        want = _sampled_nnz(case) // (2 if both else 1)
        assert key.numel() >= want
        key = torch.sort(key[torch.randperm(key.numel(), device=DEV, generator=g)[:want]])[0]
    if both:
        row, col = key // n, key % n
        key = torch.sort(torch.cat([key, (col * n + row)[row != col]]))[0]
        del row, col
    row = key // n
    col = (key - row * n).to(torch.int32)
    del key
    count = torch.bincount(row, minlength=n)
    if kind == "grid":
        vals = torch.where(row == col, 4.0, -1.0)
    elif case["values"] == "rows":
        vals = (1.0 / count)[row]
    else:
        vals = torch.rand(row.numel(), device=DEV, generator=g) * 2.0 - 1.0
    rowptr = np.zeros(n + 1, np.int64)
    rowptr[1:] = count.cumsum(0).cpu().numpy()
    return rowptr, col.cpu().numpy(), vals.to(torch.float32).cpu().numpy()


def _coo(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    skew = (3.0, 2.0, 1.5) if case["kind"] == "skewed" else (1.0, 1.0, 1.0)
    key = torch.zeros(case["samples"], dtype=torch.int64, device=DEV)
    for d, a in zip((case["I"], case["J"], case["K"]), skew):
        u = torch.rand(case["samples"], dtype=torch.float64, device=DEV, generator=g)
        key = (key << 20) | (d * u ** a).long().clamp_(max=d - 1)
    key = _distinct(key)
    vals = torch.rand(key.numel(), device=DEV, generator=g) * 2.0 - 1.0
    mask = (1 << 20) - 1
    return [t.to(torch.int32).cpu().numpy() for t in (key >> 40, (key >> 20) & mask, key & mask)] + [vals.cpu().numpy()]


# ------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------
def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed + 1)

    def normal(rows, cols):
        return torch.randn((rows, cols), device=DEV, generator=g)

    op = case["op"]
    if op == "mttkrp":
        h = binding.Csf3Mttkrp((case["I"], case["J"], case["K"]), *_coo(case, seed), device=DEV)
        A = torch.empty((case["I"], case["R"]), device=DEV)
        return {"op": op, "h": h, "B": normal(case["J"], case["R"]), "C": normal(case["K"], case["R"]), "A": A}
    h = binding.ArrowSpMM(*_csr(case, seed), case["b"], device=DEV)
    X = normal(case["n"], case["k"])
    if op == "sddmm":
        S = torch.empty(h.info["nnz"], device=DEV)
        return {"op": op, "h": h, "U": X, "V": normal(case["n"], case["k"]), "S": S}
    return {"op": op, "h": h, "X": X, "Y": torch.empty_like(X), "l": case["l"]}


def run(s):
    op, h = s["op"], s["h"]
    if op == "spmm":
        return h.spmm(s["X"], s["Y"])
    if op == "iter":                   # in place, so the start vectors are copied first
        s["Y"].copy_(s["X"])
        return h.spmm_iter(s["Y"], s["l"])
    if op == "sddmm":
        return h.sddmm(s["U"], s["V"], s["S"])
    return h.mttkrp(s["B"], s["C"], s["A"])


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------
def _expected_nnz(case):
    """Entries left after duplicates are merged: vertices are binned by how often an end of a sample
    falls on them, ends are taken as independent (for R-MAT they nearly are)."""
    n, deg = case["n"], case["deg"]
    if case["kind"] == "grid":
        return 5 * n - 4 * math.isqrt(n)
    if case["kind"] == "blocks":
        b = case["b"]
        return n * (b * (1.0 - math.exp(-deg / b)) + 2.0)
    m = n * deg
    if case["kind"] == "rmat":
        s = max(1, (n - 1).bit_length())
        ones = np.arange(s + 1)
        shrink = n / 2.0 ** s              # ids of the next power of two are scaled down to n
        count = np.array([float(math.comb(s, int(i))) for i in ones]) * shrink
        p = 0.76 ** (s - ones) * 0.24 ** ones / shrink
    else:
        edges = np.unique(np.geomspace(1, n + 1, 200).astype(np.int64))
        count = np.diff(edges).astype(np.float64)
        w = ((edges[:-1] + edges[1:] - 1) / 2.0) ** (-1.0 / 1.1)
        w = np.minimum(w * 2.0 * deg * n / (w * count).sum(), min(1e6, n / 4))
        p = w / (w * count).sum()
    both = 1.0 if case["directed"] else 2.0
    return float((np.outer(count, count) * -np.expm1(-both * m * np.outer(p, p))).sum())


def _sampled_nnz(case):
    """Entries of a sampled product's operand: a little under what the samples give."""
    return int(_expected_nnz(case) * 0.46) * 2


def work(case):
    if case["op"] == "mttkrp":
        I, J, K, m, R = (case[x] for x in ("I", "J", "K", "samples", "R"))
        nnz, fibres = float(m), float(m)       # skewed: nearly every entry is a fibre of its own
        if case["kind"] == "uniform":
            cells = float(I) * J * K
            nnz = -cells * math.expm1(-m / cells)
            fibres = -float(I) * J * math.expm1(-m / (float(I) * J))
        return {"bytes": 8.0 * nnz + 8.0 * fibres + 4.0 * R * (I + J + K), "flops": 2.0 * R * (nnz + fibres)}
    nnz, n, k, l = _expected_nnz(case), case["n"], case["k"], case["l"]
    if case["op"] == "sddmm" and case["kind"] != "grid":
        nnz = _sampled_nnz(case)
    entry = 12.0 if case["op"] == "sddmm" else 8.0      # column and value; and the result of a sampled entry
    return {"bytes": l * (entry * nnz + 4.0 * n + 8.0 * n * k), "flops": 2.0 * nnz * k * l}


def tolerance(case):
    """fp32 sums of up to some 10^5 terms in any fixed order."""
    return {"rel": 1e-5, "max": 4e-4}
