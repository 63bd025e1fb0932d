"""The work this library is used for, as measurable cases: the products of packed sparse tensors with dense operands (one
column, many columns, sampled, Khatri-Rao), the sparse-times-sparse product, and the two directions of the storage builder
(coordinates in, conversion between encodings), over the sizes, types, encodings and sparsity patterns it is used with.

A case is a dict of plain values.  `kind` is the call; `fmt` the encoding (FORMATS); `pattern` how the coordinates are
drawn; `dtype` f32 / f64; `width` the bits of pos and crd.  Everything is drawn on the GPU from the seed alone.
"""
import math

import torch

import paper_2202_04305_amd as sp

D, C = sp.SP_DENSE, sp.SP_COMPRESSED
FORMATS = {  # level types, dimension stored at each level
    "csr": ((D, C), (0, 1)), "csc": ((D, C), (1, 0)), "dcsr": ((C, C), (0, 1)), "dcsc": ((C, C), (1, 0)), "cdr": ((C, D), (0, 1)),
    "dss": ((D, C, C), (0, 1, 2)), "dss-alt": ((D, C, C), (0, 2, 1)), "csf": ((C, C, C), (0, 1, 2)), "csf-kij": ((C, C, C), (2, 0, 1)),
    "csf2": ((C, C), (0, 1)), "csf3": ((C, C, C), (0, 1, 2)), "csf4": ((C,) * 4, (0, 1, 2, 3)), "csf5": ((C,) * 5, (0, 1, 2, 3, 4)),
}
DTYPES = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # a small sparse operator applied once per step of a host loop: launches and host work are all there is
        {"name": "spmv_csr_small", "kind": "spmv", "fmt": "csr", "pattern": "per_row", "dtype": "f64", "width": 32, "m": 4096, "n": 4096, "nnz": 32768},
        # the headline: a million-row matrix with skewed row lengths times a vector (iterative solvers, graph iterations)
        {"name": "spmv_csr_powerlaw", "kind": "spmv", "fmt": "csr", "pattern": "lognormal", "dtype": "f64", "width": 32, "m": 1 << 20, "n": 1 << 20, "nnz": 16_870_001},
        # a hypersparse matrix (one row in a hundred stored) times a vector much larger than the caches
        {"name": "spmv_dcsr_hypersparse", "kind": "spmv", "fmt": "dcsr", "pattern": "hypersparse", "dtype": "f64", "width": 32, "m": 1 << 23, "n": 1 << 23, "nnz": 2_684_352},
        # the same power-law matrix times a block of vectors (block solvers, feature matrices)
        {"name": "spmm_csr_powerlaw_64", "kind": "spmm", "fmt": "csr", "pattern": "lognormal", "dtype": "f64", "width": 32, "m": 1 << 20, "n": 1 << 20, "nnz": 16_870_001, "cols": 64},
        # column-major storage, single precision, a few very popular columns (propagation of features over a graph)
        {"name": "spmm_csc_zipf_32", "kind": "spmm", "fmt": "csc", "pattern": "zipf", "dtype": "f32", "width": 32, "m": 1 << 21, "n": 1 << 21, "nnz": 33_554_392, "cols": 32},
        # nothing a power of two, the native 64-bit widths: what a user gets who tunes nothing
        {"name": "spmm_csr_ragged_33", "kind": "spmm", "fmt": "csr", "pattern": "lognormal", "dtype": "f64", "width": 64, "m": 300_007, "n": 250_013, "nnz": 5_000_011, "cols": 33},
        # sampled dense-dense product on a power-law pattern (attention scores, gradients of a factorisation)
        {"name": "sddmm_csr_powerlaw_64", "kind": "sddmm", "fmt": "csr", "pattern": "lognormal", "dtype": "f64", "width": 32, "m": 1 << 20, "n": 1 << 20, "nnz": 16_870_001, "cols": 64, "b_transposed": False},
        # the inner step of a tensor factorisation on a large rank-3 tensor
        {"name": "mttkrp_slices_42", "kind": "mttkrp", "fmt": "dss", "pattern": "slices", "dtype": "f64", "width": 32, "shape": "12092x9184x28818", "nnz": 76_879_419, "cols": 42},
        # sparse times sparse with a sparse result
        {"name": "spgemm_uniform_8192", "kind": "spgemm", "fmt": "csr", "pattern": "uniform", "dtype": "f64", "width": 32, "m": 8192, "k": 8192, "n": 8192, "nnz": 671_089, "nnz_b": 671_089},
        # the storage builder: shuffled coordinates of the power-law matrix into CSR
        {"name": "pack_csr_powerlaw", "kind": "pack", "fmt": "csr", "pattern": "lognormal", "dtype": "f64", "width": 32, "m": 1 << 20, "n": 1 << 20, "nnz": 16_870_001},
        # the storage builder on a large rank-3 tensor, every level compressed
        {"name": "pack_csf_rank3", "kind": "pack", "fmt": "csf3", "pattern": "uniform", "dtype": "f64", "width": 32, "shape": "12092x9184x28818", "nnz": 76_879_419},
        # conversion: the row-major matrix becomes a column-major one (transposition)
        {"name": "convert_csr_csc", "kind": "convert", "fmt": "csr", "to": "csc", "pattern": "lognormal", "dtype": "f64", "width": 32, "m": 1 << 20, "n": 1 << 20, "nnz": 16_870_001},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _matrix(rng, nnz_lo, nnz_hi, pattern):
    """m, n, nnz of a matrix with 2 to 64 entries per row (per stored row / column where only some are stored)."""
    nnz = _log(rng, nnz_lo, nnz_hi)
    per = _log(rng, 4, 64)
    m = max(64, nnz // per)
    n = min(1 << 23, max(512, int(m * math.exp(rng.uniform(-0.7, 0.7)))))
    if pattern == "hypersparse":
        m = min(1 << 23, m * rng.randint(20, 100))
        n = min(1 << 23, n * rng.randint(2, 20))
    if pattern == "per_row":
        nnz = m * (nnz // m)
    return m, n, min(nnz, m * n // 8)


def _sides(rng, side, rank):
    return "x".join(str(int(side * rng.uniform(0.7, 1.5)) + 2) for _ in range(rank))


def draw(rng):
    kind = rng.choice(["spmv", "spmm", "sddmm", "mttkrp", "spgemm", "pack", "convert"])
    dtype, width = rng.choice(["f64", "f64", "f32"]), rng.choice([32, 32, 64])
    case = {"kind": kind, "dtype": dtype, "width": width}
    if kind in ("spmv", "spmm"):
        fmt = rng.choice(["csr", "csr", "dcsr", "csc", "dcsc", "cdr"])
        if fmt == "cdr":                                   # the first rows full, the rest empty
            n = _log(rng, 4000, 66_000)
            rows = rng.randint(50, 1000)
            case.update(fmt=rng.choice(["cdr", "csr", "dcsr"]) if kind == "spmv" else "csr", pattern="band", m=n, n=n, rows=rows, nnz=rows * n)
            if kind == "spmm":
                case["cols"] = rng.randint(2, 16)
            return case
        pattern = {"csr": rng.choice(["lognormal", "uniform", "per_row"]), "dcsr": "hypersparse", "csc": "zipf", "dcsc": "zipf"}[fmt]
        m, n, nnz = _matrix(rng, 20_000, 16_000_000, pattern)
        case.update(fmt=fmt, pattern=pattern, m=m, n=n, nnz=nnz)
        if kind == "spmm":
            case["cols"] = rng.choice([_log(rng, 2, 128), 4 * rng.randint(1, 24), 1 << rng.randint(1, 7)])
            while case["cols"] > 8 and max(m, n) * case["cols"] > (1 << 27):
                case["cols"] //= 2
    elif kind == "sddmm":
        pattern = rng.choice(["lognormal", "uniform"])
        m, n, nnz = _matrix(rng, 20_000, 12_000_000, pattern)
        case.update(fmt=rng.choice(["csr", "dcsr"]), pattern=pattern, m=m, n=n, nnz=nnz, cols=rng.choice([_log(rng, 4, 128), 1 << rng.randint(2, 7)]),
                    b_transposed=rng.choice([False, True]))
    elif kind == "mttkrp":
        nnz = _log(rng, 30_000, 40_000_000)
        side = round(nnz ** 0.5)
        case.update(fmt=rng.choice(["dss", "dss-alt", "csf"]), pattern=rng.choice(["slices", "uniform"]), nnz=nnz, cols=_log(rng, 8, 64),
                    shape="%dx%dx%d" % (max(16, side * rng.randint(50, 200) // 100), max(256, side * rng.randint(50, 200) // 100), max(256, side * rng.randint(100, 400) // 100)))
    elif kind == "spgemm":
        if rng.random() < 0.7:                             # a row of the result fits a workspace on the chip
            n = _log(rng, 500, 9000)
            nnz = max(n, int(rng.uniform(0.003, 0.01) * n * n))
        else:
            n = _log(rng, 20_000, 300_000)
            nnz = n * rng.randint(3, 10)
        case.update(fmt=rng.choice(["csr", "csr", "dcsr"]), pattern="uniform", m=n, k=n, n=n, nnz=nnz, nnz_b=nnz)
    elif kind == "pack":
        rank = rng.choice([2, 2, 3, 4, 5])
        if rank == 2:
            pattern = rng.choice(["lognormal", "uniform", "zipf", "hypersparse"])
            m, n, nnz = _matrix(rng, 3000, 30_000_000, pattern)
            case.update(fmt=rng.choice({"zipf": ["csc", "csr"], "hypersparse": ["dcsr"]}.get(pattern, ["csr", "csf2", "csc"])), pattern=pattern, m=m, n=n, nnz=nnz)
        else:
            nnz = _log(rng, 3000, 45_000_000)
            side = max(8.0, (nnz * rng.uniform(8, 2000)) ** (1.0 / rank))
            case.update(fmt="csf%d" % rank, pattern="uniform", nnz=nnz, shape=_sides(rng, side, rank))
    else:
        if rng.random() < 0.75:
            pattern = rng.choice(["lognormal", "uniform", "zipf"])
            m, n, nnz = _matrix(rng, 10_000, 20_000_000, pattern)
            fmt, to = rng.choice([("csr", "csc"), ("csc", "csr"), ("csr", "dcsr"), ("dcsr", "dcsc")])
            case.update(fmt=fmt, to=to, pattern=pattern, m=m, n=n, nnz=nnz)
        else:
            nnz = _log(rng, 10_000, 20_000_000)
            side = (nnz * 200) ** (1 / 3)
            case.update(fmt="csf", to=rng.choice(["dss", "dss-alt", "csf-kij"]), pattern="uniform", nnz=nnz, shape=_sides(rng, side, 3))
    return case


# ---- inputs ---------------------------------------------------------------------------------
def _shape(case):
    return [int(s) for s in case["shape"].split("x")] if "shape" in case else [case["m"], case["n"]]


def _distinct(sample, nnz, g):
    """`nnz` distinct keys; sample(k) draws about k."""
    keys = torch.unique(sample(nnz + nnz // 64 + 64))
    while keys.numel() < nnz:
        keys = torch.unique(torch.cat([keys, sample(2 * (nnz - keys.numel()) + 64)]))
    return keys[torch.randperm(keys.numel(), generator=g, device="cuda")[:nnz]]


def _coordinates(pattern, shape, nnz, seeded, rows=0, structure=1, perms=None):
    """Distinct coordinates in a random order, one int64 tensor per dimension.  How many entries share a row, a fibre and so
    on is drawn once per case; the seed then renames the coordinates of every dimension (perms, where the caller has them)
    and shuffles the entries, so that other inputs give other arrays of the same lengths."""
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(structure)
    total = math.prod(shape)

    def ints(high, k):
        return torch.randint(high, (k,), generator=g, device=dev)

    def spread(weights, k, cap):                           # segment ids whose counts follow the weights, each once at least
        lens = (weights * (k / float(weights.sum()))).round().clamp(1, cap).long()
        return torch.repeat_interleave(torch.arange(lens.numel(), device=dev), lens)

    if pattern == "band":
        keys = torch.arange(rows * shape[1], device=dev)
    elif pattern == "uniform":
        keys = _distinct(lambda k: ints(total, k), nnz, g)
    elif pattern == "per_row":                             # as many entries in every row, one per stretch of columns
        m, n = shape
        per = nnz // m
        r = torch.arange(nnz, device=dev)
        width = n // per
        keys = (r // per) * n + (r % per) * width + ints(width, nnz)
    elif pattern == "lognormal":                           # row lengths lognormal with sigma 1.5
        m, n = shape
        w = torch.exp(1.5 * torch.randn(m, generator=g, device=dev, dtype=torch.float64))

        def sample(k):
            seg = spread(w, k, max(1, min(20000, n // 2)))
            return seg * n + ints(n, seg.numel())
        keys = _distinct(sample, nnz, g)
    elif pattern == "zipf":                                # column lengths follow a rank-size law, capped
        m, n = shape
        r = torch.arange(1, n + 1, device=dev, dtype=torch.float64) ** -1.2
        cap = max(1, min(50000, m // 2))
        lo, hi = 0.0, 64.0 * nnz + 64.0
        for _ in range(50):
            c = 0.5 * (lo + hi)
            lo, hi = (c, hi) if float((r * c).clamp(max=cap).sum()) < nnz * 1.02 else (lo, c)
        w = (r * hi).clamp(max=cap)
        w = w[torch.randperm(n, generator=g, device=dev)]

        def sample(k):
            cdf = torch.cumsum(w, 0)
            seg = torch.searchsorted(cdf, torch.rand(k, generator=g, device=dev, dtype=torch.float64) * float(cdf[-1])).clamp(max=n - 1)
            return ints(m, k) * n + seg
        keys = _distinct(sample, nnz, g)
    elif pattern == "hypersparse":                         # a few rows stored, 32 entries each
        m, n = shape
        live = torch.randperm(m, generator=g, device=dev)[: max(1, min(m, nnz // 32))]

        def sample(k):
            seg = live[torch.arange(k, device=dev) % live.numel()]
            return seg * n + ints(n, k)
        keys = _distinct(sample, nnz, g)
    else:                                                  # slices: slice i samples a grid of a_i x b_i coordinates of the other two dimensions
        I, K, L = shape
        a = (500.0 / math.exp(0.5) * torch.exp(torch.randn(I, generator=g, device=dev, dtype=torch.float64))).round().clamp(2, max(2, K // 2)).long()
        b = (1500.0 / math.exp(0.5) * torch.exp(torch.randn(I, generator=g, device=dev, dtype=torch.float64))).round().clamp(2, max(2, L // 2)).long()
        kpool, lpool = ints(K, int(a.sum())), ints(L, int(b.sum()))
        koff, loff = torch.cumsum(a, 0) - a, torch.cumsum(b, 0) - b
        cells = (a * b).double()

        def sample(k):
            s = spread(cells, k, 1 << 62)
            u = torch.rand(s.numel(), generator=g, device=dev)
            i = kpool[koff[s] + torch.minimum((u * a[s]).long(), a[s] - 1)]
            u = torch.rand(s.numel(), generator=g, device=dev)
            j = lpool[loff[s] + torch.minimum((u * b[s]).long(), b[s] - 1)]
            return (s * K + i) * L + j
        keys = _distinct(sample, nnz, g)
    keys = keys[torch.randperm(keys.numel(), generator=seeded, device=dev)]
    coords = []
    for size in reversed(shape[1:]):
        coords.append(keys % size)
        keys = keys // size
    coords = [keys] + coords[::-1]
    if pattern == "band":
        return coords
    perms = perms or [torch.randperm(size, generator=seeded, device=dev) for size in shape]
    return [p[c] for p, c in zip(perms, coords)]


def _uniform(shape, dtype, g):
    return torch.rand(shape, generator=g, device="cuda", dtype=dtype).mul_(2).sub_(1)


def _encoding(fmt, width):
    levels, order = FORMATS[fmt]
    return sp.sp_encode(levels, order, width, width)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind, dtype, width, shape = case["kind"], DTYPES[case["dtype"]], case["width"], _shape(case)
    a_shape = [case["m"], case["k"]] if kind == "spgemm" else shape
    perms = None
    if kind == "spgemm":                                   # rows of A, the shared dimension, columns of B
        perms = [torch.randperm(case[d], generator=g, device="cuda") for d in ("m", "k", "n")]
    coords = _coordinates(case["pattern"], a_shape, case["nnz"], g, case.get("rows", 0), perms=perms and perms[:2])
    values = _uniform((case["nnz"],), dtype, g)
    enc = _encoding(case["fmt"], width)
    state = {"kind": kind, "enc": enc}
    if kind == "pack":
        state.update(shape=shape, coords=coords, values=values)
        return state
    A = state["A"] = sp.sp_pack(enc, a_shape, coords, values)
    del coords, values
    if kind in ("spmv", "spmm"):
        cols = () if kind == "spmv" else (case["cols"],)
        state["B"] = _uniform((case["n"],) + cols, dtype, g)
        state["C"] = torch.empty((case["m"],) + cols, dtype=dtype, device="cuda")
        sp.sp_prepare(A, case.get("cols", 1))
    elif kind == "sddmm":
        K = case["cols"]
        state["tr"] = case["b_transposed"]
        state["B"] = _uniform((case["m"], K), dtype, g)
        state["D"] = _uniform((case["n"], K) if state["tr"] else (K, case["n"]), dtype, g)
        state["X"] = torch.empty(case["nnz"], dtype=dtype, device="cuda")
    elif kind == "mttkrp":
        state["B"], state["D"] = _uniform((shape[1], case["cols"]), dtype, g), _uniform((shape[2], case["cols"]), dtype, g)
        state["C"] = torch.empty((shape[0], case["cols"]), dtype=dtype, device="cuda")
    elif kind == "spgemm":
        kn = [case["k"], case["n"]]
        encb = _encoding("csr", width)
        state["B"] = sp.sp_pack(encb, kn, _coordinates(case["pattern"], kn, case["nnz_b"], g, structure=2, perms=perms[1:]), _uniform((case["nnz_b"],), dtype, g))
        state["enc"] = encb
    else:
        state["enc"] = _encoding(case["to"], width)
    torch.cuda.synchronize()
    return state


def _arrays(T, levels):
    """pos and crd of the compressed levels, and the values, of a packed tensor."""
    out = []
    for l in levels:
        out += [sp.sp_pos(T, l), sp.sp_crd(T, l)]
    return out + [sp.sp_values(T)]


def _compressed(enc_levels):
    return [l for l, t in enumerate(enc_levels) if t == C]


def run(state):
    kind = state["kind"]
    if kind in ("spmv", "spmm"):
        return sp.sp_matmul(state["A"], state["B"], state["C"])
    if kind == "sddmm":
        return sp.sp_sddmm(state["A"], state["B"], state["D"], X=state["X"], b_is_transposed=state["tr"])
    if kind == "mttkrp":
        return sp.sp_mttkrp(state["A"], state["B"], state["D"], A=state["C"])
    if kind == "pack":
        T = sp.sp_pack(state["enc"], state["shape"], state["coords"], state["values"])
    elif kind == "spgemm":
        T = sp.sp_spgemm(state["A"], state["B"], state["enc"])
    else:
        T = sp.sp_convert(state["A"], state["enc"])
    info = sp.sp_tensor_info(T)
    return _arrays(T, _compressed(list(info.levelTypes)[: info.rank]))


# ---- what a pass cannot do without -------------------------------------------------------------
def _storage(fmt, shape, nnz, case):
    """Bytes of pos, crd and values of a tensor stored under fmt (positions of outer compressed levels as for uniform draws)."""
    levels, order = FORMATS[fmt]
    w, v = case["width"] // 8, 8 if case["dtype"] == "f64" else 4
    total, positions, cells = 0.0, 1.0, 1.0
    for l, t in enumerate(levels):
        size = shape[order[l]]
        cells *= size
        if t == D:
            positions *= size
            continue
        inner = l == len(levels) - 1
        child = nnz if inner else min(nnz, cells * -math.expm1(-nnz / cells))
        if case["pattern"] == "hypersparse" and l == 0:
            child = max(1, min(size, nnz // 32)) if order[0] == 0 else child
        if case["pattern"] == "band" and l == 0:
            child = case["rows"]
        total += (positions + 1) * w + child * w
        positions = child
    return total + positions * v


def work(case):
    kind, nnz, shape = case["kind"], case["nnz"], _shape(case)
    v = 8 if case["dtype"] == "f64" else 4
    cols = case.get("cols", 1)
    if kind == "pack":
        return {"bytes": nnz * (8 * len(shape) + v) + _storage(case["fmt"], shape, nnz, case), "flops": 0}
    if kind == "convert":
        return {"bytes": _storage(case["fmt"], shape, nnz, case) + _storage(case["to"], shape, nnz, case), "flops": 0}
    if kind == "spgemm":
        m, k, n = case["m"], case["k"], case["n"]
        pairs = nnz * case["nnz_b"] / k
        nnz_c = m * n * -math.expm1(-pairs / (m * n))
        b = _storage(case["fmt"], [m, k], nnz, case) + _storage("csr", [k, n], case["nnz_b"], case) + _storage("csr", [m, n], nnz_c, case)
        return {"bytes": b, "flops": 2 * pairs}
    a = _storage(case["fmt"], shape, nnz, case)
    if kind == "mttkrp":
        return {"bytes": a + sum(shape) * cols * v, "flops": 3 * nnz * cols}
    if kind == "sddmm":
        return {"bytes": a + (min(shape[0], nnz) + min(shape[1], nnz)) * cols * v + nnz * v, "flops": 2 * nnz * cols}
    return {"bytes": a + (min(case["n"], nnz) + case["m"]) * cols * v, "flops": 2 * nnz * cols}


def tolerance(case):
    """pos, crd and moved values are the same bits.  Sums: about four times the largest differences seen between two summation
    orders of the same product, and between f32 and f64 on the same inputs, over the listed cases (f64: 4.1e-16 and 6e-14 for
    single elements, where long sums cancel; f32: 2.1e-7 and 2.5e-5)."""
    if case["kind"] in ("pack", "convert"):
        return "exact"
    return {"rel": 1.7e-15, "max": 2.5e-13} if case["dtype"] == "f64" else {"rel": 8e-7, "max": 1e-4}
