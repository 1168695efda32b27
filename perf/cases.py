"""The calls that a program makes of this library, over its range of sizes.

A case names an entry point, the modulus set, the quantiser, the product's
sizes and the spread s of its inputs, (U(0,1) - 0.5) exp(s N(0,1)) in float64
as in ``workloads``.  ``pad`` adds columns to every leading dimension (a block
of a larger matrix).  Entry points:

    dgemm     ozaki25_dgemm: the result and the workspace allocated per call
    ex        ozaki25_dgemm_ex with the caller's C and workspace
    sub       ozaki25_dgemm_ex, C <- C - A B in place
    noalloc   ozaki25_dgemm_noalloc, the library's own static workspace
    planes    A's planes kept; B deconstructed, then ozaki25_dgemm_planes
    accurate  ozaki25_dgemm_accurate with the caller's workspace
"""
import math

import torch

import paper_2609_09095_amd as oz

SETS = {"s12": oz.S12, "a15": oz.A15}
QUANTS = {"rn": oz.RN, "tz": oz.TZ}


def _case(name, entry, set_, m, n, k, s=1.0, quant="rn", pad=0):
    c = {"entry": entry, "set": set_, "quant": quant, "m": m, "n": n, "k": k, "s": s, "pad": pad}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small block through the plainest call: what a call costs
        _case("tiny_64", "dgemm", "s12", 64, 64, 64, 0.5),
        # small, every size odd, a block of a larger matrix, on the byte moduli
        _case("small_odd", "dgemm", "a15", 201, 333, 157, 1.0, pad=3),
        # a tile of a blocked factorisation, no allocation allowed
        _case("block_512", "noalloc", "s12", 512, 512, 512),
        # few outputs, a long reduction (Gram matrices, projections)
        _case("reach_256x8192", "ex", "s12", 256, 256, 8192, 0.5),
        # ordinary squares
        _case("square_1024", "noalloc", "s12", 1024, 1024, 1024),
        # ordinary and ragged: sizes just past tile edges, truncating quantiser
        _case("mid_ragged", "ex", "a15", 1537, 2049, 1031, 2.0, quant="tz"),
        # per-vector shifts from the magnitude bound
        _case("accurate_4096", "accurate", "s12", 4096, 4096, 4096, 2.0),
        # a fixed operator against blocks of new vectors, planes kept
        _case("planes_8192x96", "planes", "s12", 8192, 96, 8192),
        # block-Krylov: tall A against one block of vectors
        _case("krylov_262144x128", "ex", "s12", 262144, 128, 4096),
        # the large square
        _case("square_8192", "ex", "s12", 8192, 8192, 8192),
        # the large ragged product on the byte moduli
        _case("ragged_8191", "ex", "a15", 8191, 8209, 7937, 2.0),
        # trailing update of a blocked LU factorisation
        _case("update_32768x1024", "sub", "s12", 32768, 32768, 1024),
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi]; one in three a multiple
    of 64, the others as they come (odd ones among them)."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 1 / 3 and v >= 64:
        v = v // 64 * 64
    return max(lo, min(hi, v))


def draw(rng):
    set_ = rng.choice(["s12", "s12", "a15"])
    quant = rng.choice(["rn", "rn", "tz"])
    s = rng.choice([0.5, 1.0, 2.0])
    pad = rng.choice([0, 0, 1, 4])
    kind = rng.choice(["small", "middle", "square", "long", "tall", "update", "planes"])
    if kind == "small":
        m, n, k = (_size(rng, 16, 512) for _ in range(3))
        entry = rng.choice(["dgemm", "noalloc"])
    elif kind == "middle":
        m, n, k = (_size(rng, 256, 3072) for _ in range(3))
        entry = rng.choice(["dgemm", "ex", "accurate"])
    elif kind == "square":
        m, n, k = (_size(rng, 2048, 8192) for _ in range(3))
        entry = rng.choice(["ex", "accurate"])
    elif kind == "long":
        m, n, k = _size(rng, 16, 512), _size(rng, 16, 512), _size(rng, 2048, 32768)
        entry = "ex"
    elif kind == "tall":
        m, n, k = _size(rng, 1024, 262144), _size(rng, 8, 128), _size(rng, 256, 4096)
        entry = rng.choice(["ex", "accurate"])
    elif kind == "update":
        m, n, k = _size(rng, 1024, 32768), _size(rng, 1024, 32768), _size(rng, 128, 1024)
        entry = "sub"
    else:
        m, n, k = _size(rng, 1024, 16384), _size(rng, 8, 512), _size(rng, 1024, 8192)
        entry = "planes"
    if entry == "dgemm":  # the plain call takes the default quantiser
        quant = "rn"
    return _case(None, entry, set_, m, n, k, s, quant, pad)


def _matrix(rows, cols, s, pad, gen):
    """(U - 0.5) exp(s N), a view with `pad` columns more per row."""
    full = torch.empty((rows, cols + pad), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // max(1, cols + pad))
    for r in range(0, rows, step):
        part = full[r:r + step]
        part.uniform_(-0.5, 0.5, generator=gen)
        spread = torch.empty_like(part).normal_(0.0, s, generator=gen)
        part.mul_(spread.exp_())
    return full[:, :cols]


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    m, n, k, s, pad = (case[x] for x in ("m", "n", "k", "s", "pad"))
    A = _matrix(m, k, s, pad, gen)
    B = _matrix(k, n, s, pad, gen)
    C = _matrix(m, n, s, pad, gen) if case["entry"] == "sub" else None
    return A, B, C


def prepare(case, seed):
    A, B, C = _inputs(case, seed)
    m, n, k, pad = (case[x] for x in ("m", "n", "k", "pad"))
    entry, set_, quant = case["entry"], SETS[case["set"]], QUANTS[case["quant"]]
    st = {"entry": entry, "set": set_, "quant": quant, "k": k, "B": B}
    if C is None and entry != "dgemm":
        C = torch.empty((m, n + pad), dtype=torch.float64, device="cuda")[:, :n]
    st["C"] = C
    nbytes = 0
    if entry == "planes":
        st["planesA"], st["expsA"] = oz.ozaki25_deconstruct(0, A, set=set_, quantiser=quant)
        kb = oz.ozaki25_k_pad(k) // oz.K_ALIGN
        st["planesB"] = torch.empty((kb, oz.ozaki25_num_planes(set_), n, oz.K_ALIGN), dtype=torch.uint8,
                                    device="cuda")
        st["expsB"] = torch.empty((n,), dtype=torch.int32, device="cuda")
        nbytes = oz.ozaki25_dgemm_planes_workspace_size(m, n, k, set_)
    else:
        st["A"] = A
        if entry in ("ex", "sub"):
            nbytes = oz.ozaki25_dgemm_workspace_size(m, n, k, set_)
        elif entry == "accurate":
            nbytes = oz.ozaki25_dgemm_accurate_workspace_size(m, n, k, set_)
    if nbytes:
        st["workspace"] = torch.empty((nbytes,), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    entry, set_, quant = st["entry"], st["set"], st["quant"]
    if entry == "dgemm":
        return oz.ozaki25_dgemm(st["A"], st["B"], set=set_)
    if entry == "noalloc":
        return oz.ozaki25_dgemm_noalloc(st["A"], st["B"], st["C"], set=set_, quantiser=quant)
    if entry in ("ex", "sub"):
        return oz.ozaki25_dgemm_ex(st["A"], st["B"], st["C"], subtract=entry == "sub",
                                   workspace=st["workspace"], set=set_, quantiser=quant)
    if entry == "accurate":
        return oz.ozaki25_dgemm_accurate(st["A"], st["B"], st["C"], workspace=st["workspace"], set=set_,
                                         quantiser=quant)
    oz.ozaki25_deconstruct(1, st["B"], st["planesB"], st["expsB"], set=set_, quantiser=quant)
    C = oz.ozaki25_dgemm_planes(st["k"], st["planesA"], st["expsA"], st["planesB"], st["expsB"], st["C"],
                                workspace=st["workspace"], set=set_)
    return {"C": C, "planesB": st["planesB"], "expsB": st["expsB"]}


def work(case):
    """Each FP64 input read and each output written once, and one product of
    m n k multiply-adds on the matrix cores for every modulus of the set.
    Stored planes: A as one byte per modulus (its planes' least size), B's
    planes written."""
    m, n, k = case["m"], case["n"], case["k"]
    r = oz.ozaki25_num_moduli(SETS[case["set"]])
    if case["entry"] == "planes":
        nbytes = r * m * k + 8 * k * n + oz.ozaki25_num_planes(SETS[case["set"]]) * k * n + 8 * m * n
    else:
        nbytes = 8 * (m * k + k * n + m * n * (2 if case["entry"] == "sub" else 1))
    return {"bytes": nbytes, "flops": 2 * r * m * n * k}


def tolerance(case):
    """The method defines every output: integers, exact products of them, one
    rounding to FP64 at the end.  Planes, exponents and results are the same
    bit for bit in every correct implementation."""
    return "exact"


def exact(case, seed):
    """The FP64 product itself, which the emulation approximates."""
    A, B, C = _inputs(case, seed)
    P = torch.matmul(A, B)
    if case["entry"] == "planes":
        return {"C": P, "planesB": None, "expsB": None}
    return C - P if case["entry"] == "sub" else P
