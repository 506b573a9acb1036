"""Timed cases of the emulated GEMM library: what its callers run, through the
public Python entry points, from calls of a few microseconds of arithmetic to
the largest squares of the benchmark.

A case is a plain dict: the entry point (``op``), the sizes M, N, K of
op(A) (M x K) and op(B) (K x N), for the FP64 calls the product count
``nprod``, and where they differ from the defaults the BLAS flags and factors,
the exponent scope and the armed fallback of the DGEMM, and the class of input
values.  Inputs are drawn on the GPU from the seed alone.

Value classes (those of the tests and the benchmark):
  uniform   [-1, 1)
  normal    standard normal
  wide      s m 2^e, m uniform in [1, 2), e uniform in [-20, 20]
  rows      normal, one row in a hundred scaled by 2^16
  outside   normal times 2^e, e uniform in [-160, 160]: FP64 data that does not
            fit BF16's exponent range (the armed fallback computes it)
"""
import torch

import paper_2609_04663_amd as emu

SCOPES = {"operand": emu.SCOPE_OPERAND, "rowcol": emu.SCOPE_ROWCOL, "kbin": emu.SCOPE_KBIN}


def listed():
    return [
        # the smallest call: one 128-cube block of a serving or solver loop, on
        # the entry point that never allocates
        {"name": "dgemm6-128-noalloc", "op": "dgemm_noalloc", "M": 128, "N": 128, "K": 128,
         "nprod": 6, "inputs": "uniform"},
        # a small single-precision call
        {"name": "sgemm-256", "op": "sgemm", "M": 256, "N": 256, "K": 256, "inputs": "normal"},
        # a small call at full double precision
        {"name": "dgemm21-512", "op": "dgemm", "M": 512, "N": 512, "K": 512, "nprod": 21,
         "inputs": "normal"},
        # odd extents: no tile, vector or alignment boundary is met
        {"name": "sgemm-odd", "op": "sgemm", "M": 1111, "N": 777, "K": 1501, "inputs": "normal"},
        # the benchmark's size sweep at 1024 and 2048
        {"name": "dgemm10-1024", "op": "dgemm", "M": 1024, "N": 1024, "K": 1024, "nprod": 10,
         "inputs": "wide"},
        {"name": "dgemm6-2048", "op": "dgemm", "M": 2048, "N": 2048, "K": 2048, "nprod": 6,
         "inputs": "uniform"},
        # a residual update C = C - A^T B of a solver, with the fallback armed
        # (the inputs do not need it) and extents that are not powers of two
        {"name": "dgemm15-update", "op": "dgemm_ex", "M": 3000, "N": 2000, "K": 4000, "nprod": 15,
         "transa": "T", "alpha": -1.0, "beta": 1.0, "fallback": True, "inputs": "normal"},
        # the long-reduction workload as a Gram-type product A^T B
        {"name": "sgemm-gram-65536", "op": "sgemm_ex", "M": 1024, "N": 1024, "K": 65536,
         "transa": "T", "inputs": "normal"},
        # the short-reduction workload with badly scaled rows: row/column scope
        {"name": "dgemm10-16384-k512-rowcol", "op": "dgemm", "M": 16384, "N": 16384, "K": 512,
         "nprod": 10, "scope": "rowcol", "inputs": "rows"},
        # scale that varies along the reduction: K-binned scope
        {"name": "dgemm21-kbin", "op": "dgemm", "M": 1024, "N": 1024, "K": 16384, "nprod": 21,
         "scope": "kbin", "inputs": "rows"},
        # the benchmark's squares, single precision and the deepest of its product counts
        {"name": "sgemm-8192", "op": "sgemm", "M": 8192, "N": 8192, "K": 8192, "inputs": "normal"},
        {"name": "dgemm21-8192", "op": "dgemm", "M": 8192, "N": 8192, "K": 8192, "nprod": 21,
         "inputs": "wide"},
    ]


MAX_PRODUCTS = 21 * 8192 ** 3      # component products of the largest listed call
MAX_ELEMENTS = 16384 * 16384       # entries of its largest matrix


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi]; half of them even 64s."""
    n = int(round(lo * (hi / lo) ** rng.random()))
    return max(64, n // 64 * 64) if rng.random() < 0.5 else n


def draw(rng):
    """One more case: any entry point, option and size of the listed ranges."""
    while True:
        op = rng.choice(["sgemm", "sgemm", "sgemm_ex", "dgemm", "dgemm", "dgemm", "dgemm_ex",
                         "dgemm_noalloc"])
        top = 1024 if op == "dgemm_noalloc" else 16384
        c = {"op": op, "M": _size(rng, 64, top), "N": _size(rng, 64, top),
             "K": _size(rng, 64, min(4 * top, 65536))}
        if op.startswith("sgemm"):
            c["inputs"] = rng.choice(["normal", "uniform", "rows"])
        else:
            c["nprod"] = rng.choice([6, 10, 15, 21])
            c["inputs"] = rng.choice(["uniform", "normal", "wide"])
            r = rng.random()
            if op != "dgemm_noalloc" and r < 0.15:
                c["scope"], c["inputs"] = "rowcol", "rows"
            elif op != "dgemm_noalloc" and r < 0.25:
                c["scope"], c["inputs"] = "kbin", "rows"
            elif r < 0.45:
                c["fallback"] = True
                if r < 0.32:
                    c["inputs"] = "outside"
        if op.endswith("_ex"):
            c["transa"], c["transb"] = rng.choice("NT"), rng.choice("NT")
            c["alpha"], c["beta"] = rng.choice([(1.0, 0.0), (-1.0, 1.0), (0.5, 0.0), (2.0, -0.5)])
        M, N, K = c["M"], c["N"], c["K"]
        # an FP64 matrix multiply recomputes a call that takes the fallback: it
        # costs about as much as its 21 products
        np_ = 40 if c["inputs"] == "outside" else _nprod(c)
        if (np_ * M * N * K <= MAX_PRODUCTS and max(M * K, K * N, M * N) <= MAX_ELEMENTS
                and (op != "dgemm_noalloc" or (M + N + 512) * (K + 32) * 12 <= 48 << 20)):
            return c


def _nprod(case):
    return case.get("nprod", 6)


def _dtype(case):
    return torch.float32 if case["op"].startswith("sgemm") else torch.float64


def _values(kind, rows, cols, gen):
    dev = gen.device

    def normal():
        return torch.randn((rows, cols), generator=gen, device=dev, dtype=torch.float64)

    def uniform():
        return torch.rand((rows, cols), generator=gen, device=dev, dtype=torch.float64)

    if kind == "uniform":
        return uniform().mul_(2.0).sub_(1.0)
    if kind == "normal":
        return normal()
    if kind == "rows":
        X = normal()
        n = (rows + 99) // 100
        X[torch.randperm(rows, generator=gen, device=dev)[:n]] *= 2.0 ** 16
        return X
    span = 20 if kind == "wide" else 160
    e = torch.randint(-span, span + 1, (rows, cols), generator=gen, device=dev).double()
    if kind == "outside":
        return normal().mul_(torch.exp2(e))
    x = uniform().mul_(2.0).sub_(1.0)
    return x.sign().mul_(1.0 + x.abs()).mul_(torch.exp2(e))


def _operands(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    M, N, K = case["M"], case["N"], case["K"]
    ta, tb = case.get("transa", "N") == "T", case.get("transb", "N") == "T"
    dt = _dtype(case)
    A = _values(case["inputs"], *((K, M) if ta else (M, K)), gen).to(dt)
    B = _values(case["inputs"], *((N, K) if tb else (K, N)), gen).to(dt)
    C0 = None
    if case.get("beta", 0.0) != 0.0:
        C0 = _values("normal", M, N, gen).to(dt)
    return A, B, C0


def prepare(case, seed):
    A, B, C0 = _operands(case, seed)
    C = torch.empty((case["M"], case["N"]), dtype=A.dtype, device=A.device)
    return {"case": case, "A": A, "B": B, "C0": C0, "C": C}


def _call(case, A, B, C):
    op = case["op"]
    if op == "sgemm":
        return emu.sgemm(A, B, C)
    if op == "dgemm":
        return emu.dgemm(A, B, case["nprod"], C)
    if op == "dgemm_noalloc":
        return emu.dgemm_noalloc(A, B, case["nprod"], C)
    kw = {"transa": case.get("transa", "N"), "transb": case.get("transb", "N"),
          "alpha": case.get("alpha", 1.0), "beta": case.get("beta", 0.0)}
    if op == "sgemm_ex":
        return emu.sgemm_ex(A, B, C, **kw)
    return emu.dgemm_ex(A, B, case["nprod"], C, **kw)


def run(state):
    case, A, B, C, C0 = (state[k] for k in ("case", "A", "B", "C", "C0"))
    if C0 is not None:
        C.copy_(C0)               # the caller keeps the matrix that the call updates
    scope, fallback = case.get("scope"), case.get("fallback", False)
    if scope is None and not fallback:
        return _call(case, A, B, C)
    if scope is not None:
        emu.set_split_scope(SCOPES[scope])
    if fallback:
        emu.set_fallback(emu.FALLBACK_FP64)
    try:
        return _call(case, A, B, C)
    finally:
        emu.set_split_scope(emu.SCOPE_OPERAND)
        emu.set_fallback(emu.FALLBACK_NONE)


def work(case):
    """Each operand read once, the output written (and read for beta != 0);
    the retained component products, two operations each."""
    M, N, K = case["M"], case["N"], case["K"]
    size = 4 if case["op"].startswith("sgemm") else 8
    out = M * N * (2 if case.get("beta", 0.0) != 0.0 else 1)
    return {"bytes": size * (M * K + K * N + out), "flops": 2 * _nprod(case) * M * N * K}


def tolerance(case):
    if case["op"].startswith("sgemm"):
        # FP32 sums in another order: each is 0.9e-7 .. 1.8e-7 off the exact product
        return {"rel": 8e-7, "max": 6e-6}
    if case["inputs"] == "outside":
        # the plain FP64 product, its sums in another order
        return {"rel": 4e-15}
    # every panel product is exact and the order of the FP64 additions is part
    # of the interface: the same bits
    return "exact"


def exact(case, seed):
    """The product in FP64 from the inputs as given (for the FP32 calls exact
    products and 53-bit sums)."""
    A, B, C0 = _operands(case, seed)
    A, B = A.double(), B.double()
    P = (A.T if case.get("transa", "N") == "T" else A) @ (B.T if case.get("transb", "N") == "T" else B)
    P *= case.get("alpha", 1.0)
    if C0 is not None:
        P += case["beta"] * C0.double()
    return P
