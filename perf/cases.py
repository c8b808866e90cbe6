"""The calls whose time on one MI355X is followed from one state of the library to the next.

Each case is one call as a program makes it through the package's public
entry points, on operands it already holds in HBM: single products, batches of
uneven products, and an LU factorization with its solve.  Sizes are those of
the benchmark (4096 square, batches and requests of 64 to 1024 and 64 to 2048,
the LU of order 2048) and of the tests' ragged shapes; entries follow the
benchmark's recipe (a uniform mantissa times a power of two spread over E
bits, lower components below half an ulp).

    listed()            the cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) operands and output buffers on the GPU
    run(state)          one pass; returns the whole result
    work(case)          bytes and operations no implementation can do without
    exact(case, seed)   the result from Python integers or plain float64
"""
import math

import numpy as np
import torch

import paper_2301_09960_amd as mp

COMPS = mp.COMPONENTS


def listed():
    return [
        # the smallest request of the serving mix: launches and latency count
        dict(name="dd 64 float", kind="gemm", fmt="dd", mode="float", m=64, n=64, k=64, E=8),
        # a ragged request below one tile row per compute unit
        dict(name="td 200x150x333 float", kind="gemm", fmt="td", mode="float", m=200, n=150, k=333, E=8),
        # the smallest square of the benchmark's grid, the default form
        dict(name="dd 1024 float", kind="gemm", fmt="dd", mode="float", m=1024, n=1024, k=1024, E=16),
        # triple binary32, the format with the cheapest matrix-core work
        dict(name="ts 2048 float", kind="gemm", fmt="ts", mode="float", m=2048, n=2048, k=2048, E=8),
        # the benchmark's step: one DD and one QD product, the default form
        dict(name="dd 4096 float", kind="gemm", fmt="dd", mode="float", m=4096, n=4096, k=4096, E=16),
        dict(name="qd 4096 float", kind="gemm", fmt="qd", mode="float", m=4096, n=4096, k=4096, E=16),
        # an odd-sized request of the serving mix in the digit form
        dict(name="qd 777x1021x643 int8", kind="gemm", fmt="qd", mode="int8", m=777, n=1021, k=643, E=8),
        # the same step in the digit form
        dict(name="dd 4096 int8", kind="gemm", fmt="dd", mode="int8", m=4096, n=4096, k=4096, E=16),
        dict(name="qd 4096 int8", kind="gemm", fmt="qd", mode="int8", m=4096, n=4096, k=4096, E=16),
        # batches of uneven products, one launch each, in both forms
        dict(name="batch 128 qd float", kind="batch", fmt="qd", mode="float", count=128, lo=64, hi=1024, E=8),
        dict(name="batch 256 dd int8", kind="batch", fmt="dd", mode="int8", count=256, lo=64, hi=1024, E=8),
        # the application: LU with slice-product updates, and the solve
        dict(name="lu dd 2048 K128 float", kind="lu", fmt="dd", mode="float", n=2048, K=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choices(("gemm", "batch", "lu"), (6, 2, 1))[0]
    if kind == "lu":
        return dict(kind="lu", fmt=rng.choice(("dd", "td")), mode=rng.choice(("float", "int8")),
                    n=_log_int(rng, 128, 2048), K=rng.choice((32, 64, 128, 256)))
    fmt = rng.choice(("dd", "td", "qd", "ts"))
    mode = "float" if fmt == "ts" else rng.choice(("float", "int8"))
    if kind == "batch":
        return dict(kind="batch", fmt=fmt, mode=mode, count=_log_int(rng, 8, 256), lo=64,
                    hi=_log_int(rng, 128, 1024), E=rng.randint(0, 16))
    m, n, k = (_log_int(rng, 24, 3000) for _ in range(3))
    return dict(kind="gemm", fmt=fmt, mode=mode, m=m, n=n, k=k, E=rng.randint(0, 16))


def _entries(gen, fmt, count, E):
    """(c, count) normalized expansions: u 2^e and components below half an ulp."""
    single = fmt == "ts"
    dt, bits = (torch.float32, 24) if single else (torch.float64, 53)
    c = COMPS[fmt]
    out = torch.empty((c, count), dtype=dt, device="cuda")
    u = torch.rand(count, generator=gen, dtype=dt, device="cuda") * 2 - 1
    e = torch.randint(0, E + 1, (count,), generator=gen, device="cuda")
    out[0] = torch.ldexp(u, e.to(dt))
    for r in range(1, c):
        v = torch.rand(count, generator=gen, dtype=dt, device="cuda") - 0.5
        out[r] = out[r - 1] * 2.0 ** -bits * v
    return out


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _batch_shapes(case):
    """The sizes of a batch belong to the case, not to the seed of its entries."""
    rng = np.random.default_rng(31)
    lo, hi = case["lo"], case["hi"]
    return np.rint(lo * (hi / lo) ** rng.random((case["count"], 3))).astype(int).tolist()


def prepare(case, seed):
    gen = _generator(seed)
    fmt = case["fmt"]
    c = COMPS[fmt]
    dt = torch.float32 if fmt == "ts" else torch.float64
    s = dict(case)
    if case["kind"] == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        s["A"] = _entries(gen, fmt, m * k, case["E"]).reshape(c, k, m)
        s["B"] = _entries(gen, fmt, k * n, case["E"]).reshape(c, n, k)
        s["C"] = torch.empty((c, n, m), dtype=dt, device="cuda")
    elif case["kind"] == "batch":
        shapes = _batch_shapes(case)
        pool = _entries(gen, fmt, sum(m * k + k * n for m, n, k in shapes), case["E"])
        s["out"] = torch.empty(c * sum(m * n for m, n, k in shapes), dtype=dt, device="cuda")
        s["A"], s["B"], s["C"] = [], [], []
        at = to = 0
        for m, n, k in shapes:
            s["A"].append(pool[:, at:at + m * k].reshape(c, k, m).contiguous())
            at += m * k
            s["B"].append(pool[:, at:at + k * n].reshape(c, n, k).contiguous())
            at += k * n
            s["C"].append(s["out"][to:to + c * m * n].reshape(c, n, m))
            to += c * m * n
    else:
        n = case["n"]
        # uniform entries made diagonally dominant, as the LU's tests and timings use
        X = torch.rand((n, n), generator=gen, dtype=torch.float64, device="cuda")
        X += n * torch.eye(n, dtype=torch.float64, device="cuda")
        planes = [X]
        for _ in range(1, c):
            planes.append(planes[-1] * 2.0 ** -53 * (torch.rand((n, n), generator=gen, dtype=torch.float64,
                                                                device="cuda") - 0.5))
        s["A"] = torch.stack(planes)
        s["b"] = torch.zeros((c, n), dtype=torch.float64, device="cuda")
        s["b"][0] = 1.0 / torch.arange(1, n + 1, dtype=torch.float64, device="cuda")
    return s


def run(s):
    if s["kind"] == "gemm":
        return mp.gemm(s["fmt"], s["A"], s["B"], s["C"], mode=s["mode"])
    if s["kind"] == "batch":
        mp.gemm_batched(s["fmt"], s["A"], s["B"], s["C"], mode=s["mode"])
        return s["out"]
    LU = mp.lu(s["fmt"], s["A"].clone(), s["K"], mode=s["mode"])  # in place: the matrix is kept
    return {"lu": LU, "x": mp.lu_solve(s["fmt"], LU, s["b"])}


def work(case):
    """Operands read once and results written once; one multiply-add per pair of
    components (r, s) with r + s < c of each term, the products that reach the
    format's length."""
    c = COMPS[case["fmt"]]
    size = 4 if case["fmt"] == "ts" else 8
    pairs = c * (c + 1) // 2
    if case["kind"] == "lu":
        n = case["n"]
        return {"bytes": 2 * size * c * n * n + 2 * size * c * n, "flops": pairs * (2 * n ** 3 / 3 + 2 * n * n)}
    shapes = [(case["m"], case["n"], case["k"])] if case["kind"] == "gemm" else _batch_shapes(case)
    return {"bytes": sum(size * c * (m * k + k * n + m * n) for m, n, k in shapes),
            "flops": sum(pairs * 2 * m * n * k for m, n, k in shapes)}


def _integers(planes):
    """Object array of integers N and q with the value N 2^q of each entry."""
    planes = planes.double().cpu().numpy()
    nonzero = np.abs(planes[planes != 0])
    q = int(math.floor(math.log2(nonzero.min()))) - 60 if nonzero.size else 0
    total = np.zeros(planes.shape[1:], dtype=object)
    for p in planes:
        frac, ex = np.frexp(p)
        total = total + (np.ldexp(frac, 53).astype(np.int64).astype(object) <<
                         np.maximum(ex - 53 - q, 0).astype(object))
    return total, q


def _components(value, q, c, single):
    """The c leading components (nearest) of the integers value times 2^q."""
    out = np.zeros((c,) + value.shape, dtype=np.float64)
    for at, v in np.ndenumerate(value):
        for r in range(c):
            if v == 0:
                break
            x = float(v)
            if single:
                x = float(np.float32(math.ldexp(x, q))) / 2.0 ** q
            out[(r,) + at] = math.ldexp(x, q)
            v -= int(x)
    return out


def _exact_product(fmt, A, B):
    """C = AB as (c, n, m): every component from integers where that is quick, else
    the product in float64 in the leading component."""
    c, k, m = A.shape
    n = B.shape[1]
    if m * n * k <= 1 << 24:
        (Ai, qa), (Bi, qb) = _integers(A), _integers(B)
        q = qa + qb
        return torch.from_numpy(_components(Bi.dot(Ai), q, c, fmt == "ts"))
    C = torch.zeros((c, n, m), dtype=torch.float64, device="cuda")
    C[0] = B.double().sum(0) @ A.double().sum(0)
    return C


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "gemm":
        return _exact_product(case["fmt"], s["A"], s["B"])
    if case["kind"] == "batch":
        out = torch.zeros_like(s["out"], dtype=torch.float64)
        to = 0
        for A, B, C in zip(s["A"], s["B"], s["C"]):
            mn = C.shape[1] * C.shape[2]
            out[to:to + mn] = (B.double().sum(0) @ A.double().sum(0)).reshape(-1)
            to += C.numel()
        return out
    # elimination without pivoting on the leading components (planes are
    # column-major: row i of the matrix is X[:, i])
    n = case["n"]
    M = s["A"].sum(0).T.contiguous()
    for j in range(n - 1):
        M[j + 1:, j] /= M[j, j]
        M[j + 1:, j + 1:] -= torch.outer(M[j + 1:, j], M[j, j + 1:])
    LU = torch.zeros_like(s["A"])
    LU[0] = M.T
    x = torch.zeros_like(s["b"])
    x[0] = torch.linalg.solve(s["A"].sum(0).T, s["b"].sum(0))
    return {"lu": LU, "x": x}
