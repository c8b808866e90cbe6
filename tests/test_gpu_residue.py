"""Products by residues (csrc/residue.h): the full product of the operands
rounded to their rows' and columns' grids, at the edges of its plans, tiles and
k chunks."""
import numpy as np
import pytest

import workload as W

pytestmark = pytest.mark.gpu

COMPS = {"dd": 2, "td": 3, "qd": 4, "ts": 3}


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def mp():
    import torch
    import paper_2301_09960_amd as m
    assert torch.cuda.is_available()
    return m


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def grids(A, B, bits):
    """Half a grid step of each row of A and column of B: every element is
    rounded to a multiple of 2^(E - bits), |x| < 2^E for the whole vector."""
    ea = np.frexp(np.abs(A[0]).max(axis=0))[1]  # A is (c, k, m): one E per row of A
    eb = np.frexp(np.abs(B[0]).max(axis=1))[1]
    return np.ldexp(0.5, ea - bits), np.ldexp(0.5, eb - bits)


def rounding_bound(A, B, bits, c, absab):
    """|C - AB| for operands rounded to their grids and C rounded once to c
    components: the first-order terms, the product of both roundings, and
    2^(2 - 53 c) |A||B| for C."""
    ga, gb = grids(A, B, bits)
    sa, sb = np.abs(A[0]).sum(axis=0), np.abs(B[0]).sum(axis=1)
    k = A.shape[1]
    first = gb[:, None] * sa[None, :] + sb[:, None] * ga[None, :] + k * gb[:, None] * ga[None, :]
    return first * (1 + 2.0 ** -20) + 2.0 ** (2 - 53 * c) * absab


@pytest.mark.parametrize("fmt,D", [("dd", 1), ("dd", 2), ("dd", 7), ("td", 18), ("dd", 17), ("td", 24), ("qd", 31),
                                   ("qd", 40)])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (33, 65, 31), (130, 7, 65), (257, 129, 200)])
def test_digit_form_is_the_rounded_product(mp, orc, fmt, D, m, n, k):
    """Every digit count: plans with and without squared moduli, windows of one
    to nine words, both tile sizes, a short last k step."""
    say(f"residues {fmt} D={D} {m}x{n}x{k}")
    A, B = W.gen_pair(fmt, m, n, k, E=8, seed=D + k)
    C = mp.gemm(fmt, dev(A), dev(B), mode="int8", slices=D).cpu().numpy()
    rows = list(range(m)) if m * n * k < 1e6 else [0, 31, 32, 127, 128, 255, m - 1]
    diff, absab, _ = orc.exact_check(A, B, C, rows=rows)
    assert np.all(diff <= rounding_bound(A[:, :, rows], B, 7 * D - 1, COMPS[fmt], absab))


@pytest.mark.parametrize("k", [32768, 32769, 70000])
def test_long_k_chunks(mp, orc, k):
    """k beyond 32768 takes several chunks of result planes."""
    say(f"residues k={k}")
    m, n = 5, 4
    A, B = W.gen_pair("qd", m, n, k, E=4, seed=k)
    C = mp.gemm("qd", dev(A), dev(B), mode="int8").cpu().numpy()
    D = mp.last_num_slices()
    diff, absab, _ = orc.exact_check(A, B, C)
    assert np.all(diff <= rounding_bound(A, B, 7 * D - 1, 4, absab))


def test_extreme_digits_and_signs(mp, orc):
    """Operands at the ends of the digit range: all elements +-2^E (1 - 2^-53)
    or +-2^(E - 1), sums that cancel exactly, and rows of one sign (the largest
    |X| the moduli must hold)."""
    k, m, n = 256, 6, 5
    big = 1.0 - 2.0 ** -53
    A = np.zeros((2, k, m))
    B = np.zeros((2, n, k))
    s = np.where(np.arange(k) % 2 == 0, 1.0, -1.0)
    A[0] = np.stack([np.full(k, big), np.full(k, -big), big * s, np.full(k, 0.5), -0.5 * s, 2.0 ** 300 * s], axis=1)
    A[1] = A[0] * 2.0 ** -54
    B[0] = np.stack([np.full(k, big), np.full(k, -big), big * s, np.full(k, 0.5), 2.0 ** -300 * np.ones(k)])
    B[1] = B[0] * -2.0 ** -54
    for D in (1, 2, 7, 17, 40):
        C = mp.gemm("dd", dev(A), dev(B), mode="int8", slices=D).cpu().numpy()
        diff, absab, _ = orc.exact_check(A, B, C)
        assert np.all(diff <= rounding_bound(A, B, 7 * D - 1, 2, absab)), D


def test_integers_are_exact(mp):
    """Integer operands lie on every grid: C is the exact product, in both parts."""
    rng = np.random.default_rng(5)
    m, n, k = 70, 45, 300
    a = rng.integers(-2 ** 40, 2 ** 40, (k, m))
    b = rng.integers(-2 ** 40, 2 ** 40, (n, k))
    A = np.stack([a.astype(np.float64), np.zeros((k, m))])
    B = np.stack([b.astype(np.float64), np.zeros((n, k))])
    C = mp.gemm("dd", dev(A), dev(B), mode="int8").cpu().numpy()
    want = b.astype(object) @ a.astype(object)
    got = np.vectorize(lambda x, y: int(x) + int(y), otypes=[object])(C[0], C[1])
    assert np.all(got == want)


@pytest.mark.parametrize("mode", ["float", "int8"])
@pytest.mark.parametrize("m,n,k", [(1, 17, 48), (16, 15, 255), (17, 16, 257), (33, 1, 1041), (2, 18, 8192), (18, 2, 8193)])
def test_maxima_of_whole_vectors(mp, mode, m, n, k):
    """The largest element at a vector's end, at the edges of 16 vectors and 256
    elements, and on both sides of the longest vectors read in one piece: with
    a maximum too small the integers would not fit their words."""
    rng = np.random.default_rng(7)
    a, b = rng.integers(-2 ** 20, 2 ** 20, (k, m)), rng.integers(-2 ** 20, 2 ** 20, (n, k))
    a[k - 1, m - 1], b[n - 1, k - 1], a[0, 0], b[0, 0] = 2 ** 50, -2 ** 50, 2 ** 49 + 1, 2 ** 48 + 3
    A = np.stack([a.astype(np.float64), np.zeros((k, m))])
    B = np.stack([b.astype(np.float64), np.zeros((n, k))])
    C = mp.gemm("dd", dev(A), dev(B), mode=mode).cpu().numpy()
    want = b.astype(object) @ a.astype(object)
    got = np.vectorize(lambda x, y: int(x) + int(y), otypes=[object])(C[0], C[1])
    assert np.all(got == want)


@pytest.mark.parametrize("mode,m,n,k", [("int8", 640, 600, 50), ("float", 1100, 1050, 64), ("int8", 2180, 300, 33),
                                        ("float", 4200, 4100, 48), ("int8", 200, 4352, 32)])
def test_every_grouping_of_the_bases(mp, mode, m, n, k):
    """Tiles short of one round of the chip and past it, whose bases are cut into
    different groups: products of small integers, exact in binary64."""
    rng = np.random.default_rng(11)
    a = rng.integers(-2 ** 15, 2 ** 15, (k, m)).astype(np.float64)
    b = rng.integers(-2 ** 15, 2 ** 15, (n, k)).astype(np.float64)
    C = mp.gemm("dd", dev(np.stack([a, 0 * a])), dev(np.stack([b, 0 * b])), mode=mode).cpu().numpy()
    assert np.array_equal(C[0], b @ a) and not C[1].any()


def slices(mp, fmt, A, B):
    """The product from binary64/binary32 slices: a slice count set by the
    caller is Algorithm 1 with that many slices."""
    D = mp.num_slices(fmt, "float", A.shape[1])
    return mp.gemm(fmt, A, B, slices=D)


FLOAT_SHAPES = [(1, 1, 48), (64, 64, 64), (33, 130, 96), (130, 65, 1000), (257, 300, 129)]


@pytest.mark.parametrize("fmt", ["dd", "td", "qd", "ts"])
@pytest.mark.parametrize("m,n,k", FLOAT_SHAPES)
@pytest.mark.parametrize("E", [0, 16])
def test_float_form_no_less_exact_than_slices(mp, orc, fmt, m, n, k, E):
    """The automatic FLOAT form by residues against the same call from slices:
    the error of every entry within the rounding of the operands to D (b + 1) + 2
    bits and of C, and its root mean square no larger than the slices'."""
    A, B = W.gen_pair(fmt, m, n, k, E=E, seed=m + k + E)
    dA, dB = dev(A), dev(B)
    C = mp.gemm(fmt, dA, dB).cpu().numpy()
    S = slices(mp, fmt, dA, dB).cpu().numpy()
    D = mp.last_num_slices()
    rows = list(range(m)) if m * n * k < 1e6 else [0, m // 2, m - 1]
    diff, absab, _ = orc.exact_check(A, B, C, rows=rows)
    diff_s, _, _ = orc.exact_check(A, B, S, rows=rows)
    single = fmt == "ts"
    b = (24 if single else 53) - orc.rho(24 if single else 53, k)
    bits = max(D * (b + 1) + 2, 116 if single else 0)
    wide = A[:, :, rows].astype(np.float64), B.astype(np.float64)
    assert np.all(diff <= rounding_bound(*wide, bits - 1, COMPS[fmt] * (24 / 53 if single else 1), absab))
    rms, rms_s = np.sqrt(np.mean(diff ** 2)), np.sqrt(np.mean(diff_s ** 2))
    say(f"float {fmt} {m}x{n}x{k} E={E} D={D}: rms {rms:.3g}, slices {rms_s:.3g}")
    # both round C to the format once; the slack covers entries of a few roundings
    assert rms <= 1.05 * rms_s + 2.0 ** -(24 * 3 + 8 if single else 53 * COMPS[fmt] + 6) * absab.max()


def with_gap(fmt, m, n, k, row):
    """Short leading data, and in one row an element 2^-90 below with full
    mantissas: Algorithm 1 follows it down, a fixed grid would cut it off."""
    A, B = W.gen_pair(fmt, m, n, k, E=4, seed=k)
    A[0] = np.rint(A[0] * 2.0 ** 8) * 2.0 ** -8
    A[1:] = 0
    A[:, k - 1, row] = W.gen_matrix(fmt, 1, 1, E=0, seed=3)[:, 0, 0] * A.dtype.type(2.0 ** -90)
    return A, B


@pytest.mark.parametrize("fmt,m,n,k", [("dd", 40, 33, 64), ("dd", 130, 70, 300), ("qd", 50, 40, 200),
                                       ("dd", 33, 20, 8300)])
def test_gaps_fall_back_to_the_slices(mp, fmt, m, n, k):
    """A vector whose slices reach below the fixed grid: the result is the
    slices', bit for bit (also with slices made one pass at a time)."""
    import torch
    A, B = with_gap(fmt, m, n, k, m // 2)
    if fmt == "qd":
        A[:, k - 1, m // 2] *= 2.0 ** -120
    dA, dB = dev(A), dev(B)
    assert torch.equal(mp.gemm(fmt, dA, dB), slices(mp, fmt, dA, dB))
    # the same in a column of B
    tA, tB = dB.permute(0, 2, 1).contiguous(), dA.permute(0, 2, 1).contiguous()  # (c, k, n), (c, m, k)
    assert torch.equal(mp.gemm(fmt, tA, tB), slices(mp, fmt, tA, tB))
    # components that are not normalized
    dA2 = dA.clone()
    dA2[1] = dA2[0] * 0.75
    assert torch.equal(mp.gemm(fmt, dA2, dB), slices(mp, fmt, dA2, dB))


def test_infinities_and_nans_stay_in_their_rows(mp):
    import torch
    m, n, k = 70, 66, 128
    A, B = W.gen_pair("td", m, n, k, E=8, seed=2)
    clean = mp.gemm("td", dev(A), dev(B))
    A[0, 5, 3] = np.inf
    A[0, 7, 64] = np.nan
    B[0, 65, 100] = -np.inf
    B[:, 4, :] = 0
    dA, dB = dev(A), dev(B)
    C, S = mp.gemm("td", dA, dB), slices(mp, "td", dA, dB)
    assert torch.equal(torch.isnan(C[0]), torch.isnan(S[0]))
    keep = ~torch.isnan(C[0])
    keep[4, :] = False
    assert torch.equal(C[:, keep], clean[:, keep])
    assert bool(torch.all(C[:, 4, :3] == 0))


def test_batch_falls_back_per_product(mp):
    """Flagged products of a batch take the slices, the others the residues,
    each as its single call does; replayed with other operands."""
    import torch
    sh = [(64, 64, 64), (40, 33, 64), (130, 70, 300), (20, 20, 16), (65, 129, 700)]
    for round_ in range(3):
        pairs = []
        for i, (m, n, k) in enumerate(sh):
            gap = (i + round_) % 2 == 0 and k >= 48
            pairs.append(with_gap("dd", m, n, k, 1) if gap else W.gen_pair("dd", m, n, k, E=8, seed=i + round_))
        As, Bs = [dev(a) for a, _ in pairs], [dev(b) for _, b in pairs]
        Cs = mp.gemm_batched("dd", As, Bs)
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(As, Bs)):
            assert torch.equal(Cs[i], mp.gemm("dd", a, b)), (round_, sh[i])


@pytest.mark.parametrize("mode,m,n,k", [("float", 1500, 1400, 100), ("int8", 100, 90, 9000)])
def test_fixed_scratch_takes_the_product_in_parts(mp, mode, m, n, k):
    """Shapes whose planes exceed the scratch of mpgemm_dd_noalloc: blocks of C
    (float), groups of bases (int8), the same C."""
    import ctypes
    import torch
    A, B = W.gen_pair("dd", m, n, k, E=8, seed=4)
    dA, dB = dev(A), dev(B)
    old = mp.get_mode("dd")
    mp.set_mode("dd", mode)
    try:
        want = mp.gemm("dd", dA, dB)
        got = torch.zeros_like(want)
        P = ctypes.c_void_p
        assert mp.workspace_bytes("dd", mode, m, n, k) > 64 << 20
        st = mp.lib().mpgemm_dd_noalloc(m, n, k, P(dA.data_ptr()), m, P(dB.data_ptr()), k, P(got.data_ptr()), m,
                                        P(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
    finally:
        mp.set_mode("dd", old)
    assert st == 0 and torch.equal(got, want)


def noalloc(mp, A, B, C, mode):
    import ctypes
    import torch
    P = ctypes.c_void_p
    (k, m), n = A.shape[1:], B.shape[1]
    old = mp.get_mode("dd")
    mp.set_mode("dd", mode)
    try:
        st = mp.lib().mpgemm_dd_noalloc(m, n, k, P(A.data_ptr()), m, P(B.data_ptr()), k, P(C.data_ptr()), m,
                                        P(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
    finally:
        mp.set_mode("dd", old)
    assert st == 0
    return C


@pytest.mark.parametrize("mode,gap", [("float", False), ("float", True), ("int8", False)])
@pytest.mark.parametrize("into", ["A", "B"])
def test_result_in_the_place_of_an_operand(mp, mode, gap, into):
    """C may be A or B, also where the slices take over: one product, a batch
    whose products write each other's operands, and the fixed scratch."""
    import torch
    n = 96
    A, B = with_gap("dd", n, n, n, n // 2) if gap else W.gen_pair("dd", n, n, n, E=4, seed=n)
    dA, dB = dev(A), dev(B)
    want = mp.gemm("dd", dA, dB, mode=mode).clone()
    a, b = dA.clone(), dB.clone()
    assert torch.equal(mp.gemm("dd", a, b, a if into == "A" else b, mode=mode), want)
    As, Bs = [dA.clone() for _ in range(3)], [dB.clone() for _ in range(3)]
    Cs = [(As if into == "A" else Bs)[(i + 1) % 3] for i in range(3)]
    for C in mp.gemm_batched("dd", As, Bs, Cs, mode=mode):
        assert torch.equal(C, want)
    m = 1000 if mode == "float" else 700  # FLOAT: the fixed scratch takes it in blocks of C
    A, B = W.gen_pair("dd", m, m, 60, E=4, seed=7)
    side = torch.zeros((2, m, m), dtype=torch.float64, device="cuda")
    flat = side.reshape(-1)
    a, b = dev(A), dev(B)
    apart = noalloc(mp, a, b, torch.zeros_like(side), mode)
    x = a if into == "A" else b
    shared = flat[:x.numel()].reshape(x.shape)
    shared.copy_(x)
    got = noalloc(mp, shared if into == "A" else a, b if into == "A" else shared, side, mode)
    # slices against residues: both within the bound of the format
    scale = np.abs(B[0]) @ np.abs(A[0])
    assert np.all(((got[0] - apart[0]) + (got[1] - apart[1])).abs().cpu().numpy() <= 2.0 ** -99 * scale)


@pytest.mark.parametrize("fmt", ["dd", "td", "qd"])
@pytest.mark.parametrize("D", [1, 2, 7, 17])
def test_elements_round_to_nearest_even(mp, fmt, D):
    """Elements at and next to half a step of their grid, with the lower components
    above, below and on both sides of it: C is the element rounded to nearest,
    ties to even (a product with a unit vector), exactly."""
    from fractions import Fraction
    c = COMPS[fmt]
    bits = 7 * D - 1
    u = 2.0 ** -bits  # E = 0: |x| < 1, the largest 0.75
    rows = []
    for h in (0, 1, 2, 3, 2 ** min(bits, 50) // 3, 2 ** min(bits, 50) // 3 + 1):
        for sign in (1.0, -1.0):
            for tail in ((0, 0), (1, 0), (-1, 0), (1, -1), (-1, 1), (1, 1), (-1, -1)):
                lead = (h + 0.5) * 2.0 ** -min(bits, 50) * sign
                x = [lead, 0.0, 0.0, 0.0]
                if bits > 50:  # the half step is in a lower component
                    x[0] = h * 2.0 ** -50 * sign
                    x[1] = 0.5 * u * sign
                at = 2 if bits > 50 else 1
                for r, t in enumerate(tail):
                    if at + r < c:
                        x[at + r] = t * abs(lead if bits <= 50 else x[1]) * 2.0 ** (-60 * (r + 1))
                rows.append(x[:c])
    m, k = len(rows), 3
    A = np.zeros((c, k, m))
    A[:, 1, :] = np.array(rows).T
    A[0, 2, :] = 0.75
    B = np.zeros((c, 1, k))
    B[0, 0, 1] = 1.0
    say(f"rounding {fmt} D={D}: {m} elements")
    C = mp.gemm(fmt, dev(A), dev(B), mode="int8", slices=D).cpu().numpy()
    for i, x in enumerate(rows):
        steps = sum(map(Fraction, x)) / Fraction(u)
        assert sum(Fraction(float(v)) for v in C[:, 0, i]) == round(steps) * Fraction(u), (x, C[:, 0, i])


def structured(fmt, shape, m, n, k, seed):
    """Operands with structural zeros and a spread of exponents that the fixed grid
    cuts off: A (c, k, m) keeps the elements (p, i) of the pattern."""
    A, B = W.gen_pair(fmt, m, n, k, E=50, seed=seed)
    p, i = np.arange(k)[:, None], np.arange(m)[None, :]
    rng = np.random.default_rng(seed)
    keep = {"front": p >= 40, "lower": p * m >= (i - 8) * k, "upper": p * m <= (i + 8) * k,
            "band": np.abs(p * m - i * k) <= 12 * max(m, k), "blocks": ((p // 48 + i // 16) % 3 == 0) & (p >= 33),
            "sparse": rng.random((k, m)) < 24.0 / k}[shape]
    return A * keep, B


def flagged(mp, fmt, A, B):
    """The product, and whether it was left to the slices: the word behind the rest
    of an attached workspace."""
    import torch
    (k, m), n = A.shape[1:], B.shape[1]
    ws = torch.empty(mp.workspace_bytes(fmt, "float", m, n, k), dtype=torch.uint8, device="cuda")
    mp.set_workspace(ws)
    try:
        C = mp.gemm(fmt, A, B)
        torch.cuda.synchronize()
    finally:
        mp.set_workspace(None)
    return C, bool(ws[-256:-252].cpu().view(torch.int32)[0])


@pytest.mark.parametrize("fmt", ["dd", "td", "qd", "ts"])
@pytest.mark.parametrize("shape,m,n,k", [("front", 70, 66, 200), ("lower", 150, 40, 160), ("upper", 90, 33, 300),
                                         ("band", 200, 50, 220), ("blocks", 130, 70, 500), ("sparse", 40, 60, 1000),
                                         ("front", 33, 20, 8300), ("sparse", 18, 17, 9000)])
def test_structural_zeros_keep_the_residues(mp, orc, fmt, shape, m, n, k):
    """Triangular, banded, sparse operands, and zeros in front, are settled by the
    elements that are not zero: the product is not left to the slices, as either
    operand, meets the bound of its grid, and is the same in a batch."""
    import torch
    say(f"structured {fmt} {shape} {m}x{n}x{k}")
    A, B = structured(fmt, shape, m, n, k, seed=k + m)
    dA, dB = dev(A), dev(B)
    C, left = flagged(mp, fmt, dA, dB)
    assert not left
    D = mp.last_num_slices()
    rows = [0, m // 2, m - 1]
    diff, absab, _ = orc.exact_check(A, B, C.cpu().numpy(), rows=rows)
    single = fmt == "ts"
    b = (24 if single else 53) - orc.rho(24 if single else 53, k)
    bits = max(D * (b + 1) + 2, 116 if single else 0)
    wide = A[:, :, rows].astype(np.float64), B.astype(np.float64)
    assert np.all(diff <= rounding_bound(*wide, bits - 1, COMPS[fmt] * (24 / 53 if single else 1), absab))
    # the transposed product: the same entries
    tA, tB = dB.permute(0, 2, 1).contiguous(), dA.permute(0, 2, 1).contiguous()
    Ct, left = flagged(mp, fmt, tA, tB)
    assert not left and torch.equal(Ct.permute(0, 2, 1), C)
    X, Y = W.gen_pair(fmt, 50, 60, 70, E=8, seed=1)
    out = mp.gemm_batched(fmt, [dA, dev(X), tA], [dB, dev(Y), tB])
    assert torch.equal(out[0], C) and torch.equal(out[2].permute(0, 2, 1), C)


def test_slices_are_needed(mp):
    """The word the test above reads is set where a fixed grid would cut off what the
    slices follow, and not for a dense operand."""
    A, B = with_gap("dd", 70, 66, 200, 5)
    assert flagged(mp, "dd", dev(A), dev(B))[1]
    A, B = W.gen_pair("dd", 70, 66, 200, E=50, seed=1)
    assert not flagged(mp, "dd", dev(A), dev(B))[1]


def exact_integers(m, n, k):
    """Operands of small integers and their exact product, equal in binary64."""
    rng = np.random.default_rng(m + n + k)
    a = rng.integers(-2 ** 15, 2 ** 15, (k, m)).astype(np.float64)
    b = rng.integers(-2 ** 15, 2 ** 15, (n, k)).astype(np.float64)
    return dev(np.stack([a, 0 * a])), dev(np.stack([b, 0 * b])), b @ a


@pytest.mark.parametrize("mode", ["int8", "float"])
@pytest.mark.parametrize("tile", [1, 3])
@pytest.mark.parametrize("m,n,k", [(70, 66, 32769), (33, 300, 65536), (300, 40, 70001)])
def test_k_chunks_on_several_blocks(mp, mode, tile, m, n, k):
    """Chunks of k on more than one block of C, in both forms and tile sizes."""
    say(f"chunks {mode} tile {tile} {m}x{n}x{k}")
    A, B, want = exact_integers(m, n, k)
    mp.set_int8_tile(tile)
    try:
        C = mp.gemm("dd", A, B, mode=mode).cpu().numpy()
    finally:
        mp.set_int8_tile(0)
    assert np.array_equal(C[0], want) and not C[1].any()


@pytest.mark.parametrize("mode", ["int8", "float"])
def test_k_chunks_in_a_batch(mp, mode):
    """A batch of products with one, two and three chunks, some of one combine launch."""
    shapes = [(70, 66, 100), (65, 34, 32769), (40, 130, 70000), (33, 33, 33000), (300, 290, 32768)]
    data = [exact_integers(*s) for s in shapes]
    say(f"chunks in a batch {mode}")
    for _ in range(2):
        Cs = mp.gemm_batched("dd", [d[0] for d in data], [d[1] for d in data], mode=mode)
        for C, (_, _, want), s in zip(Cs, data, shapes):
            C = C.cpu().numpy()
            assert np.array_equal(C[0], want) and not C[1].any(), s
