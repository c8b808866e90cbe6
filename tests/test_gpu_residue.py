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
