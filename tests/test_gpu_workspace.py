"""Workspaces kept between calls on the default stream: calls from several
threads, sizes on both sides of a kept one's size and of the largest, and calls
on other streams in between give what each call gives alone."""
import threading

import pytest

pytestmark = pytest.mark.gpu

# (format, form, m, n, k): workspaces within 8 MiB, above it, and above 256 MiB
CALLS = [("dd", "int8", 64, 64, 64), ("dd", "float", 96, 64, 80), ("qd", "int8", 130, 70, 90),
         ("ts", "float", 512, 500, 300), ("td", "float", 700, 512, 256), ("dd", "float", 40, 33, 16),
         ("qd", "int8", 1600, 1500, 900)]


def operands(fmt, m, n, k, seed):
    import torch
    c = {"dd": 2, "td": 3, "qd": 4, "ts": 3}[fmt]
    dt = torch.float32 if fmt == "ts" else torch.float64
    g = torch.Generator().manual_seed(seed)
    A, B = torch.zeros((c, k, m), dtype=dt), torch.zeros((c, n, k), dtype=dt)
    A[0], B[0] = torch.rand((k, m), generator=g, dtype=dt) - 0.5, torch.rand((n, k), generator=g, dtype=dt) - 0.5
    return A.cuda(), B.cuda()


@pytest.mark.parametrize("side", [False, True])
def test_threads_share_kept_workspaces(side):
    import torch
    import paper_2301_09960_amd as mp
    data = [operands(f, m, n, k, i) for i, (f, _, m, n, k) in enumerate(CALLS)]
    want = []
    for (f, mode, *_), (A, B) in zip(CALLS, data):
        want.append(mp.gemm(f, A, B, mode=mode))
        torch.cuda.synchronize()
    wrong = []

    def work(t):
        stream = torch.cuda.Stream() if side and t % 2 else torch.cuda.default_stream()
        with torch.cuda.stream(stream):
            outs = []
            for r in range(3):
                for i in range(len(CALLS)):
                    i = (i * (t + 1) + r) % len(CALLS)
                    outs.append((i, mp.gemm(CALLS[i][0], *data[i], mode=CALLS[i][1])))
            stream.synchronize()
            wrong.extend((t, CALLS[i]) for i, C in outs if not torch.equal(C, want[i]))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def least(mp, fmt, m, n, k):
    """Bytes of the binary64/binary32 slices alone."""
    mp.set_last_slice("remainder")
    try:
        return mp.workspace_bytes(fmt, "float", m, n, k)
    finally:
        mp.set_last_slice("extract")


@pytest.mark.parametrize("fmt,m,n,k", [("dd", 1500, 1400, 100), ("qd", 1100, 300, 64), ("ts", 530, 1210, 48),
                                       ("td", 300, 290, 2000)])
def test_product_in_less_than_its_planes(fmt, m, n, k):
    """An attached workspace between what the slices need and what all residue
    planes need: the product in parts is the product, and C in an operand's place
    is the slices'; the slices alone still run, less is refused."""
    import torch
    import paper_2301_09960_amd as mp
    A, B = operands(fmt, m, n, k, 1)
    want = mp.gemm(fmt, A, B)
    by_slices = mp.gemm(fmt, A, B, slices=mp.num_slices(fmt, "float", k))
    low, full = least(mp, fmt, m, n, k), mp.workspace_bytes(fmt, "float", m, n, k)
    assert full > low
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    try:
        for size in sorted({low + 256, low + 1000, (low + full) // 2, full - 256, full}):
            print(f"workspace {fmt} {m}x{n}x{k}: {size} of {full}", flush=True)
            mp.set_workspace(ws[:size])
            assert torch.equal(mp.gemm(fmt, A, B), want), size
        mp.set_workspace(ws[:low])
        assert torch.equal(mp.gemm(fmt, A, B), by_slices)
        mp.set_workspace(ws[: low - 256])
        with pytest.raises(mp.MpgemmError) as ei:
            mp.gemm(fmt, A, B)
        assert ei.value.status == 2
        mp.set_workspace(ws[: low + 256])  # A in C's memory
        side = torch.zeros(max(A.numel(), want.numel()), dtype=A.dtype, device="cuda")
        a = side[: A.numel()].reshape(A.shape)
        a.copy_(A)
        C = mp.gemm(fmt, a, B, side[: want.numel()].reshape(want.shape))
        assert torch.equal(C, want if fmt == "td" else by_slices)  # td: whole, in groups of moduli
    finally:
        mp.set_workspace(None)


def test_digit_form_and_certificate_in_less():
    """INT8: the planes of 9000 k in groups of moduli; the certified product and
    the D+S product in a workspace below all planes."""
    import torch
    import paper_2301_09960_amd as mp
    m, n, k = 100, 90, 9000
    A, B = operands("dd", m, n, k, 2)
    want = mp.gemm("dd", A, B, mode="int8")
    full = mp.workspace_bytes("dd", "int8", m, n, k)
    D = mp.num_slices("dd", "int8", k)
    low = D * 256 * 9024 + 4 * D * 128 * 128 + 65536  # digits and sums
    assert low < full
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    try:
        mp.set_workspace(ws[:low])
        assert torch.equal(mp.gemm("dd", A, B, mode="int8"), want)
    finally:
        mp.set_workspace(None)
    m, n, k = 1500, 1400, 100
    A, B = operands("dd", m, n, k, 3)
    C, cert, worst = mp.certify("dd", A, B)
    ds = [A[:1], torch.zeros((1, k, m), dtype=torch.float32, device="cuda"), B[:1],
          torch.zeros((1, n, k), dtype=torch.float32, device="cuda")]
    hi, lo = mp.ds_gemm(*ds)
    copies = 2 * 8 * (m * k + k * n + m * n) + 768
    ws = torch.empty(least(mp, "dd", m, n, k) + 256 + copies, dtype=torch.uint8, device="cuda")
    try:
        mp.set_workspace(ws)
        hi2, lo2 = mp.ds_gemm(*ds)
        assert torch.equal(hi, hi2) and torch.equal(lo, lo2)
        mp.set_workspace(ws[: ws.numel() - copies])
        C2, cert2, worst2 = mp.certify("dd", A, B)
        assert torch.equal(C, C2) and torch.equal(cert, cert2) and torch.equal(worst, worst2)
    finally:
        mp.set_workspace(None)


def test_large_result_of_short_rows():
    """A C whose residue planes are beyond what a call takes for them (9 of 8 GiB):
    formed in blocks by the ordinary call, bit for bit the products of its parts."""
    import torch
    import paper_2301_09960_amd as mp
    m, n, k = 15900, 15700, 48
    g = torch.Generator(device="cuda").manual_seed(9)
    A, B = torch.zeros((2, k, m), dtype=torch.float64, device="cuda"), torch.zeros((2, n, k), dtype=torch.float64, device="cuda")
    A[0], B[0] = torch.rand((k, m), generator=g, device="cuda", dtype=torch.float64) - 0.5, torch.rand((n, k), generator=g, device="cuda", dtype=torch.float64) - 0.5
    A[1], B[1] = A[0] * 2.0 ** -55, B[0] * -2.0 ** -56
    assert mp.workspace_bytes("dd", "float", m, n, k) <= (8 << 30) + 256
    C = mp.gemm("dd", A, B)
    for i0, i1, j0, j1 in [(0, 700, 0, 800), (7900, 8200, 7900, 8300), (15000, m, 15100, n), (8100, 8300, 100, 5000)]:
        part = mp.gemm("dd", A[:, :, i0:i1].contiguous(), B[:, j0:j1].contiguous())
        assert torch.equal(C[:, j0:j1, i0:i1], part), (i0, j0)
