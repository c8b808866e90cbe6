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


def held(f):
    """Device memory that a call leaves allocated outside torch's allocator."""
    import torch
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    f()
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0]


def test_batch_plan_shares_planes_and_slices():
    """The slices behind a FLOAT batch's residues lie in their planes' place: a plan
    of square products takes little more than the slices alone."""
    import torch
    import paper_2301_09960_amd as mp
    n, count = 1000, 20
    A, B = operands("dd", n, n, n, 4)
    Cs = [torch.empty((2, n, n), dtype=torch.float64, device="cuda") for _ in range(count)]
    mp.batched_cache_clear()
    D = mp.num_slices("dd", "float", n)
    sliced = held(lambda: mp.gemm_batched("dd", [A] * count, [B] * count, Cs, slices=D))
    mp.batched_cache_clear()
    both = held(lambda: mp.gemm_batched("dd", [A] * count, [B] * count, Cs))
    mp.batched_cache_clear()
    print(f"plan: slices {sliced >> 20} MiB, with residues {both >> 20} MiB", flush=True)
    assert sliced >= count * D * 2 * n * n * 8
    assert both <= 1.5 * sliced


def tall(m, n, k, seed, front=0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.zeros((2, k, m), dtype=torch.float64, device="cuda")
    B = torch.zeros((2, n, k), dtype=torch.float64, device="cuda")
    A[0] = torch.rand((k, m), generator=g, device="cuda", dtype=torch.float64) - 0.5
    B[0] = torch.rand((n, k), generator=g, device="cuda", dtype=torch.float64) - 0.5
    A[1], B[1] = A[0] * 2.0 ** -55, B[0] * -2.0 ** -56
    A[:, :front] = 0
    return A, B


@pytest.mark.parametrize("shapes", [[(7000, 6800, 64)] * 6 + [(300, 200, 90), (100, 90, 30)],
                                    [(300, 200, 90), (15900, 15700, 48), (65, 600, 129)]])
def test_batch_in_runs(shapes):
    """Batches whose planes exceed 8 GiB: run by run, a product beyond it alone by
    its own call, each bit for bit as its single call; with a C in an operand's
    memory by slices; and the first way again."""
    import torch
    import paper_2301_09960_amd as mp
    mp.batched_cache_clear()
    pairs = [tall(m, n, k, i) for i, (m, n, k) in enumerate(shapes)]
    As, Bs = [a for a, _ in pairs], [b for _, b in pairs]
    Cs = [torch.empty((2, n, m), dtype=torch.float64, device="cuda") for m, n, _ in shapes]
    for attempt in range(2):
        for C in Cs:
            C.fill_(-1.0)
        used = held(lambda: mp.gemm_batched("dd", As, Bs, Cs))
        print(f"runs, attempt {attempt}: plan {used >> 20} MiB", flush=True)
        assert used <= (9 << 30)
        for i, (a, b) in enumerate(pairs):
            assert torch.equal(Cs[i], mp.gemm("dd", a, b)), (attempt, shapes[i])
        if attempt == 0:  # the last C where another product's A lies, which has entries enough
            host = Cs[-1]
            last = len(shapes) - 1
            flat = torch.zeros(max(As[0].numel(), host.numel()), dtype=torch.float64, device="cuda")
            shared_a = flat[: As[0].numel()].reshape(As[0].shape)
            shared_a.copy_(As[0])
            shared_c = flat[: host.numel()].reshape(host.shape)
            mp.gemm_batched("dd", [shared_a] + As[1:], Bs, Cs[:-1] + [shared_c])
            torch.cuda.synchronize()
            for i, (a, b) in enumerate(pairs):
                got = shared_c if i == last else Cs[i]
                k = shapes[i][2]
                assert torch.equal(got, mp.gemm("dd", a, b, slices=mp.num_slices("dd", "float", k))), shapes[i]
            del flat, shared_a, shared_c
    mp.batched_cache_clear()


def test_batch_padding_after_the_slices():
    """Odd numbers of k blocks: the slices of a flagged call lie in the planes'
    padding of k, which the next calls of the plan need to be zero."""
    import torch
    import paper_2301_09960_amd as mp
    shapes = [(70, 90, 90), (33, 40, 150), (200, 130, 65)]
    plain = [operands("dd", *s, 20 + i) for i, s in enumerate(shapes)]
    gaps = []
    for A, B in plain:  # short leading data, and full mantissas 2^-90 below in one row
        A2 = torch.zeros_like(A)
        A2[0] = torch.round(A[0] * 256) / 256
        A2[0, -1, 1] = A[0, -1, 1] * 2.0 ** -90
        A2[1, -1, 1] = A2[0, -1, 1] * 2.0 ** -54
        gaps.append((A2, B))
    mp.batched_cache_clear()
    for pairs in (gaps, plain, gaps, plain):
        Cs = mp.gemm_batched("dd", [a for a, _ in pairs], [b for _, b in pairs])
        torch.cuda.synchronize()
        for C, (a, b) in zip(Cs, pairs):
            assert torch.equal(C, mp.gemm("dd", a, b))


def trim_pool():
    """Frees what the device's stream-ordered pool keeps."""
    import ctypes
    import torch
    torch.cuda.synchronize()
    hip, pool = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), torch.cuda.current_device()) == 0
    assert hip.hipMemPoolTrimTo(pool, ctypes.c_size_t(0)) == 0


def test_when_memory_is_short():
    """A device with less memory left than a call takes: a single product makes do
    with what its slices need, a batch goes product by product; the results are the
    usual ones."""
    import torch
    import paper_2301_09960_amd as mp
    shapes = [(9000, 8800, 64), (8800, 9000, 80), (300, 200, 90), (17000, 16500, 48)]
    pairs = [tall(m, n, k, i) for i, (m, n, k) in enumerate(shapes)]
    Cs = [torch.empty((2, n, m), dtype=torch.float64, device="cuda") for m, n, _ in shapes]
    mp.batched_cache_clear()
    ws = torch.empty(max(mp.workspace_bytes("dd", "float", *s) for s in shapes), dtype=torch.uint8, device="cuda")
    mp.set_workspace(ws)
    try:
        want = [mp.gemm("dd", a, b) for a, b in pairs]
        torch.cuda.synchronize()
    finally:
        mp.set_workspace(None)
    del ws
    torch.cuda.empty_cache()
    trim_pool()
    filler = []
    try:
        while (free := torch.cuda.mem_get_info()[0]) > (6 << 30):
            filler.append(torch.empty(min(free - (5 << 30), 64 << 30), dtype=torch.uint8, device="cuda"))
        print(f"{free >> 20} MiB left", flush=True)
        assert mp.workspace_bytes("dd", "float", *shapes[3]) > free
        mp.gemm_batched("dd", [a for a, _ in pairs[:3]], [b for _, b in pairs[:3]], Cs[:3])
        for C, w in zip(Cs[:3], want):
            assert torch.equal(C, w)
        mp.gemm("dd", *pairs[3], Cs[3])
        assert torch.equal(Cs[3], want[3])
        assert mp.last_num_slices() == mp.num_slices("dd", "float", 48)
    finally:
        del filler
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        mp.batched_cache_clear()
        trim_pool()


def test_digit_form_batch_in_runs():
    """INT8 products of long k, whose planes take twice their digits: two runs, in one
    where a C lies in another product's operand; each as its single call."""
    import torch
    import paper_2301_09960_amd as mp
    shapes = [(20, 24, 300000)] * 8 + [(70, 90, 100)]
    mp.batched_cache_clear()
    pairs = [tall(m, n, k, i) for i, (m, n, k) in enumerate(shapes)]
    As, Bs = [a for a, _ in pairs], [b for _, b in pairs]
    want = [mp.gemm("dd", a, b, mode="int8") for a, b in pairs]
    Cs = [torch.empty_like(w) for w in want]
    used = held(lambda: mp.gemm_batched("dd", As, Bs, Cs, mode="int8"))
    D = mp.num_slices("dd", "int8", 300000)
    digits = 8 * D * 2 * 128 * 300032
    print(f"INT8 runs: plan {used >> 20} MiB, digits {digits >> 20} MiB", flush=True)
    assert used <= 1.8 * digits
    for C, w in zip(Cs, want):
        assert torch.equal(C, w)
    flat = As[0].clone().reshape(-1)  # the last product's C in the first one's A
    C = flat[: Cs[-1].numel()].reshape(Cs[-1].shape)
    mp.gemm_batched("dd", [flat.reshape(As[0].shape)] + As[1:], Bs, Cs[:-1] + [C], mode="int8")
    for got, w in zip(Cs[:-1] + [C], want):
        assert torch.equal(got, w)
    mp.batched_cache_clear()
