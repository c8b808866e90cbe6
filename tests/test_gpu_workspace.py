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
