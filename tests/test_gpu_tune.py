"""The autotuner times the kernels whose options it sets."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["dd", "ts"])
def test_layouts_are_timed_on_slices(fmt, monkeypatch):
    """Every timed product is formed from slices, in the layout being timed: a
    product with the automatic slice count would go by residues."""
    import torch
    import paper_2301_09960_amd as mp
    from paper_2301_09960_amd import tune
    n, seen = 256, []

    def gemm(f, A, B, C, **options):
        seen.append((mp.tile_layout(f), options.get("mode"), options.get("slices")))
        return mp.gemm(f, A, B, C, **options)

    monkeypatch.setattr(tune, "gemm", gemm)
    times = tune.time_layouts(fmt, n, reps=2)
    D = mp.num_slices(fmt, "float", n)
    assert seen == [(lay, "float", D) for lay in tune.LAYOUTS for _ in range(3)]
    assert set(times) == set(tune.LAYOUTS) and all(t > 0 for t in times.values())
    torch.cuda.synchronize()
