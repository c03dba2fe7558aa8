"""Correlators and their gradient with less device memory left than the partial sums over site
chunks would take: fewer chunks, the same numbers to rounding."""
import time

import numpy as np
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_partial_sums_that_do_not_fit():
    from paper_2201_09729_amd import dlma as D
    dims, nev = (32, 8, 8, 8), 1536  # one group: 32 chunks, 13 MB of projections each
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.2, 3)).cuda(), 0.121, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(5)
    V = torch.randn((32, nev, 8, 8, 8, 3), dtype=torch.complex128, device="cuda", generator=gen)
    x = torch.randn((4,) + dims + (4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    W = np.random.default_rng(1).normal(size=(2, 7, 32, 2))
    free = lambda: torch.cuda.mem_get_info()[0]  # noqa: E731
    D.dlma_release_cache()
    f = free()
    ref, gref = D.dlma_correlators_array(g, 3, V, x), D.dlma_correlators_grad(g, 3, V, x, None, None, W)[0]
    need = f - free()
    D.dlma_release_cache()
    torch.cuda.empty_cache()
    left, fill = 160 << 20, []
    print("contraction memory", need >> 20, "MiB", flush=True)
    assert need > 2 * left
    for _ in range(20):  # (the driver reports freed memory with a delay)
        over = free() - left
        if over > 32 << 20:
            fill.append(torch.empty(over, dtype=torch.uint8, device="cuda"))
        time.sleep(0.1)
    print("left", free() >> 20, "MiB", flush=True)
    assert free() < 256 << 20
    got, ggot = D.dlma_correlators_array(g, 3, V, x), D.dlma_correlators_grad(g, 3, V, x, None, None, W)[0]
    # sums of 1536 terms of projections over 1536 numbers each: 2^-52 times their number, twice
    tol = 2 * 3072 * 2.0**-52
    assert np.abs(got - ref).max() <= tol * np.abs(ref).max()
    del fill
    assert (ggot - gref).abs().max().item() <= tol * gref.abs().max().item()
