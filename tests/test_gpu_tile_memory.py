"""A BF16 solve in memory that holds the per-thread solver but not the right-hand-side tiles
(padded columns, larger links): the per-thread stencils take it."""
import time

import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_tiles_that_do_not_fit():
    from paper_2201_09729_amd import dlma as D
    dims, n = (10, 48, 48, 48), 13
    u = torch.from_numpy(synth.gauge_field((2, 4, 4, 4), 0.2, 3)).cuda()
    U = u.repeat(5, 12, 12, 12, 1, 1, 1)  # a periodic configuration
    gen = torch.Generator(device="cuda").manual_seed(3)
    b = torch.randn((n,) + dims + (4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    x = torch.zeros_like(b)
    free = lambda: torch.cuda.mem_get_info()[0]  # noqa: E731

    def solve(g, block):
        x.zero_()
        _, st = D.dlma_solve([g], [b], xs=[x], opts=D.default_opts(prec="mix_bf16", rhs_block=block))
        assert all(s["converged"] for s in st)

    need = {}
    for block in (1, 0, 1, 0):  # one thread per site, tiles; first what the runtime keeps for itself
        g = D.dlma_load_gauge(U, 0.119, 1.0)
        D.dlma_release_cache()
        f = free()
        solve(g, block)
        need[block] = f - free()
        g.close()
    g = D.dlma_load_gauge(U, 0.119, 1.0)
    del u, U
    D.dlma_release_cache()
    torch.cuda.empty_cache()
    extra = need[0] - need[1]
    print("solver memory", need, flush=True)
    assert extra > 400 << 20
    fill = []
    for _ in range(20):  # (the driver reports freed memory with a delay)
        over = free() - need[1] - extra // 2
        if over > 32 << 20:
            fill.append(torch.empty(over, dtype=torch.uint8, device="cuda"))
        time.sleep(0.1)
    print("left", free() >> 20, "MiB", flush=True)
    assert free() < need[0] - extra // 4
    solve(g, 0)
