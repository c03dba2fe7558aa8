"""dlma_bench_schur times the stencils that the solver runs: with well filled tiles the BF16
tile kernels (which have no adjoint), with a rhs_block of the caller's the per-thread ones,
Dhat and Dhat^dag in turn."""
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,block,tiles", [(16, 0, True), (27, 0, True), (5, 0, False), (16, 2, False)])
def test_bf16_bench_runs_the_solver_s_stencils(n, block, tiles):
    from paper_2201_09729_amd import dlma as D
    print("bench", n, block, flush=True)
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field((4, 4, 6, 8), 0.25, 3)).cuda(), 0.121, 1.2)
    D.dlma_bench_schur(g, "mix_bf16", n, block, 2)  # (tunes)
    D.dlma_profile_reset()
    D.dlma_profile_enable(True)
    ms, by = D.dlma_bench_schur(g, "mix_bf16", n, block, 6)
    D.dlma_profile_enable(False)
    assert ms > 0 and by > 0
    k1, k1dag, k2 = (D.dlma_profile_read(k)[0] for k in (0, 1, 4))
    assert (k1, k1dag, k2) == ((8, 0, 8) if tiles else (4, 4, 8))
