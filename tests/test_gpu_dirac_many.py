"""D on more right-hand sides than one launch takes: planes of 2 x 2 sites leave three of four
lanes idle, so that 2^32 threads are reached at 52 GB of fields.  Each right-hand side has to
come out as it does in a short call."""
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_dirac_beyond_one_launch():
    from paper_2201_09729_amd import dlma as D
    dims, n, k = (8, 128, 2, 2), 66000, 12
    if torch.cuda.mem_get_info()[0] < 2.2 * n * 4096 * 192:
        pytest.skip("needs 115 GB of device memory")
    print("dirac", dims, n, flush=True)
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.3, 4)).cuda(), 0.121, 1.2)
    x = torch.empty((n // k, k) + dims + (4, 3), dtype=torch.complex128, device="cuda")
    first = torch.from_numpy(synth.random_spinor(dims, k, 8)).cuda()
    x[:] = first
    y = D.dlma_apply_dw(g, x.view((n,) + dims + (4, 3))).view(x.shape)
    ref = D.dlma_apply_dw(g, first)
    assert all(bool((y[i:i + 100] == ref).all()) for i in range(0, n // k, 100))
