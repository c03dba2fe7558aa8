"""D and D^dag on canonical fields, four lanes per site and 64 sites per wave, against the
oracle: planes that fill a wave, several and none whole, slabs of timeslices and of z, rows
wider than a wave, more right-hand sides than share a place.

Tolerance: 54 complex products per number, the bound of their sum in any order,
64 * 2 * 2^-52 times the sum of their moduli, which is at most (24 + 6 max |C|) max |x|."""
import numpy as np
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_09729_amd import dlma
    return dlma


@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 3), ((6, 2, 4, 6), 14), ((4, 6, 10, 6), 1), ((6, 4, 2, 140), 1),  # four lanes
                                       ((8, 4, 8, 8), 10), ((4, 6, 10, 14), 13), ((12, 2, 6, 6), 25), ((2, 6, 4, 66), 7),
                                       ((10, 10, 14, 12), 2)])
@pytest.mark.parametrize("dagger", [False, True])
def test_dirac(D, orc, dims, nrhs, dagger):
    print("dirac", dims, nrhs, dagger, flush=True)
    U = synth.gauge_field(dims, 0.3, 4)
    C = orc.clover(U, 0.121, 1.2)
    x = synth.random_spinor(dims, nrhs, 8)
    g = D.dlma_load_gauge(torch.from_numpy(U).cuda(), 0.121, 1.2)
    y = D.dlma_apply_dw(g, torch.from_numpy(x).cuda(), dagger=dagger).cpu().numpy()
    ref = orc.dirac(U, C, x, dagger=dagger)
    assert np.abs(y - ref).max() <= 128 * 2.0**-52 * (24 + 6 * np.abs(C).max()) * np.abs(x).max()
