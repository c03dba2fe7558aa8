"""D and D^dag where a plane is cut into strips, against the oracle: 24 x 24 planes (9 waves of
64 sites) on 7 timeslices per XCD with 12 right-hand sides, five strips of two waves with a
padding one; 14 x 2 planes on 64 timeslices per XCD, strips of 8 and 6 rows, four lanes per
site.  Tolerance as in test_gpu_dirac_paths.py."""
import numpy as np
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def strips(dims, nrhs):
    """The launcher's split: (64 sites per wave, strips of a plane)."""
    T, Z, Y, X = dims
    plane, per = Y * X, min(nrhs, 12)
    pw = -(-plane // 64)
    nT = 8 if T % 8 == 0 else (4 if T % 4 == 0 else 2)
    l2 = (8 << 20) // (3 * (T // nT) * per * 192)
    if 2 * plane >= 64 * pw and T * Z * plane * nrhs >= 19200:
        return True, -(-pw // max(1, l2 // 64))
    step = 16 // np.gcd(X, 16)
    return False, -(-Y // min(max(step, l2 // X // step * step), Y))


@pytest.mark.parametrize("dims,nrhs,split", [((14, 2, 24, 24), 12, (True, 5)), ((512, 2, 14, 2), 12, (False, 2))])
@pytest.mark.parametrize("dagger", [False, True])
def test_dirac_in_strips(orc, dims, nrhs, split, dagger):
    from paper_2201_09729_amd import dlma as D
    assert strips(dims, nrhs) == split
    print("dirac strips", dims, nrhs, dagger, flush=True)
    U = synth.gauge_field(dims, 0.3, 4)
    C = orc.clover(U, 0.121, 1.2)
    x = synth.random_spinor(dims, nrhs, 8)
    g = D.dlma_load_gauge(torch.from_numpy(U).cuda(), 0.121, 1.2)
    y = D.dlma_apply_dw(g, torch.from_numpy(x).cuda(), dagger=dagger).cpu().numpy()
    ref = orc.dirac(U, C, x, dagger=dagger)
    assert np.abs(y - ref).max() <= 128 * 2.0**-52 * (24 + 6 * np.abs(C).max()) * np.abs(x).max()
