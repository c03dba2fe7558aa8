"""The projector on small and large timeslices: one-launch coefficients and the contraction
kernel, one or two column sets per wave, against the product in numpy.

Tolerance: the bound of a dot product of n terms, (n + 4) 2^-52 times the sum of the moduli,
for the coefficients (3 L3 terms) and the expansion (nev terms) in series."""
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


# L3 = 8, 144, 600 (one launch), 2048 on both sides of the rule, 3072 (contraction), 16^3 with
# enough right-hand sides for two column sets per wave; counts that leave partial sets of four
@pytest.mark.parametrize("dims,nev,nrhs", [((2, 2, 2, 2), 1, 1), ((4, 6, 4, 6), 35, 10), ((2, 10, 6, 10), 7, 5), ((2, 16, 8, 16), 9, 6),
                                           ((2, 16, 8, 16), 17, 13), ((2, 12, 16, 16), 3, 9), ((2, 16, 16, 16), 33, 27)])
def test_project(D, dims, nev, nrhs):
    print("project", dims, nev, nrhs, flush=True)
    rng = np.random.default_rng(5)
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.2, 3)).cuda(), 0.121, 1.0)
    sp = dims[1:]
    V = rng.normal(size=(nev,) + sp + (3,)) + 1j * rng.normal(size=(nev,) + sp + (3,))
    x = synth.random_spinor(dims, nrhs, 9)
    L3, t = int(np.prod(sp)), dims[0] - 1
    v, f = V.reshape(nev, L3 * 3), x[:, t].reshape(nrhs, L3, 4, 3).transpose(0, 2, 1, 3).reshape(nrhs * 4, L3 * 3)
    p, a = (f @ v.conj().T) @ v, (np.abs(f) @ np.abs(v).T) @ np.abs(v)
    tol = (3 * L3 + nev + 8) * 2.0**-52 * (a + np.abs(f))
    for mode in (0, 1):
        out = D.dlma_project(g, t, torch.from_numpy(V).cuda(), torch.from_numpy(x).cuda(), mode).cpu().numpy()
        got = out[:, t].reshape(nrhs, L3, 4, 3).transpose(0, 2, 1, 3).reshape(nrhs * 4, L3 * 3)
        assert np.all(np.abs(got - (f - p if mode else p)) <= tol)
        out[:, t] = 0
        assert not out.any()
