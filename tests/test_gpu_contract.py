"""GPU contractions at the edges of their tiles against the oracle: modes in blocks of 16
and 32, distillation groups in pairs, sites in steps of four and split over chunks."""
import numpy as np
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (dims, nev, ndist, nnoise, ndil): one site step per chunk, several chunks (L3 >= 128), one and
# several mode blocks with remainders, odd and even groups, either source kind alone
CASES = [((2, 2, 2, 2), 1, 1, 1, 1), ((4, 2, 4, 2), 15, 2, 0, 1), ((2, 4, 4, 8), 16, 3, 2, 2),
         ((2, 6, 8, 10), 17, 0, 3, 3), ((6, 4, 8, 6), 33, 5, 1, 1), ((2, 4, 4, 6), 70, 4, 6, 6)]


@pytest.mark.parametrize("dims,nev,ndist,nnoise,ndil", CASES)
def test_contractions_at_tile_edges(orc, dims, nev, ndist, nnoise, ndil):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_09729_amd import dlma as D
    print("contract", dims, nev, ndist, nnoise, flush=True)
    T = dims[0]
    t0 = T - 1
    n = 3 * int(np.prod(dims[1:]))
    rng = np.random.default_rng(nev)
    V = rng.standard_normal((T, n, nev)) + 1j * rng.standard_normal((T, n, nev))
    nev = min(nev, n)
    V = np.linalg.qr(V)[0][:, :, :nev].transpose(0, 2, 1).reshape((T, nev) + dims[1:] + (3,))
    f = [synth.random_spinor(dims, max(4 * k, 1), 30 + i)[:4 * k] for i, k in enumerate((ndist, nnoise, nnoise))]
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.3, 1)).cuda(), 0.120, 1.0)
    c = [torch.from_numpy(np.ascontiguousarray(a)).cuda() if len(a) else None for a in f]
    Vg = torch.from_numpy(np.ascontiguousarray(V)).cuda()
    got = D.dlma_correlators(g, t0, Vg, *c, ndil=ndil)
    # an empty kind enters the oracle as one group of zeros: its pieces vanish
    o = [a if len(a) else np.zeros((4,) + dims + (4, 3), complex) for a in f]
    ref = orc.correlators(V, t0, *o, ndil=ndil)
    # sums of up to n * 16 * groups products of O(1) entries in FP64: 1e-12 of the largest piece
    scale = max(np.abs(ref[a][p]).max() for a in ref for p in ref[a])
    for a in ref:
        for p in ref[a]:
            assert np.abs(got[a][p] - ref[a][p]).max() <= 1e-12 * scale, (a, p)
    G = rng.standard_normal((2, D.NPARTS, T, 2))
    if T > 2:
        G[:, :, 1] = 0  # a timeslice without weight
    grads = D.dlma_correlators_grad(g, t0, Vg, *c, G, ndil=ndil)
    Gd = {a: {p: G[i, j, :, 0] + 1j * G[i, j, :, 1] for j, p in enumerate(D.PART_NAMES)} for i, a in enumerate(D.GAMMA_NAMES)}
    want = orc.correlators_vjp(V, t0, *o, Gd, ndil=ndil)
    gs = max(np.abs(w).max() for w in want)
    for a, w in zip(grads, want):
        if a is not None:
            assert np.abs(a.cpu().numpy() - w).max() <= 1e-12 * gs


@pytest.mark.parametrize("dims,nev,nrhs", [((2, 2, 2, 2), 1, 1), ((4, 4, 2, 6), 17, 5), ((2, 6, 10, 8), 33, 9), ((2, 4, 4, 4), 0, 3),
                                           ((2, 6, 8, 8), 48, 16)])
def test_projector_at_tile_edges(orc, dims, nev, nrhs):
    """Modes in blocks of 16 and 32, right-hand sides in fours and eights with remainders, several site chunks."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_09729_amd import dlma as D
    print("project", dims, nev, nrhs, flush=True)
    n = 3 * int(np.prod(dims[1:]))
    rng = np.random.default_rng(nev + nrhs)
    V = np.linalg.qr(rng.standard_normal((n, max(nev, 1))) + 1j * rng.standard_normal((n, max(nev, 1))))[0][:, :nev]
    V = np.ascontiguousarray(V.T).reshape((nev,) + dims[1:] + (3,))
    x = synth.random_spinor(dims, nrhs, 8)
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.3, 1)).cuda(), 0.120, 1.0)
    for t, mode in ((dims[0] - 1, 0), (0, 1)):
        got = D.dlma_project(g, t, torch.from_numpy(V).cuda(), torch.from_numpy(x).cuda(), mode)
        same = torch.full_like(got, float("nan"))
        D.dlma_project_noalloc(g, t, torch.from_numpy(V).cuda(), torch.from_numpy(x).cuda(), mode, same)
        assert torch.equal(got, same)
        # orthonormal modes: FP64 sums of n products of O(1) entries
        assert np.abs(got.cpu().numpy() - orc.project(V, x, t, mode)).max() < 1e-13 * np.abs(x).max()
