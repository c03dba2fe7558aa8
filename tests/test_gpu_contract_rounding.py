"""Rounding errors of the projector and of the correlators' gradient against extended precision
(numpy's 80-bit long double): no larger than those of sums taken term by term in double
precision, over sites in 256 parts."""
import numpy as np
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LD = np.clongdouble


def rms(y, ref):
    return float(np.sqrt((np.abs(y - ref) ** 2).sum() / (np.abs(ref) ** 2).sum()))


def coefficients(f, v):
    """f v^dag in double precision: 256 partial sums over sites, term by term, then pairwise."""
    n = f.shape[1] // 3
    p = np.zeros((f.shape[0], v.shape[0], -(-n // 256) * 256, 3), dtype=np.complex128)
    p[:, :, :n] = (f[:, None] * v.conj()[None]).reshape(p.shape[:2] + (n, 3))
    acc = np.zeros(p.shape[:2] + (256,), dtype=p.dtype)
    for i in range(0, p.shape[2], 256):
        for c in range(3):
            acc += p[:, :, i:i + 256, c]
    while acc.shape[2] > 1:
        h = acc.shape[2] // 2
        acc = acc[:, :, :h] + acc[:, :, h:]
    return acc[:, :, 0]


def term_by_term(first, c, v):
    """first + sum_k c[:, k] v[k] in double precision."""
    acc = first.copy()
    for k in range(v.shape[0]):
        acc += c[:, k, None] * v[k]
    return acc


@pytest.mark.parametrize("dims,nev,nd", [((2, 8, 8, 8), 33, 4), ((2, 12, 12, 12), 16, 3), ((2, 6, 6, 6), 21, 5)])
def test_rounding_errors(dims, nev, nd):
    from paper_2201_09729_amd import dlma as D
    print("contraction rounding", dims, nev, nd, flush=True)
    rng = np.random.default_rng(2)
    T, L3 = dims[0], int(np.prod(dims[1:]))
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.25, 3)).cuda(), 0.121, 1.2)
    V = rng.normal(size=(T, nev, 3 * L3)) + 1j * rng.normal(size=(T, nev, 3 * L3))
    V = np.ascontiguousarray(np.stack([np.linalg.qr(v.T)[0].T for v in V]))
    x = synth.random_spinor(dims, 4 * nd, 9)
    W = np.zeros((2, 7, T, 2))
    W[0, 5:, :, 0] = rng.normal(size=(2, T))  # weights of Re PP_exact and Re QP_exact, pseudoscalar
    Vd, xd = torch.from_numpy(V).cuda().reshape((T, nev) + dims[1:] + (3,)), torch.from_numpy(x).cuda()
    proj = D.dlma_project(g, 1, Vd[1], xd, 0).cpu().numpy()
    grad = D.dlma_correlators_grad(g, 0, Vd, xd, None, None, W)[0].cpu().numpy()
    rows = lambda f, t: f[:, t].reshape(4 * nd, L3, 4, 3).transpose(0, 2, 1, 3).reshape(16 * nd, 3 * L3)  # noqa: E731
    f, v = rows(x, 1), V[1]
    c = f.astype(LD) @ v.astype(LD).conj().T
    ref = c @ v.astype(LD)
    cd = coefficients(f, v)
    own = rms(term_by_term(np.zeros_like(f), cd, v), ref)
    err = rms(rows(proj, 1), ref)
    # dL = 2 w5 Re <d, P d> + 2 w6 Re <d, (1 - P) d>: its gradient 2 w6 d + 2 (w5 - w6) P d
    a, b = 2 * W[0, 6, 1, 0], 2 * (W[0, 5, 1, 0] - W[0, 6, 1, 0])
    gref = LD(a) * f + LD(b) * ref
    gown = rms(term_by_term(a * f, b * cd, v), gref)
    gerr = rms(rows(grad, 1), gref)
    print("projector", err, own, "gradient", gerr, gown, flush=True)
    assert err <= own and gerr <= gown
