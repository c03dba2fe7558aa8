"""D's rounding error against extended precision (numpy's 80-bit long double): no larger than
that of the oracle's evaluation in double precision.  The diagonal of the clover term is four
times the other terms; added last it costs one rounding at its size, added first it makes every
later product round there."""
import numpy as np
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LD = np.clongdouble


def dirac_ld(U, A, x):
    """D x in long double: U [T,Z,Y,X,4,3,3], A [T,Z,Y,X,12,12] (spin * 3 + colour), x [n,T,Z,Y,X,4,3]."""
    U, x = U.astype(LD), x.astype(LD)
    s = [np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]]), np.array([[1, 0], [0, -1]])]
    g = [np.block([[np.zeros((2, 2)), -np.eye(2)], [-np.eye(2), np.zeros((2, 2))]])]
    g += [np.block([[np.zeros((2, 2)), -1j * m], [1j * m, np.zeros((2, 2))]]) for m in s]
    out = (A.astype(LD)[None] * x.reshape(x.shape[:5] + (1, 12))).sum(-1).reshape(x.shape)
    for mu, ax in enumerate((1, 4, 3, 2)):
        P, M = (np.eye(4) + g[mu]).astype(LD), (np.eye(4) - g[mu]).astype(LD)
        spin = lambda S, v: (S[:, :, None] * v[..., None, :, :]).sum(-2)  # noqa: E731
        u = U[None, ..., mu, None, :, :]
        f = (u * np.roll(x, -1, ax)[..., None, :]).sum(-1)
        b = np.roll((np.conj(np.swapaxes(u, -1, -2)) * x[..., None, :]).sum(-1), 1, ax)
        out = out - (spin(M, f) + spin(P, b)) / 2
    return out


@pytest.mark.parametrize("dims,n", [((4, 4, 4, 4), 2), ((8, 4, 8, 8), 10)])  # four lanes per site, 64 sites per wave
def test_rounding_error(orc, dims, n):
    from paper_2201_09729_amd import dlma as D
    print("dirac rounding", dims, n, flush=True)
    U = synth.gauge_field(dims, 0.25, 4)
    x = synth.random_spinor(dims, n, 8)
    g = D.dlma_load_gauge(torch.from_numpy(U).cuda(), 0.121, 1.2)
    y = D.dlma_apply_dw(g, torch.from_numpy(x).cuda()).cpu().numpy()
    C = orc.clover(U, 0.121, 1.2)
    ref = dirac_ld(U, C.reshape(dims + (12, 12)), x)
    err, own = (float(np.sqrt((np.abs(v - ref) ** 2).sum() / (np.abs(ref) ** 2).sum())) for v in (y, orc.dirac(U, C, x)))
    print("error", err, "oracle", own, flush=True)
    assert err <= own
