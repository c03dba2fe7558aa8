"""The BF16 inner solver on tiles of sixteen right-hand sides: its Schur stencils against
the oracle and its solves' true residuals, at counts that fill tiles and leave remainders.

Tolerance of the operator as in test_gpu_schur.py: 4u relative per right-hand side and 8u
site by site (a few independent storage roundings in series, FP32 accumulation)."""
import numpy as np
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PREC, TOL = "mix_bf16", 4 * 2.0**-8


@pytest.fixture(scope="module")
def D():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_09729_amd import dlma
    return dlma


def cu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# strips of y rows: whole (X/2 = 2), a shorter last one (X/2 = 10, 14), one row
# longer than a block's 48 sites (X/2 = 70); fewer timeslices than XCDs and more
@pytest.mark.parametrize("dims,nrhs", [((4, 2, 6, 4), 16), ((2, 4, 8, 20), 13), ((10, 4, 6, 28), 27), ((2, 2, 4, 140), 14),
                                       ((18, 2, 2, 2), 48), ((4, 4, 2, 6), 40)])
def test_tile_operator_matches_oracle(D, orc, dims, nrhs):
    print("tiles", dims, nrhs, flush=True)
    U = synth.gauge_field(dims, 0.25, 11)
    x = synth.random_spinor(dims, nrhs, 61)
    x *= 10.0 ** np.random.default_rng(1).uniform(-6, 3, x.shape[:-2])[..., None, None]  # site scales far apart
    ref = orc.schur(U, orc.clover(U, 0.121, 1.2), x)
    g = D.dlma_load_gauge(cu(U), 0.121, 1.2)
    y = D.dlma_apply_schur(g, cu(x), prec=PREC, rhs_block=0).cpu().numpy()
    d, r = (y - ref).reshape(nrhs, -1), ref.reshape(nrhs, -1)
    assert (np.linalg.norm(d, axis=1) / np.linalg.norm(r, axis=1)).max() <= TOL
    ds, rs = (np.linalg.norm(a.reshape(nrhs, -1, 12), axis=2).max(axis=1) for a in (d, r))
    assert (ds / rs).max() <= 2 * TOL
    D.dlma_set_mass(g, 0.119)  # the tiles' clover follows the mass
    ref = orc.schur(U, orc.clover(U, 0.119, 1.2), x)
    y = D.dlma_apply_schur(g, cu(x), prec=PREC, rhs_block=0).cpu().numpy()
    assert (np.linalg.norm((y - ref).reshape(nrhs, -1), axis=1) / np.linalg.norm(ref.reshape(nrhs, -1), axis=1)).max() <= TOL


@pytest.mark.parametrize("sizes", [[((16, 8, 8, 8), 13)], [((4, 4, 4, 4), 45)], [((8, 4, 6, 10), 26), ((4, 8, 4, 6), 16), ((2, 2, 2, 6), 14)]])
def test_tile_solves_reach_the_residual(D, orc, sizes):
    print("tile solve", sizes, flush=True)
    Us = [synth.gauge_field(d, 0.3, 2 + i) for i, (d, _) in enumerate(sizes)]
    bs = [synth.random_spinor(d, n, 21 + i) for i, (d, n) in enumerate(sizes)]
    for b in bs:
        b[1] = 0  # a zero source, and one far smaller than the others
        b[2] *= 1e-8
    gs = [D.dlma_load_gauge(cu(U), 0.120, 1.0) for U in Us]
    for dagger in (0, 1):
        xs, st = D.dlma_solve(gs, [cu(b) for b in bs], opts=D.default_opts(tol=1e-10, prec=PREC, maxiter=4000, dagger=dagger))
        assert all(s["converged"] for s in st)
        for U, b, x in zip(Us, bs, xs):
            x = x.cpu().numpy()
            assert np.all(x[1] == 0)
            keep = [i for i in range(len(b)) if i != 1]
            if dagger:
                r = orc.dirac(U, orc.clover(U, 0.120, 1.0), x[keep], dagger=True) - b[keep]
                res = np.linalg.norm(r.reshape(len(keep), -1), axis=1) / np.linalg.norm(b[keep].reshape(len(keep), -1), axis=1)
            else:
                res = orc.true_residual(U, orc.clover(U, 0.120, 1.0), x[keep], b[keep])
            assert np.all(res <= 1.001e-10), res


@pytest.mark.parametrize("single", [True, False])
def test_tile_first_pass_skipping_is_exact(D, single):
    """From x = 0 the first pass skips what is zero; an explicit x0 = 0 skips nothing and takes
    the same arithmetic: identical solutions.  Replays and direct launches agree as well."""
    dims, n = (32, 4, 4, 4), 28
    g = D.dlma_load_gauge(cu(synth.gauge_field(dims, 0.3, 2)), 0.120, 1.0)
    b = np.zeros((n,) + dims + (4, 3), dtype=np.complex128)
    r = synth.random_spinor(dims, n, 33)
    for i in range(n):
        t = 7 if single else (3, 5, 31, 0)[i % 4]
        b[i, t] = r[i, t]
    if not single:
        b[3] = r[3]  # dense
    print("tile skipping", single, flush=True)
    (x1,), s1 = D.dlma_solve([g], [cu(b)], opts=D.default_opts(prec=PREC))
    (x0,), s0 = D.dlma_solve([g], [cu(b)], xs=[torch.zeros_like(x1)], opts=D.default_opts(prec=PREC, use_x0=1))
    assert torch.equal(x1, x0)
    assert [s["inner_iters"] for s in s1] == [s["inner_iters"] for s in s0]
    (x2,), s2 = D.dlma_solve([g], [cu(b)], opts=D.default_opts(prec=PREC, graph_iters=0))
    assert torch.equal(x1, x2)
