"""dlma_set_mass with a mass for which A is not positive definite: an error, after which the
storage-precision operators are those of the handle's new A: the same numbers, infinities and
NaN of a failed inverse included, as on a handle that had no copies of the first mass."""
import pytest

from paper_2201_09729_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["mix_fp32", "mix_fp16", "mix_bf16"])
@pytest.mark.parametrize("n", [1, 16])  # BF16: one thread per site, tiles
def test_failed_mass_leaves_no_stale_copy(prec, n):
    from paper_2201_09729_amd import dlma as D
    dims = (4, 4, 4, 6)
    print("failed mass", prec, n, flush=True)
    U = torch.from_numpy(synth.gauge_field(dims, 0.2, 11)).cuda()
    x = torch.from_numpy(synth.random_spinor(dims, n, 5)).cuda()
    out = []
    for copies in (True, False):
        g = D.dlma_load_gauge(U, 0.121, 1.0)
        if copies:
            first = D.dlma_apply_schur(g, x, prec=prec)
        with pytest.raises(D.DlmaError) as e:
            D.dlma_set_mass(g, 1e6)
        assert e.value.code == D.DLMA_EINVAL and "positive definite" in str(e.value)
        out.append(torch.view_as_real(D.dlma_apply_schur(g, x, prec=prec)))
        D.dlma_set_mass(g, 0.121)  # and a good mass is good again (A to rounding)
        d = D.dlma_apply_schur(g, x, prec=prec) - first
        assert torch.linalg.vector_norm(d) <= 2.0**-5 * torch.linalg.vector_norm(first)
    a, b = out
    assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a[~a.isnan()], b[~b.isnan()])
    assert not torch.equal(a, torch.view_as_real(first))
