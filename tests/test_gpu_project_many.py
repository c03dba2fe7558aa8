"""The projector's passes through its scratch: with more right-hand sides than one contraction
takes, every coefficient is formed before the first output is written, so mode 0 (which reads
its inputs for the coefficients alone) may write over the inputs of later right-hand sides."""
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


# 32 modes on 16^3: 64 right-hand sides per contraction (allocation-free: 16); on 4^2 x 8 the
# one-launch coefficients
@pytest.mark.parametrize("dims,nev,n", [((2, 16, 16, 16), 32, 70), ((2, 4, 4, 8), 5, 21)])
@pytest.mark.parametrize("alloc", [True, False])
def test_outputs_over_later_inputs(D, dims, nev, n, alloc):
    print("project over inputs", dims, nev, n, alloc, flush=True)
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.2, 3)).cuda(), 0.121, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(7)
    V = torch.randn((nev,) + dims[1:] + (3,), dtype=torch.complex128, device="cuda", generator=gen)
    x = torch.randn((n,) + dims + (4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    ref = D.dlma_project(g, 1, V, x, 0)  # separate fields: the same kernels, the same numbers
    buf = torch.empty((n + 1,) + dims + (4, 3), dtype=torch.complex128, device="cuda")
    buf[:n] = x
    (D.dlma_project if alloc else D.dlma_project_noalloc)(g, 1, V, buf[:n], 0, buf[1:])  # one field further
    torch.cuda.synchronize()
    assert torch.equal(buf[1:], ref)
    f, v = x[:, 1].reshape(n, -1, 4, 3).cpu().numpy(), V.reshape(nev, -1, 3).cpu().numpy()
    f = f.transpose(0, 2, 1, 3).reshape(n * 4, -1)
    v = v.reshape(nev, -1)
    tol = (v.shape[1] + nev + 8) * 2.0**-52 * ((np.abs(f) @ np.abs(v).T) @ np.abs(v))
    out = ref[:, 1].reshape(n, -1, 4, 3).cpu().numpy().transpose(0, 2, 1, 3).reshape(n * 4, -1)
    assert np.all(np.abs(out - (f @ v.conj().T) @ v) <= tol)


def test_correlators_of_many_modes_and_sources(D):
    """2065 modes and 254 source groups on 32 timeslices: 2^28 projections and more, in two site
    chunks.  PP_exact of the pseudoscalar is the sum of |tau|^2, all terms positive: relative
    tolerance 2^-52 times the 96 terms of a projection (twice) and the 16 nev ndist of the sum."""
    dims, nev, nd = (32, 2, 4, 4), 2065, 254
    print("many modes", dims, nev, nd, flush=True)
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.2, 3)).cuda(), 0.121, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(9)
    V = torch.randn((32, nev, 2, 4, 4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    x = torch.randn((4 * nd,) + dims + (4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    got = D.dlma_correlators_array(g, 5, V, x)[0, 5]
    for t in range(32):
        f = x[:, t].reshape(4 * nd, 32, 4, 3).transpose(1, 2).reshape(16 * nd, 96)
        ref = (f @ V[t].reshape(nev, 96).conj().T.contiguous()).abs().square().sum().item()
        d = (t - 5) % 32
        assert abs(got[d, 0] - ref) <= (192 + 16 * nev * nd) * 2.0**-52 * ref and abs(got[d, 1]) <= 1e-9 * ref, t


# 16384 modes, the limit of the allocation-free entry: four right-hand sides per pass through its
# array, one-launch coefficients (2^3) and two site chunks of the contraction (14^3); 5 modes on
# 4^2 x 8: passes of 3272 (contraction) and 13104 (allocation-free array)
@pytest.mark.parametrize("dims,nev,n", [((2, 2, 2, 2), 16384, 9), ((2, 14, 14, 14), 16384, 9), ((2, 4, 4, 8), 5, 13110)])
def test_allocation_free_passes(D, dims, nev, n):
    print("passes", dims, nev, n, flush=True)
    g = D.dlma_load_gauge(torch.from_numpy(synth.gauge_field(dims, 0.2, 3)).cuda(), 0.121, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(11)
    V = torch.randn((nev,) + dims[1:] + (3,), dtype=torch.complex128, device="cuda", generator=gen)
    x = torch.randn((n,) + dims + (4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    out = torch.empty_like(x)
    D.dlma_project_noalloc(g, 1, V, x, 1, out)
    torch.cuda.synchronize()
    assert torch.equal(out, D.dlma_project(g, 1, V, x, 1))
    keep = sorted({0, 3, 4, n - 1} | ({3271, 3272, 13103, 13104} if n > 13104 else set()))
    f = x[keep, 1].reshape(len(keep), -1, 4, 3).transpose(1, 2).reshape(4 * len(keep), -1)
    v = V.reshape(nev, -1)
    ref = f - (f @ v.conj().T.contiguous()) @ v
    tol = (v.shape[1] + nev + 8) * 2.0**-52 * ((f.abs() @ v.abs().T.contiguous()) @ v.abs() + f.abs())
    got = out[keep, 1].reshape(len(keep), -1, 4, 3).transpose(1, 2).reshape(4 * len(keep), -1)
    assert bool(((got - ref).abs() <= tol).all())
